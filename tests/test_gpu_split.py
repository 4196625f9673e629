"""The split-operand 3x3 / 3x3x3 kernels (prox_split.hip) where their blocks, chunks and channel groups end: module steps
against the oracle at the float32 tolerance, per layer and per element (tests/test_gpu_parity.py check_module)."""
import pytest

from paper_2207_08393_amd import synth
from tests.test_gpu_parity import K2, K3, check_module

pytestmark = pytest.mark.gpu


def cases():
    # (name, geometry, prox): blocks are 8 x 32 pixels x 32 output channels, chunks 16 input channels
    yield "one_pixel_past_a_block", synth.Geom(2, 2, 2, 1, 1, 10, 46), synth.resblock_prox(32, 1)
    yield "narrower_and_lower_than_a_block", synth.Geom(2, 1, 2, 1, 1, 4, 6), synth.resblock_prox(64, 1)
    yield "whole_blocks_only", synth.Geom(2, 1, 2, 1, 1, 16, 32), synth.resblock_prox(32, 2)
    yield "odd_rows_batched", synth.Geom(1, 1, 2, 1, 3, 9, 64), synth.resblock_prox(16, 1)
    for h in (1, 2, 3):   # fewer rows than a thread's four, between slices that must stay as they are
        yield f"{h}_rows_many_slices", synth.Geom(1, 2, 2, 1, 5, h, 46), synth.resblock_prox(36, 1)
    yield "2_rows_sign_words", synth.Geom(1, 1, 2, 1, 6, 2, 64), synth.chain_prox([2, 32, 64, 32, 2], [K2] * 4)
    yield "ragged_channels", synth.Geom(2, 1, 2, 1, 1, 12, 20), synth.chain_prox([2, 36, 12, 60, 2], [K2] * 4)
    yield "ragged_chunk_many_blocks", synth.Geom(2, 2, 2, 3, 1, 32, 96), synth.resblock_prox(20, 2)
    yield "narrow_between_wide", synth.Geom(2, 1, 2, 1, 1, 20, 46), synth.chain_prox([2, 64, 4, 64, 2], [K2] * 4)
    yield "wide_and_ragged", synth.Geom(2, 1, 2, 1, 1, 10, 46), synth.chain_prox([2, 100, 128, 68, 2], [K2] * 4)
    yield "one_slice", synth.Geom(2, 1, 2, 1, 1, 10, 46), synth.chain_prox([2, 32, 32, 2], [K3] * 3)
    yield "slices_ragged_channels", synth.Geom(3, 2, 2, 1, 4, 10, 46), synth.chain_prox([2, 20, 36, 2], [K3] * 3)
    yield "plane_then_volume", synth.Geom(3, 1, 2, 1, 6, 12, 20), synth.chain_prox([2, 32, 32, 32, 2], [K2, K3, K2, K3])


@pytest.mark.parametrize("name,geom,prox", list(cases()), ids=[c[0] for c in cases()])
def test_split_operand_kernels_match_oracle(name, geom, prox):
    c = synth.make_custom(101, geom, prox, accel=2.0, centre=2, bias_std=0.1, alpha=0.8)
    print("case split", name, flush=True)
    check_module(c)
