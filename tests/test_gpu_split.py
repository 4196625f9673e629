"""The split-operand 3x3 / 3x3x3 kernels (prox_split.hip) where their blocks, chunks and channel groups end: module steps
against the oracle at the float32 tolerance, per layer and per element (tests/test_gpu_parity.py check_module)."""
import numpy as np
import pytest

from oracle import gleam_oracle as og
from paper_2207_08393_amd import synth
from tests.gpu_util import ModuleRunner, rel_l2, theta_slices
from tests.test_gpu_parity import K2, K3, TOL, check_module

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


@pytest.mark.parametrize("prox", [synth.chain_prox([2, 24, 24, 24, 2], [K2] * 4), synth.chain_prox([2, 100, 100, 2], [K2] * 3),
                                  synth.resblock_prox(36, 1), synth.resblock_prox(64, 2), synth.chain_prox([2, 20, 32, 2], [K3] * 3)],
                         ids=["chain24", "chain100", "res36", "res64", "chain20_32_volume"])
def test_an_overflow_stays_visible(prox):
    """A spot of 1e30 in the image and layer-2 weights of 1e10 (all weights positive): every output pixel whose exact value is
    beyond float32 must come out as infinity or NaN through the ReLUs and the skips that follow, and so must the loss; the
    rest of the image is as ever."""
    n_dim = 3 if prox.layers[0].kd == 3 else 2
    geom = synth.Geom(n_dim, 1, 2, 1, 4 if n_dim == 3 else 1, 32, 46)
    c = synth.make_custom(103, geom, prox, accel=2.0, centre=2, bias_std=0.1, alpha=0.0)   # alpha = 0: the prox sees x_in itself
    c.theta = np.abs(c.theta)
    for layer, kind, part in theta_slices(prox):
        if layer == 2 and kind == "W":
            c.theta[part] *= 1e10
    c.x_in[..., 4:6, 5:8] = 1e30
    z = og.prox_fwd(prox.layers, c.theta.astype(np.float64), c.x_in.astype(np.complex128))[0][-1]
    over = (np.abs(z) > np.finfo(np.float32).max).any(-1)
    assert 30 <= over[0, 0, 0].sum() <= 200
    print("case overflow", [l.cout for l in prox.layers], flush=True)
    r = ModuleRunner(c)
    r.fwd()
    x_out, loss, _ = r.results()
    assert not np.isfinite(x_out[over]).any() and not np.isfinite(loss)
    far = np.s_[..., 20:, :]
    assert rel_l2(x_out[far], og.channels_to_complex(z)[far]) <= TOL


def test_a_nan_weight_stays_visible():
    """Every bit pattern of NaN among the weights, also the one whose rounding to bfloat16 by integers wraps around to zero."""
    geom = synth.Geom(2, 1, 2, 1, 1, 12, 20)
    prox = synth.chain_prox([2, 24, 24, 2], [K2] * 3)
    for bits in (0x7fc00000, 0xffc00000, 0x7fffffff, 0xffffffff, 0x7f800001):
        c = synth.make_custom(104, geom, prox, accel=2.0, centre=2, bias_std=0.1, alpha=0.8)
        at = next(part.start for layer, kind, part in theta_slices(prox) if layer == 2) + 24 * 4   # centre tap, first channels
        c.theta.view(np.uint32)[at] = bits
        print("case NaN weight", hex(bits), flush=True)
        r = ModuleRunner(c)
        r.step()
        x_out, loss, grad = r.results()
        assert not np.isfinite(x_out).any() and not np.isfinite(loss) and np.isnan(grad).any()
