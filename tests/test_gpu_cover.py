"""The direct float32 kernels with every output channel in one workgroup (prox_cover.hip) and the weight gradient in blocks
across the taps (wgrad_pipe_kernel<.., COVER>), which give the same bits as the kernels they stand in for: a batch large enough for
them against its samples one by one, and the calls' 64-bit results."""
import dataclasses

import numpy as np
import pytest

from paper_2207_08393_amd import binding as gb
from paper_2207_08393_amd import synth
from paper_2207_08393_amd.runner import ModuleRunner
from tests.gpu_util import rel_l2
from tests.test_gpu_parity import K2, K3, check_module, kernel_policy  # noqa: F401

pytestmark = pytest.mark.gpu


def sample(c, b):
    part = {k: getattr(c, k)[b:b + 1] for k in ("x_true", "S", "M", "y", "x_in")}
    return dataclasses.replace(c, geom=dataclasses.replace(c.geom, B=1), **part)


# 131072 pixels are the least; the last block of 256 is ragged, the number of rows odd; input channels: whole chunks, half of the
# last one, more than half of it; output channels: every count of whole blocks and fours, and some that stay where they were
@pytest.mark.parametrize("chans,taps", [((100, 100), K2), ((36, 96), K2), ((44, 72, 36), K2), ((112, 40, 76), K2), ((68, 68), K2),
                                        ((104, 48), K2), ((36, 36), K3)], ids=lambda v: "x".join(map(str, v)))
def test_batch_and_its_samples_alike(chans, taps, kernel_policy):
    kernel_policy(gb.POLICY_NO_WINOGRAD)
    geom = synth.Geom(1, 2, 2, 1, 5, 285, 46) if taps == K3 else synth.Geom(1, 2, 2, 1, 1, 1425, 46)
    assert geom.B * geom.D * geom.H * geom.W >= 131072 > geom.D * geom.H * geom.W
    relu_chain = [2, chans[0], *chans, 2]
    # alpha = 0: the prox sees x_in itself
    c = synth.make_custom(7, geom, synth.chain_prox(relu_chain, [taps] * (len(relu_chain) - 1)), bias_std=0.1, alpha=0.0)
    print("case cover", chans, taps, flush=True)
    whole = ModuleRunner(c)
    whole.step()
    x, grad = whole.x_out.cpu().numpy(), whole.grad.cpu().numpy()
    parts = []
    for b in range(2):
        r = ModuleRunner(sample(c, b))
        r.step()
        assert np.array_equal(r.x_out.cpu().numpy()[0], x[b])
        parts.append(r.grad.cpu().numpy().astype(np.float64))
    # the loss is a mean over the pixels; sums in float32 over other runs of pixels: 2e-7 seen, a lost or doubled term of one
    # pixel in 1e5 would be 1e-5
    assert rel_l2(grad, 0.5 * (parts[0] + parts[1])) <= 2e-6


# rows and columns that leave blocks of 4 x 4 on both sides, on one, on none; up to sixteen waves of units and small blocks
@pytest.mark.parametrize("ci,co", [(100, 100), (96, 96), (72, 72), (80, 68), (96, 100), (100, 68), (68, 104), (128, 68), (84, 84)])
def test_weight_gradient_in_blocks_across_the_taps(ci, co, kernel_policy):
    kernel_policy(gb.POLICY_NO_WINOGRAD)
    print("case cover weights", ci, co, flush=True)
    check_module(synth.make_custom(9, synth.Geom(1, 2, 2, 1, 1, 11, 46), synth.chain_prox([2, ci, co, 2], [K2] * 3), accel=2.0, centre=2,
                                   bias_std=0.1, alpha=0.8))
