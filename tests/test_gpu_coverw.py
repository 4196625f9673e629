"""The weight gradient of 68 to 124 x 68 to 100 channels (prox_coverw.hip) gives the bits of wgrad_pipe_kernel: layer 2 of [2, ci, co, 2]
and of [2, ci, 128, 2], whose further channels have zero weights and which goes by nine taps a wave.  The gradient that reaches
layer 2 is the same bits in both: the reference image is 2^40 in size, so that z - x is -x whatever z was rounded to, and layer 3 has
one weight for each of its input channels, so that nothing is summed there."""
import dataclasses

import numpy as np
import pytest

from paper_2207_08393_amd import binding as gb
from paper_2207_08393_amd import synth
from paper_2207_08393_amd.runner import ModuleRunner
from tests.test_gpu_parity import K2, kernel_policy  # noqa: F401

pytestmark = pytest.mark.gpu


# Chunks per workgroup: none or one (few), six or seven with a ragged one in each row (many); rows of whole chunks; row taps in depth
# and in time, at their ends too.  Waves: 14 and 2 of small blocks (100 x 100), no small blocks (96 x 96), waves with neither (68 x 72)
@pytest.mark.parametrize("ci,co", [(100, 100), (96, 96), (72, 68), (100, 124)])
@pytest.mark.parametrize("geom,taps", [(synth.Geom(1, 1, 2, 1, 1, 2, 20), K2), (synth.Geom(1, 3, 2, 1, 1, 285, 46), K2), (synth.Geom(1, 1, 2, 1, 1, 33, 64), K2),
                                       (synth.Geom(1, 2, 2, 1, 4, 36, 46), (1, 3, 1, 3)), (synth.Geom(1, 2, 2, 5, 1, 36, 46), (3, 1, 1, 3))],
                         ids=["few", "many", "whole", "depth", "time"])
def test_weight_gradient_has_the_bits_of_the_pipelined_kernel(ci, co, geom, taps, kernel_policy):
    kernel_policy(gb.POLICY_NO_WINOGRAD)
    print("case coverw", ci, co, taps, geom, flush=True)
    rng = np.random.default_rng(ci + co)
    ref = (rng.uniform(1, 2, (2,) + geom.image_shape) * rng.choice((-1.0, 1.0), (2,) + geom.image_shape) * 2.0 ** 40).astype(np.float32)
    w3 = np.zeros((2, 9, 128), np.float32)
    w3[np.arange(128) % 2, np.arange(128) * 5 % 9, np.arange(128)] = rng.standard_normal(128)
    w3[:, :, co:] = 0
    w2, b2 = rng.standard_normal((128, 9, ci)).astype(np.float32) / np.float32(np.sqrt(9 * ci)), rng.standard_normal(128).astype(np.float32)
    w2[co:], b2[co:] = 0, 0
    w1, b1 = rng.standard_normal((ci, 9, 2)).astype(np.float32), rng.standard_normal(ci).astype(np.float32)
    grads = []
    for n in (co, 128):
        c = synth.make_custom(19, geom, synth.chain_prox([2, ci, n, 2], [taps] * 3), alpha=0.0)
        theta = np.concatenate([w1.ravel(), b1, w2[:n].ravel(), b2[:n], w3[:, :, :n].ravel(), np.zeros(2, np.float32)])
        r = ModuleRunner(dataclasses.replace(c, x_true=ref[0] + 1j * ref[1], theta=theta))
        r.step()
        g = r.grad.cpu().numpy()[ci * 19:]
        grads.append((g[:n * 9 * ci].reshape(n, -1)[:co], g[n * 9 * ci:][:co]))
    # (two rows: each row tap of the layers above and below but the middle one sees one of them)
    assert np.all(np.isfinite(grads[0][0])) and np.count_nonzero(grads[0][0]) > (0.9 if geom.H > 2 else 0.9 / 2 ** 2) * grads[0][0].size
    assert all(np.array_equal(a, b) for a, b in zip(*grads))
