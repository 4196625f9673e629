"""The direct float32 kernels with every output channel in one workgroup (prox_cover.hip) and the weight gradient in blocks
across the taps (prox_coverw.hip), which give the same bits as the kernels they stand in for: a batch large enough for
them against its samples one by one, and the calls' 64-bit results."""
import dataclasses

import numpy as np
import pytest

from paper_2207_08393_amd import binding as gb
from paper_2207_08393_amd import synth
from paper_2207_08393_amd.runner import ModuleRunner
from tests.gpu_util import rel_l2, theta_slices
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


# Residual networks: ReLU on the operands, a tensor added behind the convolution, its gradient added behind a mask; no bias.  Fours and
# half a last chunk of input channels (100), whole blocks (96), half a chunk (40), more than half of one (36, 68), three taps deep
@pytest.mark.parametrize("nf,taps,has_bias", [(100, K2, 1), (100, K2, 0), (96, K2, 1), (40, K2, 0), (36, K2, 1), (68, K2, 1), (36, K3, 0)],
                         ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_residual_batch_and_its_samples_alike(nf, taps, has_bias, kernel_policy):
    kernel_policy(gb.POLICY_NO_WINOGRAD)
    geom = synth.Geom(1, 2, 2, 1, 5, 285, 46) if taps == K3 else synth.Geom(1, 2, 2, 1, 1, 1425, 46)
    c = synth.make_custom(13, geom, synth.resblock_prox(nf, 1, taps, has_bias), bias_std=0.1, alpha=0.0)
    print("case cover residual", nf, taps, has_bias, flush=True)
    whole = ModuleRunner(c)
    whole.step()
    x, grad = whole.x_out.cpu().numpy(), whole.grad.cpu().numpy()
    parts = []
    for b in range(2):
        r = ModuleRunner(sample(c, b))
        r.step()
        assert np.array_equal(r.x_out.cpu().numpy()[0], x[b])
        parts.append(r.grad.cpu().numpy().astype(np.float64))
    for layer, kind, part in theta_slices(c.prox):   # (the bound of the test above; layer by layer, so that none hides)
        assert rel_l2(grad[part], 0.5 * (parts[0] + parts[1])[part]) <= 2e-6, (layer, kind)


@pytest.mark.parametrize("ci,co", [(100, 100), (96, 96), (72, 72), (100, 68), (68, 104), (84, 84)])
def test_weight_gradient_has_the_bits_of_the_kernel_it_stands_in_for(ci, co, kernel_policy):
    """Layer 2 of [2, ci, co, 2] and of [2, ci, 128, 2], whose further channels have zero weights: 128 output channels go by nine taps a
    wave.  The gradient that reaches layer 2 is the same bits in both: the reference image is 2^40 in size, so that z - x is -x
    whatever z was rounded to, and layer 3 has one weight for each of its input channels, so that nothing is summed there."""
    kernel_policy(gb.POLICY_NO_WINOGRAD)
    print("case cover weight bits", ci, co, flush=True)
    geom = synth.Geom(1, 2, 2, 1, 1, 11, 46)
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
        c = synth.make_custom(17, geom, synth.chain_prox([2, ci, n, 2], [K2] * 3), alpha=0.0)
        theta = np.concatenate([w1.ravel(), b1, w2[:n].ravel(), b2[:n], w3[:, :, :n].ravel(), np.zeros(2, np.float32)])
        r = ModuleRunner(dataclasses.replace(c, x_true=ref[0] + 1j * ref[1], theta=theta))
        r.step()
        g = r.grad.cpu().numpy()[ci * 19:]
        grads.append((g[:n * 9 * ci].reshape(n, -1)[:co], g[n * 9 * ci:][:co]))
    assert np.all(np.isfinite(grads[0][0])) and np.count_nonzero(grads[0][0]) > 0.9 * grads[0][0].size
    assert all(np.array_equal(a, b) for a, b in zip(*grads))
