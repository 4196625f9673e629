"""The direct convolution with two output channels (prox_pair.hip) gives the bits of the direct convolution in blocks of 32 that it
stands in for: layer 2 of a network [2, n, 2] against the first two channels of layer 2 of [2, n, 4, 2]."""
import numpy as np
import pytest

from paper_2207_08393_amd import binding as gb
from paper_2207_08393_amd import synth
from paper_2207_08393_amd.runner import ModuleRunner
from tests.test_gpu_parity import K2, K3, KT, check_module, kernel_policy  # noqa: F401

pytestmark = pytest.mark.gpu


def align(n):
    return (n + 255) // 256 * 256


# channel counts of one chunk of 8, of 16, ragged ones with four and with eight channels in the last chunk; pixels just above the
# 32768 it begins at, no multiple of a wave's 64 or a workgroup's 256; planes smaller than a wave; taps along one axis only
@pytest.mark.parametrize("n", [8, 12, 20, 24, 36, 100])
@pytest.mark.parametrize("geom,k", [(synth.Geom(2, 73, 2, 1, 1, 10, 46), K2), (synth.Geom(3, 23, 2, 1, 6, 12, 20), K3), (synth.Geom(2, 111, 2, 5, 1, 6, 10), KT),
                                    (synth.Geom(2, 1366, 2, 1, 1, 4, 6), K2), (synth.Geom(1, 6, 2, 1, 1, 97, 64), K2), (synth.Geom(2, 82, 2, 1, 1, 20, 20), (1, 1, 1, 1)),
                                    (synth.Geom(2, 1, 2, 1, 1, 4, 6), K2)],
                         ids=["ragged", "volume", "time", "planes", "many", "one_tap", "below"])
def test_two_output_channels_have_the_bits_of_the_direct_kernel(n, geom, k, kernel_policy):
    kernel_policy(gb.POLICY_NO_WINOGRAD)
    taps = int(np.prod(k))
    rng = np.random.default_rng(n)
    w1, b1 = rng.standard_normal((n, taps, 2)), rng.standard_normal(n)
    w2, b2 = rng.standard_normal((4, taps, n)) / np.sqrt(taps * n), rng.standard_normal(4)
    first = synth.ConvLayer(2, n, *k, 0, 0, 1, -1)
    print("case pair", n, k, geom, flush=True)
    for relu_in in (0, 1):
        two = synth.ProxDesc([first, synth.ConvLayer(n, 2, *k, relu_in, 0, 1, -1)])
        four = synth.ProxDesc([first, synth.ConvLayer(n, 4, *k, relu_in, 0, 1, -1), synth.ConvLayer(4, 2, *k, 0, 0, 1, -1)])
        c = synth.make_custom(91, geom, two, accel=2.0, centre=2, alpha=0.0)   # the prox sees x_in itself
        a, b = ModuleRunner(c, theta=np.concatenate([v.ravel() for v in (w1, b1, w2[:2], b2[:2])])), None
        a.fwd()
        c.prox = four
        b = ModuleRunner(c, theta=np.concatenate([v.ravel() for v in (w1, b1, w2, b2, np.zeros((2, taps, 4)), np.zeros(2))]))
        b.fwd()
        q = a.x_out.numel() // 2
        at = align(q * 8) + align(q * n * 4)
        t2 = b.saved[at:at + q * 16].cpu().numpy().view(np.float32).reshape(q, 4)
        got = a.x_out.cpu().numpy().reshape(q, 2)
        assert np.all(np.isfinite(got)) and np.abs(got).max() > 0.1
        assert np.array_equal(got, t2[:, :2]), relu_in


@pytest.mark.parametrize("prox", [synth.resblock_prox(20, 1), synth.chain_prox([2, 12, 100, 2], [K2] * 3, loss_kind=1), synth.chain_prox([2, 8, 8, 2], [K3] * 3, has_bias=0)],
                         ids=["res20", "chain100", "volume8"])
def test_networks_ending_in_it_match_the_oracle(prox):
    geom = synth.Geom(3, 41, 2, 1, 4, 10, 20) if prox.layers[0].kd == 3 else synth.Geom(2, 60, 2, 1, 1, 12, 46)
    check_module(synth.make_custom(92, geom, prox, accel=2.0, centre=2, bias_std=0.1, alpha=0.8))
