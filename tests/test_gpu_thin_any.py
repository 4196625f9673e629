"""The two-channel-input convolution on the matrix cores (prox_thin.hip) for channel counts that are no whole blocks of 32 gives the
bits of the vector kernel it stands in for (conv_thin_in_kernel), in the forward pass and as the data gradient of the last layer."""
import numpy as np
import pytest

from paper_2207_08393_amd import binding as gb
from paper_2207_08393_amd import synth
from paper_2207_08393_amd.runner import ModuleRunner
from tests.test_gpu_parity import K2, K3, kernel_policy  # noqa: F401

pytestmark = pytest.mark.gpu


# one, two, three and four blocks of 32 channels, the last of four channels, of 28, whole; rows of one ragged segment, of whole ones and
# of both; planes of one row; slices at both ends; 8192 pixels and few more, where it begins, and fewer
@pytest.mark.parametrize("n", [8, 28, 36, 60, 68, 96, 100, 124])
@pytest.mark.parametrize("geom,k", [(synth.Geom(1, 18, 2, 1, 1, 10, 46), K2), (synth.Geom(1, 128, 2, 1, 1, 1, 64), K2), (synth.Geom(1, 12, 2, 1, 1, 37, 20), K2),
                                    (synth.Geom(1, 9, 2, 1, 3, 7, 46), K3), (synth.Geom(1, 2, 2, 1, 1, 10, 46), K2)],
                         ids=["ragged", "row", "narrow", "volume", "below"])
@pytest.mark.parametrize("dtype", [0, 1])
def test_any_channels_have_the_bits_of_the_vector_kernel(n, geom, k, dtype, kernel_policy):
    if k == K3:
        n = min(n, 104)   # (more have no weight gradient in float32)
    if dtype and n % 8:
        n += 4 if n % 32 == 4 else -4   # (multiples of 8)
    print("case thin any", n, k, geom, dtype, flush=True)
    check_bits(geom, [synth.chain_prox([2, n, n, 2], [k] * 3, dtype=dtype), synth.resblock_prox(n, 1, k, dtype=dtype)], kernel_policy)


def check_bits(geom, proxes, kernel_policy):
    # the first layer with and without a ReLU behind it; the last one's data gradient with a mask and an addition (residual), with a
    # mask alone (chain)
    for prox in proxes:
        c = synth.make_custom(95, geom, prox, accel=2.0, centre=2, bias_std=0.1, alpha=0.8)
        got = []
        for policy in (gb.POLICY_NO_WINOGRAD, gb.POLICY_NO_WINOGRAD | gb.POLICY_NO_THIN_MFMA):
            kernel_policy(policy)
            r = ModuleRunner(c)
            r.step()
            got.append((r.x_out.cpu().numpy(), r.grad.cpu().numpy(), r.loss.cpu().numpy()))
        assert np.all(np.isfinite(got[0][1])) and np.count_nonzero(got[0][1]) > 0
        assert all(np.array_equal(a, b) for a, b in zip(*got))


# 27 taps with a mask: from 20480 pixels on; float32 rows that begin in the middle of 32 bytes, with a mask: the last of the vector
# kernel's and the first beyond its line, 48 MB
@pytest.mark.parametrize("geom,k,n,dtype", [(synth.Geom(1, 22, 2, 1, 3, 7, 46), K3, 8, 1), (synth.Geom(1, 22, 2, 1, 3, 7, 46), K3, 36, 0),
                                            (synth.Geom(1, 22, 2, 1, 3, 7, 46), K3, 100, 0), (synth.Geom(1, 4, 2, 1, 1, 500, 96), K2, 60, 0),
                                            (synth.Geom(1, 4, 2, 1, 1, 521, 96), K2, 60, 0), (synth.Geom(1, 3, 2, 1, 1, 500, 64), K2, 124, 0),
                                            (synth.Geom(1, 3, 2, 1, 1, 505, 64), K2, 124, 0)])
def test_masked_calls_have_the_bits_of_the_vector_kernel(geom, k, n, dtype, kernel_policy):
    print("case thin masked", n, k, geom, dtype, flush=True)
    check_bits(geom, [synth.chain_prox([2, n, 8, n, 2], [k] * 4, dtype=dtype), synth.resblock_prox(n, 1, k, dtype=dtype)], kernel_policy)
