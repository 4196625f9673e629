"""Launches that serve several layers at once: the partial sums of a backward pass (reduce_partials_kernel)."""
import pytest

from paper_2207_08393_amd import binding as gb
from paper_2207_08393_amd import synth
from paper_2207_08393_amd.runner import ModuleRunner
from tests.test_gpu_parity import K2, check_module

pytestmark = pytest.mark.gpu


def reduces(records):
    return sum(r[0] == "wgrad_reduce" for r in records)


# twenty layers: more than a batch of jobs holds; layers with many and with few sums together; partial sums that are no multiples of 4 floats, with and without bias; sums of more than the 8 MB
# that wait (128 x 128 channels, 3x3, eight splits and more: 4.7 MB and more a layer)
@pytest.mark.parametrize("prox,launches", [(synth.chain_prox([2] + [8] * 19 + [2], [K2] * 20), 2),
                                           (synth.chain_prox([2, 12, 64, 64, 20, 2], [K2] * 5), 1),
                                           (synth.chain_prox([2, 9, 7, 2], [K2] * 3, has_bias=0), 1),
                                           (synth.chain_prox([2, 128, 128, 128, 128, 2], [K2] * 5), 2)],
                         ids=["twenty_layers", "mixed", "odd", "beyond_the_limit"])
def test_partial_sums_of_several_layers(prox, launches):
    c = synth.make_custom(71, synth.Geom(2, 1, 2, 1, 1, 24, 46), prox, accel=2.0, centre=2, bias_std=0.1, alpha=0.5)
    print("case partial sums", [l.cout for l in prox.layers], flush=True)
    c.theta *= np.float32(0.6 if len(prox.layers) > 10 else 1.0)
    r = ModuleRunner(c)
    gb.gleam_profile_begin()
    r.step()
    assert reduces(gb.gleam_profile_end()) == launches
    check_module(c)
