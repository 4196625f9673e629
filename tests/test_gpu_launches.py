"""Launches that serve several layers or modules at once, and small calls that need one launch fewer: the partial sums of a backward
pass (reduce_partials_kernel), the weights of several modules (prepare_weights_kernel), the loss in one workgroup."""
import numpy as np
import pytest

from paper_2207_08393_amd import binding as gb
from paper_2207_08393_amd import synth
from paper_2207_08393_amd.runner import GreedyRunner, ModuleRunner, to_complex
from tests.test_gpu_parity import K2, K3, KS, KT, check_module, kernel_policy  # noqa: F401
from tests.test_gpu_split import modules_by_hand

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


@pytest.mark.parametrize("W,H,loss_kind", [(64, 256, 0), (64, 256, 1), (64, 257, 0), (20, 20, 1), (64, 33, 0), (64, 128, 0), (64, 128, 1), (64, 129, 1)])
def test_loss_in_one_workgroup_and_in_many(W, H, loss_kind):
    """8192 pixels are the most of one workgroup; sizes that its 1024 threads with four pixels each divide and such that they do not."""
    prox = synth.chain_prox([2, 8, 2], [K2] * 2, loss_kind=loss_kind)
    c = synth.make_custom(72, synth.Geom(1, 1, 2, 1, 1, H, W), prox, accel=2.0, centre=2, bias_std=0.1, alpha=0.5)
    print("case loss", W, H, loss_kind, flush=True)
    check_module(c)


@pytest.mark.parametrize("prox", [synth.resblock_prox(36, 1), synth.chain_prox([2, 64, 64, 2], [KS, KT, KS]), synth.chain_prox([2, 16, 16, 2], [K2] * 3, dtype=1)],
                         ids=["res36", "time64", "bf16"])
def test_weights_of_several_modules_at_once(prox):
    """Nineteen modules, more than the sixteen whose weights are made at once: the chain is the same bits as its modules one by one."""
    c = synth.make_custom(73, synth.Geom(2, 1, 2, 2, 1, 10, 12), prox, accel=2.0, centre=2, bias_std=0.1, alpha=0.5)
    rng = np.random.default_rng(3)
    thetas = [(0.5 * c.theta * rng.uniform(0.5, 1, c.theta.size)).astype(np.float32) for _ in range(19)]
    print("case modules at once", [l.cout for l in prox.layers], flush=True)
    r = GreedyRunner(c, thetas, 1e-3)
    x = r.infer()
    part, tmp = r.x0, r.x0.clone()
    for i in range(19):
        out = tmp if i % 2 == 0 else r.x_tmp
        gb.gleam_module_fwd(r.geom, r.prox, part, r.S, r.M, r.y, r.alpha, r.theta[i], r.x_ref, out, r.losses, r.saved, r.ws)
        part = out
    assert np.array_equal(x, to_complex(part))


@pytest.mark.parametrize("prox", [synth.resblock_prox(36, 1), synth.chain_prox([2, 9, 7, 2], [K2] * 3), synth.chain_prox([2, 16, 16, 2], [K3] * 3, dtype=1),
                                  synth.chain_prox([2] + [12] * 17 + [2], [K2] * 18), synth.chain_prox([2, 64, 36, 2], [KS, KT, KS])],
                         ids=["res36", "odd", "bf16_volume", "eighteen_layers", "time64"])
def test_greedy_iteration_of_many_modules_and_the_same_calls_by_hand(prox, kernel_policy):
    """Ten modules, more than the eight whose weights of both passes are made at once; eighteen layers, whose two passes take a launch
    each.  Bit for bit the modules one by one, whose weights are made call by call."""
    kernel_policy(gb.POLICY_NO_WINOGRAD)
    geom = synth.Geom(3, 1, 2, 1, 8, 10, 12) if prox.layers[0].kd == 3 else synth.Geom(2, 1, 2, 4 if prox.layers[1].kt == 3 else 1, 1, 20, 46)
    c = synth.make_custom(74, geom, prox, accel=2.0, centre=2, bias_std=0.1, alpha=0.5)
    thetas = [(c.theta * np.float32(0.5 + 0.04 * i)).astype(np.float32) for i in range(10)]
    print("case greedy many", [l.cout for l in prox.layers], flush=True)
    r = GreedyRunner(c, thetas, 1e-3)
    r.iteration(1)
    assert all(np.array_equal(a, b) for a, b in zip(r.results(), modules_by_hand(c, thetas, 1e-3)))
