"""Temporal 3x1x1 layers on split operands (prox_time_split.hip) where their segments, runs of frames, chunks and channel blocks end,
against the oracle; their precision as in test_gpu_split.py."""
import numpy as np
import pytest

from oracle import gleam_oracle as og
from paper_2207_08393_amd import binding as gb
from paper_2207_08393_amd import synth
from paper_2207_08393_amd.runner import ModuleRunner
from tests.gpu_util import rel_l2, theta_slices
from tests.test_gpu_parity import KS, KT, TOL, check_module
from tests.test_gpu_split import linear_prox
from tests.test_split_arithmetic import BOUND

pytestmark = pytest.mark.gpu


def cases():
    # (name, geometry, prox): segments are 64 or 128 pixels, chunks 16 input channels, blocks 32 output channels; runs of four
    # frames and more
    yield "every_chunk_count", synth.Geom(2, 1, 2, 5, 1, 6, 12), synth.chain_prox([2, 4, 20, 36, 60, 92, 128, 2], [KS] + [KT] * 5 + [KS])
    yield "two_blocks_a_group", synth.Geom(2, 2, 2, 9, 1, 10, 46), synth.chain_prox([2, 64, 64, 2], [KS, KT, KS])
    yield "three_blocks", synth.Geom(2, 1, 2, 6, 1, 6, 20), synth.chain_prox([2, 36, 96, 68, 2], [KS, KT, KT, KS])
    yield "one_frame", synth.Geom(2, 2, 2, 1, 1, 6, 10), synth.chain_prox([2, 32, 64, 2], [KS, KT, KS], has_bias=0)
    yield "two_frames_l1", synth.Geom(2, 1, 2, 2, 1, 8, 8), synth.chain_prox([2, 24, 100, 2], [KS, KT, KS], loss_kind=1)
    yield "runs_end_ragged", synth.Geom(2, 1, 2, 11, 1, 4, 6), synth.chain_prox([2, 16, 16, 16, 2], [KT] * 4)
    yield "frames_a_multiple_of_a_run", synth.Geom(2, 2, 2, 16, 1, 8, 16), synth.chain_prox([2, 48, 48, 2], [KS, KT, KS])
    yield "slices", synth.Geom(2, 1, 2, 5, 3, 6, 10), synth.chain_prox([2, 12, 40, 2], [KS, KT, KS])
    yield "skips_and_masks", synth.Geom(2, 1, 2, 7, 1, 10, 20), synth.resblock_prox(36, 2, KT)
    yield "skips_and_masks_64", synth.Geom(2, 2, 2, 5, 1, 6, 10), synth.resblock_prox(64, 1, KT, 0)
    yield "wider_than_the_kernel", synth.Geom(2, 1, 2, 3, 1, 6, 8), synth.chain_prox([2, 132, 36, 2], [KS, KT, KS])


@pytest.mark.parametrize("name,geom,prox", list(cases()), ids=[c[0] for c in cases()])
def test_time_layers_on_split_operands_match_oracle(name, geom, prox):
    c = synth.make_custom(81, geom, prox, accel=2.0, centre=2, bias_std=0.1, alpha=0.8)
    print("case time split", name, flush=True)
    r = ModuleRunner(c)
    gb.gleam_profile_begin()
    r.step()
    ran = {n: round(m / f, 3) for n, f, _, _, m in gb.gleam_profile_end() if n.endswith("_t3") and "_2to" not in n and "to2_" not in n}
    # more than 128 input channels: the forward launch by the kernels on the float32 matrix cores
    assert ran and ran == {n: 1.0 if n.startswith("conv_fwd_132to") else 6.0 for n in ran}, ran
    assert name != "wider_than_the_kernel" or set(ran) == {"conv_fwd_132to36_t3", "conv_dgrad_36to132_t3", "conv_wgrad_132to36_t3"}
    check_module(c)


@pytest.mark.parametrize("chans", [(32, 32, 32), (36, 60, 20), (100, 100), (64, 64, 64), (128, 128)], ids=lambda v: "x".join(map(str, v)))
def test_time_layers_keep_the_precision_of_float32(chans):
    """Output and gradients of every layer within the bound of test_gpu_split.py of the 64-bit oracle."""
    prox = linear_prox([2, *chans, 2], KT)
    for seed in (1, 2):
        c = synth.make_custom(seed, synth.Geom(2, 1, 2, 6, 1, 10, 46), prox, accel=2.0, centre=2, bias_std=0.1, alpha=0.8)
        print("case time precision", chans, seed, flush=True)
        r = ModuleRunner(c)
        r.step()
        x_out, loss, grad = r.results()
        f = og.module_fwd(c.geom, c.prox, c.x_in, c.S, c.M, c.y, c.alpha, c.theta, c.x_true)
        g = og.module_bwd(c.prox, c.theta, f)
        errs = {"x_out": rel_l2(x_out, f["x_out"]), "loss": abs(loss / f["loss"] - 1)}
        errs.update({f"{layer}{kind}": rel_l2(grad[part], g[part]) for layer, kind, part in theta_slices(c.prox)})
        print({name: float(f"{e:.1e}") for name, e in errs.items()}, flush=True)
        assert max(errs.values()) <= BOUND, errs


@pytest.mark.parametrize("nf", [36, 64])
def test_an_overflow_stays_visible_through_time_layers(nf):
    """A spot of 1e30 and weights of 1e10: pixels whose exact value is beyond float32 leave as infinity or NaN through the ReLUs."""
    geom = synth.Geom(2, 1, 2, 10, 1, 8, 16)
    for prox in (synth.chain_prox([2, nf, nf, 2], [KS, KT, KS]), synth.resblock_prox(nf, 1, KT)):
        c = synth.make_custom(82, geom, prox, accel=2.0, centre=2, bias_std=0.1, alpha=0.0)
        c.theta = np.abs(c.theta)
        for layer, kind, part in theta_slices(prox):
            if layer == 2 and kind == "W":
                c.theta[part] *= 1e10
        c.x_in[:, 2, :, 4:6, 5:8] = 1e30
        z = og.prox_fwd(prox.layers, c.theta.astype(np.float64), c.x_in.astype(np.complex128))[0][-1]
        over = (np.abs(z) > np.finfo(np.float32).max).any(-1)
        assert over.any() and not over[:, 7:].any()   # four temporal layers carry the spot of frame 2 to frame 6
        print("case time overflow", nf, flush=True)
        r = ModuleRunner(c)
        r.fwd()
        x_out, loss, _ = r.results()
        assert not np.isfinite(x_out[over]).any() and not np.isfinite(loss)
        assert rel_l2(x_out[:, 7:], og.channels_to_complex(z)[:, 7:]) <= TOL
