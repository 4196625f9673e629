"""The operator's sweeps at the edges of their tiles, against the oracle's explicit transforms.

A value passes 2 d transforms of at most two butterflies each; a butterfly of R <= 32 points is at most log2(R) + 2 roundings
deep, its twiddles one more.  With roundings of 2^-24 / sqrt(3) that are independent of one another, three transformed axes give
sqrt(6 * 2 * 8) * 3.4e-8 = 3.4e-7; the bound is three times that (measured 1.0e-7 to 1.8e-7)."""
import dataclasses

import numpy as np
import pytest

from oracle import gleam_oracle as og
from paper_2207_08393_amd import binding as gb
from paper_2207_08393_amd import synth
from paper_2207_08393_amd.runner import ModuleRunner
from tests.gpu_util import assert_image_close, run_sense_normal
from tests.test_gpu_parity import kernel_policy  # noqa: F401

pytestmark = pytest.mark.gpu
TOL = 1e-6
LENGTHS = (4, 6, 8, 10, 12, 16, 20, 24, 32, 46, 64, 96, 128, 160, 192, 256, 320, 368, 640)


def inputs(nd, B, C, T, D, H, W, centred, seed):
    r = np.random.default_rng(seed)
    z = lambda *s: (r.standard_normal(s) + 1j * r.standard_normal(s)).astype(np.complex64)  # noqa: E731
    return (synth.Geom(nd, B, C, T, D, H, W, centred=centred), z(B, T, D, H, W), z(B, C, D, H, W),
            (r.random((B, T, D, H, W)) < 0.4).astype(np.uint8), z(B, C, T, D, H, W))


def check(geom, x, S, M, y):
    import torch
    print("case", geom, flush=True)
    cen = bool(geom.centred)
    got = run_sense_normal(geom, x, S, M)
    assert_image_close(got, og.sense_normal(x, S, M, geom.ndim_fft, centred=cen), TOL, "A^H A x")
    g = gb.gleam_geom(geom.ndim_fft, geom.centred, *(x.shape[:1] + S.shape[1:2] + x.shape[1:]))
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    real = lambda a: torch.view_as_real(dev(a)).contiguous()  # noqa: E731
    out, ws = torch.empty(x.shape + (2,), device="cuda"), torch.empty(
        int(gb.gleam_workspace_bytes(g, None)[0]) + x.nbytes + 512, dtype=torch.uint8, device="cuda")
    gb.gleam_sense_adjoint(g, real(S), dev(M), real(y), out, ws)
    got = torch.view_as_complex(out).cpu().numpy()
    ref = og.sense_adjoint(y.astype(np.complex128) * M[:, None], S, M, geom.ndim_fft, centred=cen)
    assert_image_close(got, ref, TOL, "A^H y")


# coils and rows that leave a tile of 16, 8 or 64 lines ragged: one coil, a full tile, one more, more than 64
@pytest.mark.parametrize("coils", [1, 3, 16, 17, 65])
@pytest.mark.parametrize("W", [20, 32, 46, 64, 160, 368, 640])
def test_rows_and_coils_that_do_not_fill_a_tile(W, coils):
    for nd, H in ((2, 6), (1, 19)):
        check(*inputs(nd, 1, coils, 2, 1, H, W, coils % 2, W + coils))


# Tiles of 128 rows of 8 to 12 points and of 64 rows of 32, which calls of 131072 and of 32768 coil rows and more take, on both sides
# of these lines: coils that fill a tile, leave it ragged, need a second one; frames that end inside a tile
@pytest.mark.parametrize("W,coils,D,H", [(8, 2, 1092, 10), (8, 2, 1093, 10), (8, 16, 137, 10), (10, 3, 729, 10), (12, 127, 4, 46),
                                         (12, 128, 4, 46), (12, 129, 4, 46), (32, 2, 273, 10), (32, 2, 274, 10), (32, 63, 1, 128),
                                         (32, 64, 1, 96), (32, 65, 1, 96), (32, 129, 1, 46)])
def test_short_rows_and_coils_that_do_not_fill_a_tile(W, coils, D, H):
    check(*inputs(2, 2, coils, 3, D, H, W, coils % 2, W + coils))


# rows of 640 points with so few coils that a tile takes three rows of them, or two: rows that do not divide by that
@pytest.mark.parametrize("coils", [1, 2, 3, 4, 5])
def test_long_rows_of_few_coils(coils):
    for nd, D, H in ((2, 1, 20), (3, 4, 10)):
        check(*inputs(nd, 2, coils, 2, D, H, 640, coils % 2, coils))
    test_solver(2, coils, 10, 640)


# One transformed axis: the kernel in registers and the one staged through LDS, on both sides of the lines between them (without y and
# with y): few tiles and many, short rows, frames of few rows, few coils, 46 points with y.
@pytest.mark.parametrize("centred", [0, 1])
@pytest.mark.parametrize("W,coils,B,T,H,staged", [
    (24, 4, 2, 16, 16, (0, 0)), (24, 4, 2, 129, 20, (1, 1)), (24, 4, 5, 103, 16, (0, 1)), (24, 4, 7, 110, 16, (1, 1)), (20, 3, 1, 1, 641, (0, 0)),
    (8, 16, 3, 257, 4, (0, 1)), (8, 16, 3, 256, 4, (0, 0)), (16, 1, 13, 60, 62, (1, 1)), (8, 16, 129, 4, 5, (1, 1)),
    (160, 4, 1, 513, 1, (1, 1)), (160, 4, 1, 512, 1, (0, 0)), (64, 4, 2, 257, 7, (0, 0)), (64, 4, 2, 257, 6, (1, 1)),
    (192, 1, 1, 103, 25, (0, 1)), (192, 2, 1, 103, 25, (0, 0)), (46, 2, 2, 8, 641, (0, 1)), (46, 8, 1, 1, 320, (0, 0)),
    (46, 70, 1, 1, 257, (0, 1)), (32, 16, 4, 5, 97, (0, 0)), (4, 1, 5, 1, 7, (0, 0)), (320, 2, 1, 1, 9, (1, 1)), (256, 16, 1, 1, 640, (0, 0))])
def test_one_axis_on_both_kernels(W, coils, B, T, H, staged, centred):
    geom, *arrays = inputs(1, B, coils, T, 1, H, W, centred, W + coils + H)
    gb.gleam_profile_begin()
    check(geom, *arrays)
    ran = [r[0] for r in gb.gleam_profile_end() if r[0].startswith("sense_rows_fused")]
    assert [n.endswith("staged") for n in ran] == [bool(s) for s in staged]


# every length along both strided axes; W = 20 and 46 leave the column tiles ragged, and the mask's rows unaligned
@pytest.mark.parametrize("N", LENGTHS)
def test_every_length_along_the_strided_axes(N):
    for nd, D, H, W in ((2, 2, N, 20), (3, N, 4, 46), (3, 4, N, 16)):
        check(*inputs(nd, 1, 2, 1, D, H, W, N % 4 == 0, N + D))


# The sweeps staged through LDS, which float32 layers with kernels on split operands take when those are switched off (and greedy
# iterations): the data-consistency step alone, by a network whose weights are zero.  Every length along every axis, centred or not.
@pytest.mark.parametrize("centred", [0, 1])
@pytest.mark.parametrize("N", LENGTHS)
def test_data_consistency_on_the_staged_sweeps(N, centred, kernel_policy):
    kernel_policy(gb.POLICY_NO_WINOGRAD)
    prox = synth.chain_prox([2, 4, 4, 2], [(1, 1, 3, 3)] * 3)
    for nd, coils, D, H, W in ((2, 3, 2, N, 20), (2, 17, 1, 6, N), (3, 2, N, 4, 46), (3, 2, 4, N, 16), (1, 3, 1, 7, N)):
        geom, x, S, M, y = inputs(nd, 2, coils, 2, D, H, W, centred, N + nd)
        print("case staged", geom, flush=True)
        c = synth.make_custom(3, geom, prox, alpha=0.8)
        c = dataclasses.replace(c, x_in=x, S=S, M=M, y=y, theta=np.zeros_like(c.theta))
        r = ModuleRunner(c)
        gb.gleam_profile_begin()
        r.fwd()
        ran = [rec[0] for rec in gb.gleam_profile_end() if rec[0].startswith("sense_")]
        assert len(ran) == 2 * nd - 1 and all(n.endswith("_staged") for n in ran), ran
        assert_image_close(r.results()[0], og.dc_step(x, S, M, y, 0.8, nd, centred=bool(centred)), TOL, "DC")


# so many tiles that the columns go 32 at a time and a workgroup of the first sweep takes several coils
@pytest.mark.parametrize("H, W", [(96, 32), (256, 20)])
def test_many_tiles(H, W):
    check(*inputs(2, 1, 8, 1, 256 * 96 // H, H, W, 0, H))


# the solver's sweeps: rows that do not divide into tiles, the update of the search direction, one sample and three
@pytest.mark.parametrize("B, C, H, W", [(1, 5, 46, 20), (3, 3, 6, 46), (2, 8, 10, 160), (1, 16, 20, 368), (2, 7, 24, 640)])
def test_solver(B, C, H, W):
    from paper_2207_08393_amd.runner import ModlRunner
    geom = synth.Geom(2, B, C, 1, 1, H, W)
    c = synth.make_custom(H + W, geom, synth.chain_prox([2, 8, 2], [(1, 1, 3, 3)] * 2), accel=3.0, centre=2)
    print("case", geom, flush=True)
    r = ModlRunner(c, 0.5, 4)
    r.step()
    x = r.results()[0]
    aty = og.sense_adjoint(c.y.astype(np.complex128), c.S, c.M, 2)
    f = og.modl_module_fwd(c.geom, c.prox, c.x_in, c.S, c.M, aty, 0.5, 4, c.theta, c.x_true)
    assert_image_close(x, f["x_out"], 4 * TOL, "MoDL x_out")   # four steps, each with an operator of its own in float32


# ... with 64 rows of 32 points and 128 of 8 to a tile: coils of a row in one tile, and in two
@pytest.mark.parametrize("B,coils,W", [(1, 52, 32), (1, 65, 32), (2, 103, 8), (2, 129, 8)])
def test_solver_with_many_short_rows(B, coils, W):
    test_solver(B, coils, 640, W)
