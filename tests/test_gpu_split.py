"""The split-operand 3x3 / 3x3x3 kernels (prox_split.hip) where their blocks, chunks and channel groups end: module steps
against the oracle at the float32 tolerance, per layer and per element (tests/test_gpu_parity.py check_module)."""
import dataclasses

import numpy as np
import pytest

from oracle import gleam_oracle as og
from paper_2207_08393_amd import binding as gb
from paper_2207_08393_amd import synth
from tests.gpu_util import ModuleRunner, assert_grad_close, assert_image_close, rel_l2, theta_slices
from tests.test_gpu_parity import K2, K3, KT, TOL, check_module, kernel_policy  # noqa: F401
from tests.test_split_arithmetic import BOUND

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


def linear_prox(chans, k):
    """Convolutions only: no ReLU that a rounding could decide the other way, no skip that dilutes the error."""
    return synth.ProxDesc([synth.ConvLayer(a, b, *k, 0, 0, 1, -1) for a, b in zip(chans, chans[1:])])


@pytest.mark.parametrize("chans,k", [([2, 32, 32, 32, 2], K2), ([2, 36, 60, 20, 2], K2), ([2, 100, 100, 2], K2), ([2, 64, 64, 64, 2], K2),
                                     ([2, 20, 36, 2], K3), ([2, 32, 32, 2], K3)], ids=["32", "ragged", "100", "64", "volume_ragged", "volume_32"])
def test_split_operands_keep_the_precision_of_float32(chans, k):
    """Output and the gradients of every layer within 1e-6 of the 64-bit oracle: a float32 sum of these lengths is off by 1e-7 to
    7e-7 (the direct float32 kernels on such networks: 5e-8 to 6.8e-7), and a product that has lost one of its six parts by 3e-6
    in a single layer (tests/test_split_arithmetic.py)."""
    geom = synth.Geom(3, 1, 2, 1, 6, 12, 20) if k == K3 else synth.Geom(2, 2, 2, 1, 1, 20, 46)
    for seed in (1, 2):
        c = synth.make_custom(seed, geom, linear_prox(chans, k), accel=2.0, centre=2, bias_std=0.1, alpha=0.8)
        print("case split precision", chans, seed, flush=True)
        r = ModuleRunner(c)
        r.step()
        x_out, loss, grad = r.results()
        f = og.module_fwd(c.geom, c.prox, c.x_in, c.S, c.M, c.y, c.alpha, c.theta, c.x_true)
        g = og.module_bwd(c.prox, c.theta, f)
        errs = {"x_out": rel_l2(x_out, f["x_out"]), "loss": abs(loss / f["loss"] - 1)}
        errs.update({f"{layer}{kind}": rel_l2(grad[part], g[part]) for layer, kind, part in theta_slices(c.prox)})
        print({name: float(f"{e:.1e}") for name, e in errs.items()}, flush=True)
        assert max(errs.values()) <= BOUND, errs


def wide_convolutions(records):
    """Matrix-core flops issued per flop of the direct convolution, of every convolution between wide layers."""
    return {n: round(m / f, 3) for n, f, _, _, m in records if n.startswith("conv_") and "_2to" not in n and "to2_" not in n}


def winograd_cases():
    # (name, geometry, prox, Winograd): networks as greedy iterations and MoDL modules run them.  64-multiples of channels (3x3)
    # and 32-multiples (3x3x3) take the Winograd kernels there: sizes that their 4 x 32, 2 x 32 and 8 x 32 pixel blocks do not
    # divide, several images, two channel blocks on either side, one and two slices, no bias
    yield "ragged", synth.Geom(2, 2, 2, 1, 1, 10, 46), synth.resblock_prox(64, 1), True
    yield "two_blocks", synth.Geom(2, 1, 2, 1, 1, 6, 96), synth.chain_prox([2, 64, 128, 64, 2], [K2] * 4), True
    yield "nobias_l1", synth.Geom(2, 1, 2, 3, 1, 6, 46), synth.chain_prox([2, 64, 64, 2], [K2] * 3, has_bias=0, loss_kind=1), True
    yield "volume_ragged", synth.Geom(3, 2, 2, 1, 6, 6, 46), synth.chain_prox([2, 32, 64, 32, 2], [K3] * 4), True
    yield "two_slices_l1", synth.Geom(2, 1, 2, 1, 2, 10, 12), synth.chain_prox([2, 32, 32, 2], [K3] * 3, has_bias=0, loss_kind=1), True
    yield "one_slice", synth.Geom(2, 1, 2, 1, 1, 10, 46), synth.chain_prox([2, 32, 32, 2], [K3] * 3), True
    yield "direct_100", synth.Geom(2, 1, 2, 1, 1, 10, 46), synth.resblock_prox(100, 1), False
    yield "direct_ragged", synth.Geom(2, 1, 2, 1, 1, 12, 20), synth.chain_prox([2, 36, 12, 60, 2], [K2] * 4), False


@pytest.mark.parametrize("name,geom,prox,winograd", list(winograd_cases()), ids=[c[0] for c in winograd_cases()])
def test_float32_matrix_core_kernels_of_greedy_and_modl_calls(name, geom, prox, winograd):
    """The float32 Winograd and direct kernels against the oracle: a greedy iteration of one module (Adam's first moment is a tenth of
    the gradient), which keeps them, and a MoDL module, whose forward pass does.  The library's own records tell what ran."""
    from paper_2207_08393_amd.runner import GreedyRunner, ModlRunner
    c = synth.make_custom(31, geom, prox, accel=2.0, centre=2, bias_std=0.1, alpha=0.8)
    print("case float32 kernels", name, flush=True)
    r = GreedyRunner(c, [c.theta], 1e-3)
    gb.gleam_profile_begin()
    r.iteration(1)
    ran = wide_convolutions(gb.gleam_profile_end())
    assert len(ran) >= 3 and set(ran.values()) == {0.444 if winograd else 1.0}, ran
    x, losses, _, m, _ = r.results()
    f = og.module_fwd(c.geom, c.prox, c.x_in, c.S, c.M, c.y, c.alpha, c.theta, c.x_true)
    assert_image_close(x, f["x_out"], TOL)
    assert abs(losses[0] - f["loss"]) <= TOL * abs(f["loss"])
    assert_grad_close(c.prox, m[0], 0.1 * og.module_bwd(c.prox, c.theta, f), TOL, "Adam m")

    mu, n_cg = 0.5, 3
    r = ModlRunner(c, mu, n_cg)
    gb.gleam_profile_begin()
    r.step()
    ran = wide_convolutions(gb.gleam_profile_end())
    assert {v for n, v in ran.items() if "fwd" in n} == {0.444 if winograd else 1.0}, ran
    assert {v for n, v in ran.items() if "dgrad" in n} == {4.0}, ran
    assert {v for n, v in ran.items() if "wgrad" in n} == {0.444 if prox.layers[1].kd == 3 else 4.0}, ran
    x, loss, grad, _ = r.results()
    aty = og.sense_adjoint(c.y.astype(np.complex128), c.S, c.M, geom.ndim_fft)
    f = og.modl_module_fwd(c.geom, c.prox, c.x_in, c.S, c.M, aty, mu, n_cg, c.theta, c.x_true)
    g = og.modl_module_bwd(c.geom, c.prox, c.S, c.M, mu, n_cg, c.theta, f)
    assert_image_close(x, f["x_out"], TOL)
    assert rel_l2(grad, g) <= TOL

    # a plain module of the same network runs on split operands (the weight gradient of whole 3x3x3 blocks excepted)
    r = ModuleRunner(c)
    gb.gleam_profile_begin()
    r.step()
    ran = wide_convolutions(gb.gleam_profile_end())
    assert {v for n, v in ran.items() if "wgrad" not in n} == {4.0}, ran
    assert {v for n, v in ran.items() if "wgrad" in n} == {0.444 if prox.layers[1].kd == 3 else 4.0}, ran


def time_layers(prox, *layers):
    """The same network with these layers along the frames."""
    for l in layers:
        prox.layers[l] = dataclasses.replace(prox.layers[l], kt=3, kd=1, kh=1, kw=1)
    return prox


# channels that the forward kernels take by Winograd, whose sign words the backward launches must not read, and directly; skips and a
# mask behind the sum; temporal layers, whose forward pass walks the frames on the float32 matrix cores (64 channels) or takes one tap
# at a time, alone and beside 3x3 ones, on either side of a mask and of a sum
@pytest.mark.parametrize("geom,prox", [(synth.Geom(2, 2, 2, 1, 1, 64, 32), synth.chain_prox([2, 64, 128, 64, 2], [K2] * 4, loss_kind=1)),
                                       (synth.Geom(2, 1, 2, 1, 2, 46, 46), synth.resblock_prox(36, 1)),
                                       (synth.Geom(2, 1, 2, 1, 1, 96, 46), synth.resblock_prox(64, 1)),
                                       (synth.Geom(3, 1, 2, 1, 8, 20, 32), synth.chain_prox([2, 32, 64, 32, 2], [K3] * 4)),
                                       (synth.Geom(2, 1, 2, 1, 1, 4, 6), synth.resblock_prox(64, 1)),
                                       (synth.Geom(2, 1, 2, 8, 1, 24, 32), time_layers(synth.resblock_prox(64, 1), 2)),
                                       (synth.Geom(2, 1, 2, 6, 1, 20, 46), time_layers(synth.resblock_prox(36, 2), 1, 4)),
                                       (synth.Geom(2, 2, 2, 5, 1, 24, 20), time_layers(synth.chain_prox([2, 64, 64, 36, 2], [K2] * 4, loss_kind=1), 1, 2))],
                         ids=["words_4096", "res36", "res64", "volume", "24_pixels", "time_res64", "time_res36", "time_chain"])
def test_modl_backward_on_split_operands(geom, prox):
    """The backward pass of a MoDL module on split operands behind a forward pass on the float32 matrix cores."""
    from paper_2207_08393_amd.runner import ModlRunner
    c = synth.make_custom(32, geom, prox, accel=2.0, centre=2, bias_std=0.1)
    mu, n_cg = 0.5, 2
    print("case modl backward", [l.cout for l in prox.layers], flush=True)
    r = ModlRunner(c, mu, n_cg)
    gb.gleam_profile_begin()
    r.step()
    ran = wide_convolutions(gb.gleam_profile_end())
    assert {v for n, v in ran.items() if "fwd" in n} <= {0.444, 1.0} and len(ran) >= 3, ran
    assert {n: v for n, v in ran.items() if "fwd" not in n} == {n: 6.0 if n.endswith("_t3") else 4.0 for n in ran if "fwd" not in n}, ran
    assert any(n.endswith("_t3") for n in ran) == any(l.kt == 3 for l in prox.layers)
    x, loss, grad, aty = r.results()
    f = og.modl_module_fwd(c.geom, c.prox, c.x_in, c.S, c.M, aty.astype(np.complex128), mu, n_cg, c.theta, c.x_true)
    g = og.modl_module_bwd(c.geom, c.prox, c.S, c.M, mu, n_cg, c.theta, f)
    assert_image_close(x, f["x_out"], TOL)
    assert rel_l2(grad, g) <= TOL


def modules_by_hand(c, thetas, lr):
    """What gleam_greedy_iteration does, call by call: x, losses, theta, m, v."""
    from paper_2207_08393_amd.runner import GreedyRunner
    r = GreedyRunner(c, thetas, lr)
    x_in = r.x0
    for i in range(len(thetas)):
        x = r.x_out if (len(thetas) - 1 - i) % 2 == 0 else r.x_tmp
        gb.gleam_module_fwd(r.geom, r.prox, x_in, r.S, r.M, r.y, r.alpha, r.theta[i], r.x_ref, x, r.losses[i:], r.saved, r.ws)
        gb.gleam_module_bwd(r.geom, r.prox, r.theta[i], r.saved, r.grad, r.ws)
        gb.gleam_adam_step(r.hyper, 1, r.theta[i], r.grad, r.m[i], r.v[i])
        x_in = x
    return r.results()


@pytest.mark.parametrize("geom,prox,one_kernel", [(synth.Geom(2, 2, 3, 1, 1, 12, 46), synth.resblock_prox(64, 1), False),
                                                  (synth.Geom(2, 2, 3, 1, 1, 12, 46), synth.resblock_prox(36, 1), False),
                                                  (synth.Geom(2, 2, 3, 1, 1, 12, 46), synth.resblock_prox(6, 1), True),
                                                  (synth.Geom(2, 1, 3, 6, 1, 12, 20), time_layers(synth.resblock_prox(64, 1), 2), False),
                                                  (synth.Geom(2, 1, 3, 6, 1, 12, 20), synth.resblock_prox(36, 1, KT), False),
                                                  (synth.Geom(2, 1, 3, 6, 1, 12, 20), synth.resblock_prox(6, 1, KT), True)],
                         ids=["64", "36", "6", "mixed64", "time36", "time6"])
def test_greedy_iteration_and_the_same_calls_by_hand(geom, prox, one_kernel, kernel_policy):
    """Bit for bit the same where a layer has one kernel for both (6 channels, or GLEAM_POLICY_NO_WINOGRAD).  Otherwise the
    modules by hand run on split operands and the iteration does not: each is within 1e-6 of the 64-bit results in its first
    module (test above, and TOL for the iteration), a second module starts from an input that differs by that much; no further
    apart than 1e-5 in the outputs and the first moments, where no ReLU of these networks is decided the other way."""
    from paper_2207_08393_amd.runner import GreedyRunner
    c = synth.make_custom(21, geom, prox, accel=2.0, centre=2, bias_std=0.1, alpha=0.8)
    thetas = [c.theta, c.theta + np.float32(0.03) * np.random.default_rng(2).standard_normal(c.theta.size).astype(np.float32)]
    for policy in (0, gb.POLICY_NO_WINOGRAD):
        kernel_policy(policy)
        print("case greedy by hand", [(l.cout, l.kt) for l in prox.layers], policy, flush=True)
        r = GreedyRunner(c, thetas, 1e-3)
        r.iteration(1)
        whole, parts = r.results(), modules_by_hand(c, thetas, 1e-3)
        if policy or one_kernel:
            assert all(np.array_equal(a, b) for a, b in zip(whole, parts))
            continue
        x, losses, _, m, _ = whole
        errs = [rel_l2(parts[0], x), rel_l2(parts[1], losses)] + [rel_l2(parts[3][i], m[i]) for i in range(2)]
        print("apart", errs, flush=True)
        assert 0 < max(errs) <= 1e-5


@pytest.mark.parametrize("geom,chans", [(synth.Geom(3, 1, 2, 1, 8, 20, 46), (32, 64, 32)), (synth.Geom(3, 2, 2, 1, 4, 20, 20), (32, 32, 64))],
                         ids=["320_segments", "160_segments"])
def test_weight_gradient_of_whole_3x3x3_blocks_on_split_operands(geom, chans):
    """From 160 row segments on, 3x3x3 layers between multiples of 32 channels take the split-operand weight gradient too."""
    c = synth.make_custom(41, geom, synth.chain_prox([2, *chans, 2], [K3] * 4), accel=2.0, centre=2, bias_std=0.1, alpha=0.8)
    print("case whole 3x3x3 blocks", chans, flush=True)
    r = ModuleRunner(c)
    gb.gleam_profile_begin()
    r.step()
    ran = wide_convolutions(gb.gleam_profile_end())
    assert set(ran.values()) == {4.0}, ran
    check_module(c)


# the last grid of 4-row blocks and the first of 8-row ones (256 workgroups, 128 with 27 taps), with sign words between two launches;
# heights that leave a 4-row block ragged
@pytest.mark.parametrize("H", [253, 256, 257])
def test_blocks_of_four_and_eight_rows_2d(H):
    check_module(synth.make_custom(51, synth.Geom(1, 1, 2, 1, 4, H, 46), synth.chain_prox([2, 20, 32, 2], [K2] * 3), accel=2.0, centre=2,
                                   bias_std=0.1, alpha=0.8))


@pytest.mark.parametrize("D", [64, 96])
def test_blocks_of_four_and_eight_rows_3d(D):
    check_module(synth.make_custom(52, synth.Geom(3, 1, 2, 1, D, 10, 20), synth.chain_prox([2, 20, 32, 20, 2], [K3] * 4), accel=2.0,
                                   centre=2, bias_std=0.1, alpha=0.8))


# blocks of eight rows whose input lies inside the image, between such that reach over its border; several blocks
# per workgroup, of several images; sign words between two launches, a mask with a tensor to add, a ReLU on the input
@pytest.mark.parametrize("geom,prox", [(synth.Geom(1, 1, 2, 1, 4, 180, 96), synth.chain_prox([2, 20, 32, 64, 2], [K2] * 4)),
                                       (synth.Geom(2, 2, 2, 1, 2, 192, 160), synth.resblock_prox(36, 1)),
                                       (synth.Geom(3, 1, 2, 1, 8, 46, 96), synth.chain_prox([2, 32, 32, 20, 2], [K3] * 4))],
                         ids=["words", "residual", "volume"])
def test_blocks_inside_the_image(geom, prox):
    print("case inside", [l.cout for l in prox.layers], flush=True)
    check_module(synth.make_custom(53, geom, prox, accel=2.0, centre=2, bias_std=0.1, alpha=0.8))


@pytest.mark.parametrize("geom,k,modl", [(synth.Geom(2, 1, 2, 1, 1, 20, 46), K2, False), (synth.Geom(3, 1, 2, 1, 8, 20, 46), K3, False),
                                         (synth.Geom(2, 1, 2, 6, 1, 10, 20), KT, False), (synth.Geom(2, 1, 2, 1, 1, 20, 46), K2, True),
                                         (synth.Geom(2, 1, 2, 6, 1, 10, 20), KT, True)], ids=["2d", "3d", "time", "modl_2d", "modl_time"])
def test_range_of_the_weight_gradient(geom, k, modl):
    """What lies below 2^-126 of an operand's parts and of their products is lost (csrc/split.h).  As in test_gpu_cover.py the gradient
    of layer 2 is one product per value, so scaling the weights of layer 3 by a power of two scales it exactly, and the weight
    gradient of layer 2 with it, but for that loss.  A product has six partial products of up to eight multiplied bits each whose
    smallest are 2^-126 when it is 2^-102: 6 * 8 losses of 2^-126 against values of 2^a .. 2^(a + 2), activations of order one (44 to
    56 seen where it is more than the rounding of the result).  Nothing down to 2^-94 = 5e-29.  An infinity shows.
    In a MoDL module dL/dz is that of the loss divided by 1 + (A^H A) / mu, here within a tenth of one: half the values at most."""
    from paper_2207_08393_amd.runner import ModlRunner
    taps, n = int(np.prod(k)), 32
    rng = np.random.default_rng(5)
    shape = geom.image_shape
    ref = (rng.uniform(1, 2, (2,) + shape) * rng.choice((-1.0, 1.0), (2,) + shape) * 2.0 ** 40).astype(np.float32)
    w1, b1 = rng.standard_normal((n, taps, 2)), rng.standard_normal(n)
    w2, b2 = rng.standard_normal((n, taps, n)) / np.sqrt(taps * n), rng.standard_normal(n)
    c = synth.make_custom(19, geom, synth.chain_prox([2, n, n, 2], [k] * 3), alpha=0.0)
    part = next(p for layer, kind, p in theta_slices(c.prox) if layer == 2 and kind == "W")
    g_z = 2.0 ** 41 / (geom.B * geom.T * geom.D * geom.H * geom.W)     # of the smallest value of ref

    def weight_gradient(a, x_in=c.x_in):
        w3 = np.zeros((2, taps, n))
        w3[np.arange(n) % 2, np.arange(n) * 5 % taps, np.arange(n)] = np.random.default_rng(6).uniform(1, 2, n)
        w3 *= 2.0 ** (a - np.floor(np.log2(g_z)))
        theta = np.concatenate([v.ravel() for v in (w1, b1, w2, b2, w3, np.zeros(2))]).astype(np.float32)
        case = dataclasses.replace(c, x_true=ref[0] + 1j * ref[1], theta=theta, x_in=x_in)
        r = ModlRunner(case, 64.0, 2) if modl else ModuleRunner(case)
        gb.gleam_profile_begin()
        r.step()
        ran = wide_convolutions(gb.gleam_profile_end())
        assert {v for name, v in ran.items() if "wgrad" in name} == {6.0 if k == KT else 4.0}, ran
        return r.grad.cpu().numpy()[part].astype(np.float64)

    print("case range", k, modl, flush=True)
    base = weight_gradient(0)
    assert np.all(np.isfinite(base)) and rel_l2(base, np.zeros_like(base) + base.mean()) > 0.1
    for a in (-60, -94, -104, -112):
        err = rel_l2(weight_gradient(a) * 2.0 ** -a, base)
        print("smallest output gradient 2 ^", a, "apart", err, flush=True)
        assert err <= (0 if a >= -94 else (128 if modl else 64) * 2.0 ** (-126 - a))
    x_in = c.x_in.copy()
    x_in[..., 5, 7] = np.inf
    assert not np.isfinite(weight_gradient(0, x_in)).all()
