"""Which partial products of split float32 operands (csrc/split.h) the 3x3 kernels cannot do without: the F(2, 3) row transform
on operands of three bfloat16 parts, in numpy with 64-bit sums, with the products that the header lists and with each of them
left out.  tests/test_gpu_split.py holds the kernels to a bound between the two."""
import os
import re

import numpy as np
import pytest

from paper_2207_08393_amd import synth

HEADER = os.path.join(os.path.dirname(synth.__file__), "csrc", "split.h")
BOUND = 1e-6       # what test_gpu_split.py allows a module


def bf16(x):
    u = np.asarray(x, np.float32).view(np.uint32).astype(np.uint64)
    return ((u + 0x7fff + ((u >> 16) & 1)) & 0xffff0000).astype(np.uint32).view(np.float32)


def split(x):
    parts, r = [], np.asarray(x, np.float32)
    for _ in range(3):
        parts.append(bf16(r).astype(np.float64))
        r = r - bf16(r)
    assert not r.any()                                        # exact
    return parts


def products():
    text = open(HEADER).read()
    a, b = (re.search(name + r"\[kProducts\] = \{([^}]*)\}", text).group(1) for name in ("kPartA", "kPartB"))
    return list(zip((int(v) for v in a.split(",")), (int(v) for v in b.split(","))))


def transformed_input(x, W):
    d = [x[:, i:i + W:2] for i in range(4)]
    return [d[0] - d[2], d[1] + d[2], d[2] - d[1], d[1] - d[3]]


def conv(x, w, pairs):
    """x [H+2][W+2][K], w [N][3][3][K] -> [H][W][N]"""
    H, W = x.shape[0] - 2, x.shape[1] - 2
    half = np.float32(0.5)
    g = [w[:, :, i] for i in range(3)]
    U = [g[0], half * (g[0] + g[1] + g[2]), half * (g[0] - g[1] + g[2]), g[2]]
    M = []
    for V, u in zip(transformed_input(x, W), U):
        sv, su = split(V), split(u)
        M.append(sum(sv[b][ky:ky + H] @ su[a][:, ky].T for ky in range(3) for a, b in pairs))
    y = np.empty((H, W, w.shape[0]))
    y[:, 0::2], y[:, 1::2] = M[0] + M[1] + M[2], M[1] - M[2] - M[3]
    return y


def wgrad(x, dy, pairs):
    """dy [H][W][N] -> [N][3][3][K]"""
    H, W = dy.shape[:2]
    y0, y1 = dy[:, 0::2], dy[:, 1::2]
    out = np.empty((dy.shape[2], 3, 3, x.shape[2]))
    for ky in range(3):
        p = []
        for V, A in zip(transformed_input(x, W), (y0, y0 + y1, y0 - y1, y1)):
            sv, sa = split(V[ky:ky + H]), split(A)
            p.append(sum(np.einsum("hwn,hwk->nk", sa[a], sv[b]) for a, b in pairs))
        out[:, ky, 0] = p[0] + 0.5 * (p[1] + p[2])
        out[:, ky, 1] = 0.5 * (p[1] - p[2])
        out[:, ky, 2] = 0.5 * (p[1] + p[2]) - p[3]
    return out


def cases():
    rng = np.random.default_rng(0)
    K, N, H, W = 32, 24, 10, 20
    x = np.zeros((H + 2, W + 2, K), np.float32)
    x[1:-1, 1:-1] = rng.standard_normal((H, W, K))
    w = (rng.standard_normal((N, 3, 3, K)) * np.sqrt(2 / (9 * K))).astype(np.float32)
    dy = rng.standard_normal((H, W, N)).astype(np.float32)
    views = [[x[i:i + H, j:j + W].astype(np.float64) for j in range(3)] for i in range(3)]
    ref_y = sum(views[i][j] @ w[:, i, j].astype(np.float64).T for i in range(3) for j in range(3))
    ref_w = np.stack([np.stack([np.einsum("hwn,hwk->nk", dy.astype(np.float64), views[i][j]) for j in range(3)], 1) for i in range(3)], 1)
    # position 3 of the gradient: (-y1) . (d1 - d3); the kernel takes y1 and turns the sign at the end
    return [("conv", lambda p: conv(x, w, p), ref_y), ("wgrad", lambda p: wgrad(x, dy, p), ref_w)]


@pytest.mark.parametrize("name,run,ref", cases(), ids=[c[0] for c in cases()])
def test_no_partial_product_can_be_left_out(name, run, ref):
    pairs = products()
    assert sorted(pairs) == [(0, 0), (0, 1), (0, 2), (1, 0), (1, 1), (2, 0)]
    err = lambda y: np.linalg.norm(y - ref) / np.linalg.norm(ref)
    assert err(run(pairs)) <= 0.2 * BOUND                      # (the transforms round in float32)
    for gone in pairs:
        assert err(run([p for p in pairs if p != gone])) >= 2 * BOUND, gone
