"""GPU parity at values and sizes that a kernel's padding, splitting or indexing can get wrong:
infinities next to padded rows and columns, weights at the ends of the fp32 range, more
workgroups than one grid dimension takes.

An infinite norm gives C_i = 0, so the sample drops out; a NaN norm would make the whole gradient NaN.
"""
import numpy as np
import pytest

import synth_inputs as si
from oracle import bk_oracle as o

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

TOL = 1e-5                                   # fp32 sums of exact products, as in test_gpu_shapes.py
HALF = [si.BF16, si.F16]


@pytest.fixture(scope="module")
def dp():
    import paper_2311_11822_amd.binding as b
    return b


def dev(x):
    return torch.from_numpy(x.view(np.int16) if x.dtype == np.uint16 else x).cuda()


def host(t):
    torch.cuda.synchronize()
    return t.detach().cpu().numpy().astype(np.float64)


def frob(got, want):
    return np.linalg.norm(got - want) / max(np.linalg.norm(want), 1e-300)


def dtype_code(dp, dtype):
    return {si.F32: dp.DP_F32, si.BF16: dp.DP_BF16, si.F16: dp.DP_F16}[dtype]


def check_infinite_norms(dp, dtype, path, B, T, d, p, where, positive=False):
    """Infinities in two samples' a or g: those norms are infinite, the others exact, and C is 0 there."""
    w = si.small_workload("inf", dtype, B, T, [(d, p)], g_std=1.0 if dtype == si.F32 else 1e-2)
    a, g = (x.copy() for x in si.gen_layer(w, 0))
    if positive:                             # then every pair's product of a ghost norm is +inf, none -inf
        a, g = (np.abs(x) if x.dtype != np.uint16 else x & 0x7FFF for x in (a, g))
    inf = 0x7F80 if dtype == si.BF16 else np.inf
    x = a if where == "a" else g
    x[0, 0, 0] = inf
    x[B - 1, T - 1, x.shape[2] - 1] = inf
    dt = dtype_code(dp, dtype)
    ws = torch.empty(dp.dp_norm_workspace_bytes(path, dt, B, T, d, p), dtype=torch.uint8, device="cuda")
    out = torch.full((1, B), -1.0, device="cuda")
    (dp.dp_ghost_norm, dp.dp_perex_norm)[path](dev(a), dev(g), dt, B, T, d, p, out, ws)
    a64, g64 = si.to_f64(a), si.to_f64(g)
    got = host(out)[0]
    assert np.isposinf(got[0]) and np.isposinf(got[B - 1])
    fin = slice(1, B - 1)
    np.testing.assert_allclose(got[fin], (o.ghost_sqnorm, o.perex_sqnorm)[path](a64[fin], g64[fin]), rtol=TOL)
    C = torch.full((B,), -1.0, device="cuda")
    dp.dp_clip_factors(out, 1, B, 0, 0.5, 0.01, C)
    c = host(C)
    assert c[0] == 0.0 and c[B - 1] == 0.0 and np.all(c[fin] > 0)


# fp32: few tiles (the waves share a tile's tokens) and many, each side off the 32-wide tiles; one-token and
# longer ghost norms, whose padding is token rows.
@pytest.mark.parametrize("where", ["a", "g"])
@pytest.mark.parametrize("path,B,T,d,p", [
    (1, 4, 5, 20, 20), (1, 3, 40, 32, 20), (1, 3, 40, 20, 32), (1, 3, 5, 100, 130), (1, 3, 17, 128, 97),
    (0, 5, 1, 20, 20), (0, 4, 1, 7, 3), (0, 3, 31, 12, 40), (0, 3, 40, 20, 8),
])
def test_infinite_norms_fp32(dp, path, B, T, d, p, where):
    check_infinite_norms(dp, si.F32, path, B, T, d, p, where, positive=path == 0)


# 16-bit instantiated norms: 256 x 256 tiles whose edge lies inside a 128 x 128 one (256 of them, 576 of 128 x 128),
# 128 x 128 tiles with and without padding, the narrow tiles.
@pytest.mark.parametrize("dtype", HALF)
@pytest.mark.parametrize("where", ["a", "g"])
@pytest.mark.parametrize("B,T,d,p", [(64, 40, 384, 384), (3, 33, 384, 128), (3, 70, 200, 136), (3, 40, 768, 16),
                                     (3, 40, 24, 200), (3, 40, 104, 56), (3, 40, 40, 136)])
def test_infinite_instantiated_norms(dp, dtype, where, B, T, d, p):
    check_infinite_norms(dp, dtype, 1, B, T, d, p, where)
