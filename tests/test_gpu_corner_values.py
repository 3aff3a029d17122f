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


# 16-bit ghost norms of 33 to 64 tokens: rows past the sample in one half of a tile, the other, both or none.
@pytest.mark.parametrize("dtype", HALF)
@pytest.mark.parametrize("where", ["a", "g"])
@pytest.mark.parametrize("B,T,d,p", [(3, 33, 136, 120), (4, 40, 8, 24), (3, 63, 64, 200), (3, 64, 72, 64)])
def test_infinite_ghost_norms_of_33_to_64_tokens(dp, dtype, where, B, T, d, p):
    check_infinite_norms(dp, dtype, 0, B, T, d, p, where, positive=True)


def norms_of_copies(dp, dtype, path, L, B, T, d, p):
    """Squared norms of a stack of L layers that all hold the same a and g, and these on the device."""
    tdt = {si.F32: torch.float32, si.BF16: torch.bfloat16, si.F16: torch.float16}[dtype]
    gen = torch.Generator(device="cuda").manual_seed(B + T)
    a = torch.randn(B, T, d, device="cuda", generator=gen).to(tdt)
    g = torch.randn(B, T, p, device="cuda", generator=gen).to(tdt)
    desc = dp.layer_array([(a, g, T, d, p, path)] * L)
    dt = dtype_code(dp, dtype)
    ws = torch.empty(dp.dp_norms_multi_workspace_bytes(desc, dt, B), dtype=torch.uint8, device="cuda")
    out = torch.full((L, B), -1.0, device="cuda")
    dp.dp_norms_multi(desc, dt, B, out, ws)
    return out, a, g


# More workgroups of 512 threads than one grid dimension holds (2^23): a stack of 48 layers whose samples have one
# each, and a single layer.
@pytest.mark.parametrize("path", [0, 1])
@pytest.mark.parametrize("L,B", [(48, 180000), (1, 2 ** 23 + 5)])
def test_fp32_norms_of_very_many_samples(dp, path, L, B):
    out, a, g = norms_of_copies(dp, si.F32, path, L, B, 1, 4, 3)
    want = a.double().square().sum((1, 2)) * g.double().square().sum((1, 2))          # one token: ||a||^2 ||g||^2
    assert torch.all((out.double() - want).abs() <= TOL * want)


@pytest.mark.parametrize("dtype,T", [(si.BF16, 17), (si.F16, 32)])
def test_ghost_norms_of_very_many_short_samples(dp, dtype, T):
    L, B = 48, 180000
    out, a, g = norms_of_copies(dp, dtype, 0, L, B, T, 8, 8)
    assert torch.all(out == out[:1])                                                   # every layer, every sample
    pick = [0, 1, B // 3, B - 2, B - 1]
    np.testing.assert_allclose(host(out[0, pick]), o.ghost_sqnorm(host(a[pick].float()), host(g[pick].float())), rtol=TOL)


def test_fp32_gradient_of_very_many_tiles(dp):
    p = 2 ** 28 + 64                                                                   # 2^23 + 2 tiles of 32 columns
    a, C = torch.full((1, 1, 1), 3.0, device="cuda"), torch.full((1,), 0.5, device="cuda")
    g = torch.arange(p, device="cuda", dtype=torch.int32).remainder_(1009).float()
    grad = torch.full((p,), -1.0, device="cuda")
    dp.dp_clipped_grad(a, g, dp.DP_F32, 1, 1, 1, p, C, grad, 0)
    assert torch.equal(grad, g.mul_(1.5))                                              # exact products


def test_bias_of_nearly_2_31_columns(dp):
    p = 2 ** 31 - 512                                    # inside the last 4096: the indices of the last round pass 2^31
    g = torch.ones((1, 1, p), dtype=torch.bfloat16, device="cuda")
    colsum = torch.empty((1, p), device="cuda")
    sq = torch.zeros(1, device="cuda")
    dp.dp_bias_norm(g, dp.DP_BF16, 1, 1, p, colsum, sq)
    assert abs(sq.item() - p) <= 1e-6 * p
    del g
    grad = torch.full((p,), -1.0, device="cuda")
    dp.dp_clipped_bias_grad(colsum, 1, p, torch.full((1,), 0.5, device="cuda"), grad, 0)
    assert grad.min().item() == 0.5 and grad.max().item() == 0.5


@pytest.mark.parametrize("dtype", HALF)
@pytest.mark.parametrize("B,T,d,p", [(40, 1, 136, 264), (5, 40, 200, 16), (6, 7, 24, 136), (3, 100, 48, 136)])
def test_packed_rows_with_nan_weight(dp, dtype, B, T, d, p):
    """A NaN weight makes every entry NaN, the others' zeros included."""
    w = si.small_workload("nanw", dtype, B, T, [(d, p)])
    a, g = (x.copy() for x in si.gen_layer(w, 0))
    a[:, :, 0] = 0
    grad = torch.zeros((d, p), device="cuda")
    C = np.full(B, 0.5, dtype=np.float32)
    C[B // 2] = np.nan
    dp.dp_clipped_grad(dev(a), dev(g), dtype_code(dp, dtype), B, T, d, p, dev(C), grad, 0)
    assert np.all(np.isnan(host(grad)))


def test_packed_rows_with_infinity_take_no_detour(dp):
    """Forming a tile again, without the split, costs about the pass it repeats (once 25 times as long)."""
    B, T, d, p = 16, 2048, 768, 16
    a = torch.randn(B, T, d, device="cuda").to(torch.bfloat16)
    g = torch.randn(B, T, p, device="cuda").to(torch.bfloat16)
    C, grad = torch.full((B,), 0.5, device="cuda"), torch.zeros(d, p, device="cuda")

    def shortest():
        us = []
        for _ in range(6):
            begin, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            begin.record()
            dp.dp_clipped_grad(a, g, dp.DP_BF16, B, T, d, p, C, grad, 0)
            end.record()
            torch.cuda.synchronize()
            us.append(begin.elapsed_time(end) * 1e3)
        return min(us)

    clean = shortest()
    a[:, 7, ::32] = float("inf")
    assert shortest() <= 8 * clean
    assert not torch.isfinite(grad[::32]).any() and torch.isfinite(grad[1::32]).all()


def check_weighted_gradient(dp, dtype, B, T, d, p, C, a_scale=1.0, g_scale=1.0, edit=None):
    """Gradient under weights C against the oracle, row by row (a row of the gradient sees one column of a)."""
    rng = np.random.default_rng([B, T, d, p])
    tdt = torch.bfloat16 if dtype == si.BF16 else torch.float16
    a = torch.from_numpy(rng.standard_normal((B, T, d)) * a_scale).to(tdt)
    g = torch.from_numpy(rng.standard_normal((B, T, p)) * g_scale).to(tdt)
    if edit is not None:
        edit(a, g)
    C = np.asarray(C, dtype=np.float32)
    grad = torch.full((d, p), 3.0, device="cuda")
    dp.dp_clipped_grad(a.cuda(), g.cuda(), dtype_code(dp, dtype), B, T, d, p, dev(C), grad, 0)
    want = o.clipped_grad(a.double().numpy(), g.double().numpy(), C.astype(np.float64))
    got = host(grad)
    assert np.all(np.isfinite(got))
    err = np.linalg.norm(got - want, axis=1) / np.linalg.norm(want, axis=1)
    assert err.max() <= TOL, err.max()


# Weights go onto the exact products of the packed-row kernel too, whatever their size: shapes it takes, in each
# tile shape.
PACKED = [(6, 1, 136, 264), (6, 7, 264, 136), (6, 70, 16, 200), (6, 70, 200, 16), (6, 40, 48, 136), (6, 33, 136, 64)]


@pytest.mark.parametrize("dtype", HALF)
@pytest.mark.parametrize("B,T,d,p", PACKED)
def test_packed_rows_weight_ranges(dp, dtype, B, T, d, p):
    for C in ([1e-8, 1e2, 1e-8, 3e-3, 1e2, 1.0], [-1.0, 1e2, 0.0, -1e-8, 1.0, 1e2], [1e-30] * 6, [3e-36] * 6,
              [1e30, 1e28, 1e30, 2e30, 1e30, 1e30]):
        check_weighted_gradient(dp, dtype, B, T, d, p, C)
    # columns that only one sample reaches, whose weight is far below the others'
    def one_sample(a, g):
        a[:5, :, :8] = 0
    check_weighted_gradient(dp, dtype, B, T, d, p, [1.0, 0.5, 1.0, 2.0, 1.0, 1e-33], edit=one_sample)


@pytest.mark.parametrize("B,T,d,p", PACKED)
def test_packed_rows_operand_ranges(dp, B, T, d, p):
    # bf16: weight times activation below and above the fp32 range, results inside it
    check_weighted_gradient(dp, si.BF16, B, T, d, p, [1e-30] * 6, a_scale=1e-12, g_scale=1e20)
    check_weighted_gradient(dp, si.BF16, B, T, d, p, [2.0 ** -100] * 6, a_scale=2.0 ** -80, g_scale=2.0 ** 120)
    check_weighted_gradient(dp, si.BF16, B, T, d, p, [1e30] * 6, a_scale=1e20, g_scale=1e-30)
    check_weighted_gradient(dp, si.BF16, B, T, d, p, [0.5, 1e-3, 1e-5, 1.0, 0.1, 0.0], a_scale=1e-35, g_scale=1e15)
    # one tiny activation among ordinary ones
    def tiny(a, g):
        a[2, 0, 3] = 2.0 ** -126
        a[:, :, 5] = 2.0 ** -120
    check_weighted_gradient(dp, si.BF16, B, T, d, p, [0.5, 1e-3, 1e-5, 1.0, 0.1, 0.7], edit=tiny)


# Narrow layers whose operands of the whole batch pass 2 GiB, the packed-row kernel's addressing: the 128 x 128 tiles
# take them as long as one sample's slab fits, with the noise in the same pass.
@pytest.mark.parametrize("B,T,d,p", [(16, 4224, 8, 16384), (33000, 1, 32768, 8)])
def test_narrow_layers_beyond_the_packed_batch(dp, B, T, d, p):
    gen = torch.Generator(device="cuda").manual_seed(B)
    a = torch.randn(B, T, d, device="cuda", generator=gen).to(torch.bfloat16)
    g = torch.randn(B, T, p, device="cuda", generator=gen).to(torch.bfloat16)
    assert B * T * max(d, p) * 2 > 2 ** 31
    C = torch.rand(B, device="cuda", generator=gen)
    C[B // 2] = 0
    want = torch.zeros(d, p, dtype=torch.float64)
    step = max(1, B // 16)
    for i in range(0, B, step):
        ca = a[i:i + step].double() * C[i:i + step].double()[:, None, None]
        want += (ca.reshape(-1, d).t() @ g[i:i + step].double().reshape(-1, p)).cpu()
    want = want.numpy()
    desc = dp.layer_array([(a, g, T, d, p, 0)])
    plain, noisy = torch.empty(d * p, device="cuda"), torch.empty(d * p, device="cuda")
    dp.dp_clipped_grad_multi(desc, dp.DP_BF16, B, C, [plain])
    assert frob(host(plain).reshape(d, p), want) <= TOL
    lo, n = 6, d * p - 17
    dp.dp_clipped_grad_noise_multi(desc, dp.DP_BF16, B, C, [noisy], [0], 0, lo, n, 0.5, 2.0, 3, 4)
    dp.dp_add_noise(plain[lo:], lo, n, 0.5, 2.0, 3, 4)
    assert torch.equal(noisy, plain)


# A layer's squared norms do not depend on the stack it stands in, though the tiles do: 256 x 256 ones where a launch
# fills whole rounds of them.
@pytest.mark.parametrize("dtype", HALF)
@pytest.mark.parametrize("L,B,T,d,p", [(32, 8, 70, 256, 256), (10, 16, 40, 384, 520), (24, 16, 33, 200, 264)])
def test_instantiated_norms_do_not_depend_on_the_stack(dp, dtype, L, B, T, d, p):
    check_stack_independence(dp, dtype, 1, L, B, T, d, p)


def check_stack_independence(dp, dtype, path, L, B, T, d, p):
    stack, a, g = norms_of_copies(dp, dtype, path, L, B, T, d, p)
    alone, a1, g1 = norms_of_copies(dp, dtype, path, 1, B, T, d, p)
    assert torch.equal(a, a1) and torch.equal(g, g1)
    assert torch.all(stack == alone)
    np.testing.assert_allclose(host(alone[0]), (o.ghost_sqnorm, o.perex_sqnorm)[path](host(a.float()), host(g.float())),
                               rtol=TOL)


# Ghost norms of 96 .. 128 tokens and widths off the 64-column k-blocks: the number of samples of the call chooses between
# 128 x 128 tiles and the large-tile kernel, with the same bits.
@pytest.mark.parametrize("dtype", HALF)
@pytest.mark.parametrize("L,B,T,d,p", [(12, 40, 112, 392, 296), (9, 30, 96, 24, 136), (20, 60, 128, 264, 1000),
                                       (3, 90, 105, 520, 72), (12, 40, 120, 256, 64)])
def test_ghost_norms_do_not_depend_on_the_stack(dp, dtype, L, B, T, d, p):
    check_stack_independence(dp, dtype, 0, L, B, T, d, p)
