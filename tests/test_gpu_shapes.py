"""GPU parity at the shapes where a kernel's tiles, remainders or packing can go wrong: whole steps
(norms, clip factors, gradients with the noise in the same pass) against the CPU oracle.

Tolerances: fp32 and 16-bit inputs alike enter products exactly or with one fp32 rounding and are
summed in fp32, so norms and gradients lie within 1e-5 (2-norm) of the 64-bit oracle; the noise is
compared as in test_gpu_parity.py.
"""
import numpy as np
import pytest

import synth_inputs as si
from oracle import bk_oracle as o

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

TOL = 1e-5


def dev(x):
    return torch.from_numpy(x.view(np.int16) if x.dtype == np.uint16 else x).cuda()


def host(t):
    torch.cuda.synchronize()
    return t.detach().cpu().numpy().astype(np.float64)


def frob(got, want):
    return np.linalg.norm(got - want) / max(np.linalg.norm(want), 1e-300)


def check_step(dtype, B, T, dims, mode=o.CLIP_STANDARD, R=0.5, paths=None, mask=()):
    """One step without and one with noise on an uneven shard; samples in `mask` get a zero weight
    and NaN activations in the gradient pass (a masked sample is not read)."""
    from paper_2311_11822_amd import binding as dp
    from paper_2311_11822_amd.pipeline import BkPipeline
    w = si.small_workload("shapes", dtype, B, T, dims, g_std=1.0 if dtype == si.F32 else 1e-2)
    layers = [si.gen_layer(w, l) for l in range(w.L)]
    l64 = [(si.to_f64(a), si.to_f64(g)) for a, g in layers]
    pipe = BkPipeline([(dev(a), dev(g)) for a, g in layers], paths)
    if dtype == si.BF16:
        assert pipe.dt == dp.DP_BF16
    pipe.norms()
    sq = np.array([o.ghost_sqnorm(a, g) if T * T < a.shape[2] * g.shape[2] else o.perex_sqnorm(a, g) for a, g in l64])
    np.testing.assert_allclose(host(pipe.sqnorm), sq, rtol=TOL)
    pipe.clip(mode, R, 0.01)
    C, norm = o.clip_factors(sq, mode, R, 0.01)
    np.testing.assert_allclose(host(pipe.C), C, rtol=TOL)
    if mask:
        C = C.copy()
        for i in mask:
            C[i] = 0.0
            pipe.C[i] = 0.0
            for a, _ in pipe.layers:
                a[i] = float("nan") if a.dtype != torch.int16 else 0x7FC0
    want = [o.clipped_grad(a, g, C) for a, g in l64]
    pipe.flat.fill_(float("nan"))
    pipe.grad()
    for got, G in zip(pipe.grads, want):
        assert frob(host(got), G) <= TOL
    clean = host(pipe.flat)
    pipe.grad(accumulate=1)
    np.testing.assert_array_equal(host(pipe.flat), 2 * clean)
    lo = min(5, pipe.psi - 1)
    cnt = max(1, pipe.psi - lo - 3)
    sigma, R_noise = 0.5, 2.0
    pipe.grad_noise(sigma, R_noise, 9, 2, lo, cnt)
    fused = pipe.flat.clone()
    pipe.grad()
    pipe.noise(sigma, R_noise, 9, 2, lo, cnt)
    assert torch.equal(fused, pipe.flat)                      # same values as the separate pass
    z = host(fused)[lo:lo + cnt] - clean[lo:lo + cnt]
    zw = o.normals(9, 2, lo, cnt)
    bound = 2e-5 * np.maximum(1, np.abs(zw)) + 2e-7 * np.abs(clean[lo:lo + cnt])   # one more fp32 rounding of G + z
    assert np.all(np.abs(z - zw) <= bound)


# Edges of the 32 x 32 tiles, widths off the vector loads (not multiples of 4), runs that straddle
# generator blocks, fewer and more tiles and token chunks than waves, both norm forms.
@pytest.mark.parametrize("B,T,dims", [
    (4, 8, [(16, 16)]), (1, 1, [(4, 1), (3, 2)]), (2, 17, [(32, 32), (66, 6), (31, 33)]),
    (3, 70, [(20, 20), (4, 160)]), (33, 33, [(96, 384), (10, 7)]), (2, 150, [(104, 97)]),
])
def test_fp32_stack(B, T, dims):
    check_step(si.F32, B, T, dims)
    check_step(si.F32, B, T, dims, mode=o.CLIP_AUTOMATIC, mask=[B - 1] if B > 1 else ())


def test_fp32_more_layers_than_one_launch():
    check_step(si.F32, 2, 5, [(4 * (1 + l % 5), 3 + l % 7) if l % 2 else (8, 4) for l in range(50)],
               paths=[l % 2 for l in range(50)])


HALF = [si.BF16, si.F16]


# Packed-row gradient (short samples, narrow layers): one token, tokens that divide no 32-row block, a
# total below and off a multiple of 32, tile edges and the five tile shapes, masked samples
# that hold NaN (first, inside, last).
@pytest.mark.parametrize("dtype", HALF)
@pytest.mark.parametrize("B,T,dims", [
    (1, 1, [(8, 8)]), (70, 1, [(136, 264), (128, 128)]), (9, 7, [(200, 328), (24, 304), (304, 24)]),
    (5, 31, [(72, 72), (64, 200), (200, 64)]), (2, 33, [(256, 8), (8, 256)]), (3, 70, [(16, 1104), (1104, 40)]),
])
def test_packed_rows(dtype, B, T, dims):
    check_step(dtype, B, T, dims, paths=[0] * len(dims))
    check_step(dtype, B, T, dims, mode=o.CLIP_AUTOMATIC, mask=sorted({0, B // 2, B - 1}) if B > 2 else ())


@pytest.mark.parametrize("dtype", HALF)
@pytest.mark.parametrize("where", ["a", "g", "both"])
def test_packed_rows_with_infinities(dtype, where):
    """An infinity stays where it belongs: same infinities and NaNs as sample-by-sample sums, the rest untouched."""
    from paper_2311_11822_amd import binding as dp
    B, T, d, p = 6, 5, 136, 152
    w = si.small_workload("inf", dtype, B, T, [(d, p)], g_std=1e-2)
    a, g = si.gen_layer(w, 0)
    one, inf = (0x3F80, 0x7F80) if dtype == si.BF16 else (1.0, np.inf)
    a[:, :, 3] = one                                     # exact in one part: the others are zero
    if where in ("a", "both"):
        a[2, 4, 5] = inf
    if where in ("g", "both"):
        g[1, 0, 140] = inf
        g[4, 2, 0] = inf
    C = np.array([1.0, 0.5, 0.25, 0.0, 2.0, 0.7], dtype=np.float32)
    with np.errstate(invalid="ignore"):
        want = o.clipped_grad(si.to_f64(a), si.to_f64(g), C.astype(np.float64))
    grad = torch.zeros((d, p), device="cuda")
    dt = dp.DP_BF16 if dtype == si.BF16 else dp.DP_F16
    dp.dp_clipped_grad(dev(a), dev(g), dt, B, T, d, p, dev(C), grad, 0)
    got = host(grad)
    np.testing.assert_array_equal(np.isnan(got), np.isnan(want))
    np.testing.assert_array_equal(np.isposinf(got), np.isposinf(want))
    np.testing.assert_array_equal(np.isneginf(got), np.isneginf(want))
    ok = np.isfinite(want)
    assert ok.sum() > 0.9 * ok.size and frob(got[ok], want[ok]) <= TOL


@pytest.mark.parametrize("dtype,T", [(si.BF16, 32), (si.F16, 32), (si.BF16, 64)])
def test_half_gradient_of_short_samples(dtype, T):
    """The 16-bit gradient is the fp32 one rounded once, whichever kernel the token count selects."""
    from paper_2311_11822_amd import binding as dp
    B, dims = 5, [(136, 264), (128, 128)]
    w = si.small_workload("h16", dtype, B, T, dims)
    keep = [tuple(dev(x) for x in si.gen_layer(w, l)) for l in range(2)]
    dt, tdt = (dp.DP_BF16, torch.bfloat16) if dtype == si.BF16 else (dp.DP_F16, torch.float16)
    desc = dp.layer_array([(a, g, T, d, p, 0) for (a, g), (d, p) in zip(keep, dims)])
    C = dev(np.array([0.7, 0.0, 0.05, 1.0, 0.3], dtype=np.float32))
    offs, n = [0, dims[0][0] * dims[0][1]], sum(d * p for d, p in dims)
    old = [(torch.randn(d, p, device="cuda") * 0.05).to(tdt) for d, p in dims]
    got, ref = [x.clone() for x in old], [x.float() for x in old]
    dp.dp_clipped_grad_noise_multi_h16(desc, dt, B, C, got, offs, 1, 6, n - 9, 0.01, 2.0, 5, 9)
    dp.dp_clipped_grad_noise_multi(desc, dt, B, C, ref, offs, 1, 6, n - 9, 0.01, 2.0, 5, 9)
    for x, y in zip(got, ref):
        assert torch.equal(x.view(torch.int16), y.to(tdt).view(torch.int16))


# Ghost norm of short samples: several samples to a workgroup (the last one not full), one sample of 17 .. 32
# rows, widths that end inside a 16-column step, more columns than the waves take in one go.
@pytest.mark.parametrize("dtype", HALF)
@pytest.mark.parametrize("B,T,d,p", [
    (1, 1, 8, 8), (33, 1, 24, 1032), (67, 2, 136, 40), (31, 3, 2056, 64), (7, 16, 72, 200), (3, 17, 264, 88),
    (2, 32, 1160, 8), (5, 31, 16, 4104), (45, 3, 40, 24), (2600, 3, 16, 8), (5, 1, 40, 24), (3, 2, 264, 16),
])
def test_ghost_norm_of_short_samples(dtype, B, T, d, p):
    from paper_2311_11822_amd import binding as dp
    w = si.small_workload("brief", dtype, B, T, [(d, p)], g_std=1e-2)
    a, g = si.gen_layer(w, 0)
    dt = dp.DP_BF16 if dtype == si.BF16 else dp.DP_F16
    out = torch.full((B + 1,), -1.0, device="cuda")
    ws = torch.empty(max(16, dp.dp_norm_workspace_bytes(0, dt, B, T, d, p)), dtype=torch.uint8, device="cuda")
    dp.dp_ghost_norm(dev(a), dev(g), dt, B, T, d, p, out, ws)
    want = o.ghost_sqnorm(si.to_f64(a), si.to_f64(g))
    # sums of d + p exact products: relative to the sum of their magnitudes, which the diagonal bounds
    np.testing.assert_allclose(host(out)[:B], want, rtol=TOL)
    assert host(out)[B] == -1.0


# Token counts that end inside a 32-token k-block: last block of 1, 16, 17 and 31 rows, one block only,
# on large tiles (168 of 256 x 256) and on the sub-tiles that smaller launches take (56 and a few tiles, and
# 160 tiles whose padding makes sub-tiles the better choice).
@pytest.mark.parametrize("dtype", HALF)
@pytest.mark.parametrize("B,T,dims", [
    (3, 49, [(1800, 1544)]), (2, 65, [(1800, 1544), (136, 520)]), (3, 100, [(264, 136), (128, 2048)]),
    (2, 127, [(1800, 1544)]), (1, 80, [(1800, 1544)]),
    (2, 49, [(2824, 3336)]), (2, 21, [(264, 264)] * 40),
])
def test_ragged_tokens(dtype, B, T, dims):
    check_step(dtype, B, T, dims, paths=[0] * len(dims))
    check_step(dtype, B, T, dims, mode=o.CLIP_AUTOMATIC, mask=[1] if B > 1 else ())


# Instantiated norms and kept gradients on 256 x 256 tiles (168 of them, 572 of 128 x 128) and on 128 x 128 ones, odd
# and even numbers of k-blocks, a last block that is not full.
@pytest.mark.parametrize("dtype", HALF)
@pytest.mark.parametrize("B,T,dims", [(4, 40, [(1544, 1288)]), (3, 97, [(392, 136)]), (2, 64, [(128, 264)])])
def test_instantiated_norm_tiles(dtype, B, T, dims):
    check_step(dtype, B, T, dims, paths=[1] * len(dims))


# Narrow layers on the instantiated path: sides of up to 32 and up to 64, wide sides off the 128-column tiles, fewer
# tokens than the stages hold, a last k-block of one row.
@pytest.mark.parametrize("dtype", HALF)
@pytest.mark.parametrize("B,T,dims", [
    (3, 97, [(264, 16), (16, 264), (392, 64), (64, 392)]), (2, 40, [(40, 40), (8, 8), (24, 48), (136, 40)]),
    (5, 256, [(768, 16), (16, 768)]), (1, 33, [(48, 1032), (1032, 32)]),
])
def test_narrow_instantiated(dtype, B, T, dims):
    check_step(dtype, B, T, dims, paths=[1] * len(dims))


# Ghost norms of widths that end inside a 64-column k-block (8, 16, 56 columns of the last one; narrower than a
# block), in each of the kernels of more than 95 tokens: compact, whole-sample and large tiles.
@pytest.mark.parametrize("dtype", HALF)
@pytest.mark.parametrize("T", [97, 128, 130, 256, 257, 400])
def test_ghost_norm_ragged_widths(dtype, T):
    from paper_2311_11822_amd import binding as dp
    B, dt = 3, dp.DP_BF16 if dtype == si.BF16 else dp.DP_F16
    for d, p in [(72, 264), (136, 56), (24, 120), (64, 8)]:
        w = si.small_workload("widths", dtype, B, T, [(d, p)], g_std=1e-2)
        a, g = si.gen_layer(w, 0)
        out = torch.zeros(B, device="cuda")
        ws = torch.empty(max(16, dp.dp_norm_workspace_bytes(0, dt, B, T, d, p)), dtype=torch.uint8, device="cuda")
        dp.dp_ghost_norm(dev(a), dev(g), dt, B, T, d, p, out, ws)
        np.testing.assert_allclose(host(out), o.ghost_sqnorm(si.to_f64(a), si.to_f64(g)), rtol=TOL)


# Narrow sides on either side of the token counts at which they change from packed rows to the 128 x 128 tiles, one and
# two sides narrow, next to a wide layer in one launch.
@pytest.mark.parametrize("dtype,T,dims", [
    (si.BF16, 47, [(72, 264), (264, 120), (120, 96)]), (si.BF16, 48, [(72, 264), (264, 120), (120, 96)]),
    (si.F16, 17, [(72, 264), (264, 120), (120, 96)]), (si.F16, 18, [(72, 264), (264, 120), (120, 96)]),
    (si.F16, 27, [(40, 264), (264, 64), (48, 120)]), (si.F16, 28, [(40, 264), (264, 64), (48, 120)]),
    (si.F16, 47, [(16, 264), (264, 32), (8, 24)]), (si.F16, 48, [(16, 264), (264, 32), (8, 24)]),
    (si.F16, 70, [(24, 1104), (392, 520), (1104, 88), (56, 136)]), (si.BF16, 9, [(128, 520), (72, 264), (264, 264)]),
])
@pytest.mark.parametrize("B", [2, 4, 40])                       # 40 samples: more rows than the line of narrow fp16 sides
def test_narrow_sides_at_the_packed_lines(dtype, T, dims, B):
    check_step(dtype, B, T, dims, paths=[0] * len(dims))
    check_step(dtype, B, T, dims, paths=[0] * len(dims), mode=o.CLIP_AUTOMATIC, mask=[1])


# Short contractions, whose tiles are cut into 128 x 128 throughout (60 and 280 large tiles), just below and above the
# line.
@pytest.mark.parametrize("dtype", HALF)
@pytest.mark.parametrize("B,T,dims", [(1, 70, [(1800, 1928)]), (15, 31, [(1800, 1928)]), (17, 31, [(1800, 1928)]),
                                      (2, 33, [(1800, 1928), (1544, 1288), (2824, 3336)])])
def test_short_contractions(dtype, B, T, dims):
    check_step(dtype, B, T, dims, paths=[0] * len(dims))


def test_fp16_narrow_layers_keep_pace_with_bf16():
    """Long fp16 samples of narrow layers take as many matrix instructions as bf16 ones (six times as many once)."""
    from paper_2311_11822_amd.pipeline import BkPipeline

    def shortest(dt):
        dims = [(1024, 96), (96, 1024)] * 8
        pipe = BkPipeline([(torch.randn(64, 128, d, device="cuda").to(dt), torch.randn(64, 128, p, device="cuda").to(dt))
                           for d, p in dims], [0] * len(dims))
        pipe.C.fill_(0.5)
        us = []
        for _ in range(8):
            begin, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            begin.record()
            pipe.grad()
            end.record()
            torch.cuda.synchronize()
            us.append(begin.elapsed_time(end) * 1e3)
        return min(us)

    assert shortest(torch.float16) <= 1.4 * shortest(torch.bfloat16)


# The weighted contraction's stream on 256 x 256 tiles (a whole round of them) and on 128 x 128: samples that end inside
# a 32-row block (odd numbers of 16-row steps), samples of one block with and without gaps, fewer and more samples
# than the 64 whose weights a wave holds, windows without a sample that counts, and equal weights.
@pytest.mark.parametrize("side,n", [(2048, 4), (1536, 1)])
@pytest.mark.parametrize("B,T,zero", [
    (3, 21, ()), (64, 32, ()), (65, 32, (0, 63, 64)), (67, 20, ()), (131, 24, tuple(range(64, 128))), (66, 33, (1, 2, 65)),
    (5, 48, (4,)), (7, 40, (0, 1, 3)), (3, 49, ()), (2, 112, ()), (4, 33, (0, 1, 2, 3)),
    (1, 40, ()), (1, 64, ()), (1, 24, (0,)), (2, 48, (0,)), (65, 48, tuple(range(64))), (66, 24, (65,)), (129, 40, ()),
])
def test_weighted_stream(side, n, B, T, zero):
    from paper_2311_11822_amd import binding as dp
    gen = torch.Generator(device="cuda")
    gen.manual_seed(B * 1000 + T)
    layers = [tuple(torch.randn((B, T, side), generator=gen, device="cuda").to(torch.bfloat16) for _ in range(2))
              for _ in range(n)]
    desc = dp.layer_array([(a, g, T, side, side, dp.DP_PATH_GHOST) for a, g in layers])
    C = torch.rand(B, generator=gen, device="cuda") + 0.1
    C[B // 2:B // 2 + 2] = 0.75                           # two equal weights in a row: no multiply between them
    for i in zero:
        C[i] = 0.0
        for a, _ in layers:
            a[i] = float("nan")
    grads = [torch.full((side, side), float("nan"), device="cuda") for _ in layers]
    dp.dp_clipped_grad_multi(desc, dp.DP_BF16, B, C, grads)
    keep = C != 0
    for (a, g), got in zip(layers, grads):
        weighted = (a[keep].double() * C[keep].double()[:, None, None]).reshape(-1, side)
        want = weighted.t().contiguous() @ g[keep].double().reshape(-1, side)
        assert torch.linalg.norm(got.double() - want) <= TOL * torch.linalg.norm(want)


# Samples in whole 32-row k-blocks, a workgroup to a tile: 128 x 128 tiles of three stages (the first four cases) and of
# five, 256 x 256 with more than 64 samples; an odd number of 16-row steps, a group without a sample that counts between
# others, one sample alone, runs of equal weights; the same bits on the tiles of a layer by itself.
@pytest.mark.parametrize("dtype", [si.BF16, si.F16])
@pytest.mark.parametrize("B,T", [(2, 65 + 31), (3, 64), (5, 64), (1, 160), (4, 225), (65, 64), (130, 49)])
def test_whole_k_blocks(dtype, B, T):
    from paper_2311_11822_amd import binding as dp
    d, p, n = 2056, 2312, 6
    dt, tdt = (dp.DP_BF16, torch.bfloat16) if dtype == si.BF16 else (dp.DP_F16, torch.float16)
    gen = torch.Generator(device="cuda").manual_seed(B * T)
    layers = [tuple((torch.randn((B, T, w), generator=gen, device="cuda") * s).to(tdt) for w, s in ((d, 1.0), (p, 0.01)))
              for _ in range(n)]
    C = torch.rand((n, B), generator=gen, device="cuda") + 0.1
    C[1, B // 2:B // 2 + 2] = 0.5
    C[2] = 0.0                                            # nothing of this layer
    C[3, 1:] = 0.0                                        # one sample
    C[4, ::2] = 0.0
    C[5] = 0.25                                           # one weight
    grads = [torch.full((d, p), float("nan"), device="cuda") for _ in layers]
    desc = dp.layer_array([(a, g, T, d, p, dp.DP_PATH_GHOST) for a, g in layers])
    dp.dp_clipped_grad_grouped(desc, dt, B, C, list(range(n)), n, grads)
    for l, (a, g) in enumerate(layers):
        alone = torch.empty((d, p), device="cuda")
        dp.dp_clipped_grad(a, g, dt, B, T, d, p, C[l].contiguous(), alone, 0)
        assert torch.equal(grads[l], alone)               # whichever tiles the launch takes
        w = (a.double() * C[l].double()[:, None, None]).reshape(B * T, d)
        want = w.t().contiguous() @ g.double().reshape(B * T, p)
        # exact products, sums of up to 6500 terms and B re-expressions in fp32
        assert float((grads[l].double() - want).norm()) <= 3e-6 * float(want.norm())
    clean = torch.cat([x.reshape(-1) for x in grads])
    dp.dp_clipped_grad_grouped(desc, dt, B, C, list(range(n)), n, grads, 1)
    assert torch.equal(torch.cat([x.reshape(-1) for x in grads]), 2 * clean)
    flat = torch.empty(n * d * p, device="cuda")
    pieces, offs = list(flat.view(n, d, p)), [l * d * p for l in range(n)]
    noise = (1001, n * d * p - 2002, 0.5, 1.0, 3, 4)
    dp.dp_clipped_grad_noise_multi(desc, dt, B, C[0].contiguous(), pieces, offs, 0, *noise)
    fused = flat.clone()
    dp.dp_clipped_grad_multi(desc, dt, B, C[0].contiguous(), pieces)
    dp.dp_add_noise(flat.data_ptr() + 4 * noise[0], *noise)
    assert torch.equal(fused, flat)


# Tile after tile in one workgroup, every one of them two 256 x 256 tiles (eight layers) or some three and some two (eleven): a tile of
# the first round is followed by one of the fourth layer after it.  Too few k-blocks to join two tiles (fewer than the ring's
# five) and just enough, on either side; nothing that counts before, behind or between; samples of one weight, samples that
# begin in the joined tile's first blocks, an odd number of 16-row steps.  Samples that do not count hold NaN.
@pytest.mark.parametrize("dtype", [si.BF16, si.F16])
@pytest.mark.parametrize("n,B,T", [(8, 2, 96), (8, 3, 64), (8, 5, 64), (8, 1, 160), (8, 4, 225), (11, 5, 128), (11, 64, 64)])
def test_joined_tiles(dtype, n, B, T):
    from paper_2311_11822_amd import binding as dp
    side = 2040
    dt, tdt = (dp.DP_BF16, torch.bfloat16) if dtype == si.BF16 else (dp.DP_F16, torch.float16)
    gen = torch.Generator(device="cuda").manual_seed(B * T + n)
    layers = [tuple((torch.randn((B, T, side), generator=gen, device="cuda") * s).to(tdt) for s in (1.0, 0.01)) for _ in range(n)]
    desc = dp.layer_array([(a, g, T, side, side, dp.DP_PATH_GHOST) for a, g in layers])

    def joined(out16):
        plan = dp.dp_clipped_grad_launches(desc, dt, B, out16)
        return plan["tiles"] == 64 * n and plan["workgroups"] == 256 and plan["whole_blocks"] == 1 and plan["cut"] == 0

    assert joined(False)
    blocks = -(-T // 32)
    some = lambda k: (torch.arange(B, device="cuda") < min(k, B)).float()           # the first k samples
    C = torch.rand((n, B), generator=gen, device="cuda") + 0.1
    C[1] = 0.0                                            # nothing, then something
    C[2] *= some(4 // blocks)                             # up to four blocks, then all
    C[3] *= some(-(-5 // blocks))                         # five blocks, or the next number there is, then as few
    C[7] = C[7].flip(0) * some(-(-5 // blocks)).flip(0)
    C[5] *= some(4 // blocks)
    C[6] = 0.0                                            # few blocks, then nothing
    C[4, B // 2:B // 2 + 2] = 0.5
    if n > 8:
        C[8] = 0.25                                       # one weight
        C[9, ::2] = 0.0
    for (a, _), c in zip(layers, C):
        a[c == 0] = float("nan")
    groups = list(range(n))
    grads = [torch.full((side, side), float("nan"), device="cuda") for _ in layers]
    dp.dp_clipped_grad_grouped(desc, dt, B, C, groups, n, grads)
    for l, (a, g) in enumerate(layers):
        alone = torch.empty((side, side), device="cuda")
        dp.dp_clipped_grad(a, g, dt, B, T, side, side, C[l].contiguous(), alone, 0)
        assert torch.equal(grads[l], alone)
        keep = C[l] != 0
        w = (a[keep].double() * C[l][keep].double()[:, None, None]).reshape(-1, side)
        want = w.t().contiguous() @ g[keep].double().reshape(-1, side)
        # exact products, sums of up to 4096 terms and B re-expressions in fp32
        assert float((grads[l].double() - want).norm()) <= 3e-6 * float(want.norm())
    clean = torch.cat([x.reshape(-1) for x in grads])
    dp.dp_clipped_grad_grouped(desc, dt, B, C, groups, n, grads, 1)                  # old values while the stream runs on
    assert torch.equal(torch.cat([x.reshape(-1) for x in grads]), 2 * clean)
    # one group of weights; noise on an uneven shard, stored in 32 and in 16 bits
    for a, _ in layers:
        a.nan_to_num_(0.5)
    one = C[9 if n > 8 else 0].contiguous()
    flat = torch.empty(n * side * side, device="cuda")
    pieces, offs = list(flat.view(n, side, side)), [l * side * side for l in range(n)]
    noise = (1001, n * side * side - 2002, 0.5, 1.0, 3, 4)
    dp.dp_clipped_grad_noise_multi(desc, dt, B, one, pieces, offs, 0, *noise)
    fused = flat.clone()
    dp.dp_clipped_grad_multi(desc, dt, B, one, pieces)
    dp.dp_add_noise(flat.data_ptr() + 4 * noise[0], *noise)
    assert torch.equal(fused, flat)
    if T % 32 == 0:                                       # what the 16-bit call takes
        assert joined(True)
        flat16 = torch.empty(n * side * side, dtype=tdt, device="cuda")
        pieces16 = list(flat16.view(n, side, side))
        dp.dp_clipped_grad_noise_multi_h16(desc, dt, B, one, pieces16, offs, 0, *noise)
        assert torch.equal(flat16, fused.to(tdt))


# Large tiles on part of the chip alone stay on 16-row steps, more of them take whole k-blocks: the same bits.
@pytest.mark.parametrize("dtype", [si.BF16, si.F16])
@pytest.mark.parametrize("B,T", [(7, 160), (5, 250), (65, 64)])
def test_whole_k_blocks_against_steps(dtype, B, T):
    from paper_2311_11822_amd import binding as dp
    side = 1016
    dt, tdt = (dp.DP_BF16, torch.bfloat16) if dtype == si.BF16 else (dp.DP_F16, torch.float16)
    gen = torch.Generator(device="cuda").manual_seed(B * T)
    layers = [tuple((torch.randn((B, T, side), generator=gen, device="cuda") * s).to(tdt) for s in (1.0, 0.01)) for _ in range(12)]
    C = torch.rand(B, generator=gen, device="cuda") + 0.1
    C[B // 2] = 0.0
    grads = {}
    for n, whole in ((9, 0), (12, 1)):
        desc = dp.layer_array([(a, g, T, side, side, dp.DP_PATH_GHOST) for a, g in layers[:n]])
        plan = dp.dp_clipped_grad_launches(desc, dt, B)
        assert (plan["tiles"], plan["whole_blocks"], plan["cut"]) == (16 * n, whole, 0)
        grads[n] = torch.full((n, side, side), float("nan"), device="cuda")
        dp.dp_clipped_grad_multi(desc, dt, B, C, list(grads[n]))
    assert torch.equal(grads[9], grads[12][:9])
    for (a, g), got in zip(layers, grads[12]):
        want = (a.double() * C.double()[:, None, None]).reshape(B * T, side).t().contiguous() @ g.double().reshape(B * T, side)
        # exact products, sums of up to 4160 terms and B re-expressions in fp32
        assert float((got.double() - want).norm()) <= 3e-6 * float(want.norm())


# Launches on either side of the lines between streaming and cached stores (rows of whole 128-byte lines and others, 32, 200 and 256 MB, with
# noise and without, 128 and 512 rows): the bits of the layers alone, on all tiles, packed rows among them.
@pytest.mark.parametrize("n,side,B,T", [(7, 1016, 4, 64), (9, 1016, 4, 64), (9, 1016, 9, 64), (9, 1024, 4, 64), (47, 1024, 2, 64),
                                        (48, 1032, 2, 64), (48, 1088, 2, 64), (9, 1016, 64, 2), (9, 1016, 65, 2), (9, 1024, 64, 2), (48, 1192, 20, 2), (48, 1192, 2, 64), (48, 1192, 5, 32),
                                        (32, 512, 4, 33)])
def test_gradients_of_large_and_small_launches(n, side, B, T):
    from paper_2311_11822_amd import binding as dp
    gen = torch.Generator(device="cuda").manual_seed(n * side)
    layers = [tuple((torch.randn((B, T, side), generator=gen, device="cuda") * s).to(torch.bfloat16) for s in (1.0, 0.01))
              for _ in range(n)]
    desc = dp.layer_array([(a, g, T, side, side, dp.DP_PATH_GHOST) for a, g in layers])
    C = torch.rand(B, generator=gen, device="cuda") + 0.1
    flat, alone = torch.empty((n, side, side), device="cuda"), torch.empty((n, side, side), device="cuda")
    pieces, offs = list(flat), [l * side * side for l in range(n)]
    for l, (a, g) in enumerate(layers):
        dp.dp_clipped_grad(a, g, dp.DP_BF16, B, T, side, side, C, alone[l], 0)
    dp.dp_clipped_grad_multi(desc, dp.DP_BF16, B, C, pieces)
    assert torch.equal(flat, alone)
    dp.dp_clipped_grad_multi(desc, dp.DP_BF16, B, C, pieces, 1)
    assert torch.equal(flat, 2 * alone)
    noise = (1001, n * side * side // 8, 0.5, 1.0, 3, 4)
    dp.dp_clipped_grad_noise_multi(desc, dp.DP_BF16, B, C, pieces, offs, 0, *noise)
    dp.dp_add_noise(alone.data_ptr() + 4 * noise[0], *noise)
    assert torch.equal(flat, alone)


# The same on 64 x 64 tiles alone: odd and even numbers of k-blocks, fewer than the ring's eight on their way, more samples than a
# window, windows and samples that do not count, columns past the last tile's edge.
@pytest.mark.parametrize("side", [512, 392])
@pytest.mark.parametrize("B,T,zero", [
    (1, 40, ()), (1, 96, ()), (3, 64, (1,)), (3, 64, (0,)), (5, 33, (4,)), (2, 300, ()), (7, 288, (0, 3)), (65, 40, (0, 63)), (130, 36, tuple(range(64, 128))),
    (4, 48, (0, 1, 2, 3)),
])
def test_weighted_stream_of_small_tiles(side, B, T, zero):
    test_weighted_stream(side, 2, B, T, zero)


# Column sums and their norm in one launch and in two: fewer and more rows than a thread takes at once, row groups that
# do not come out even, the widest row of the one-launch form and one beyond, both sides of its line.
@pytest.mark.parametrize("dtype", HALF)
@pytest.mark.parametrize("B,T,p", [
    (1, 1, 8), (3, 7, 8), (2, 9, 24), (5, 70, 264), (2, 8, 8192), (2, 7, 8200), (3, 160, 512), (3, 161, 512), (2, 700, 256),
    (2, 700, 264), (1, 4097, 16), (300, 1, 8), (300, 9, 40), (300, 33, 128), (300, 1, 264), (255, 330, 256), (256, 330, 256),
])
def test_bias_norm_forms(dtype, B, T, p):
    from paper_2311_11822_amd import binding as dp
    dt = {si.BF16: dp.DP_BF16, si.F16: dp.DP_F16}[dtype]
    w = si.small_workload("bias", dtype, B, T, [(8, p)], g_std=1.0)
    g = si.gen_layer(w, 0)[1]
    colsum = torch.full((B, p), float("nan"), device="cuda")
    sq = torch.full((B,), float("nan"), device="cuda")
    dp.dp_bias_norm(dev(g), dt, B, T, p, colsum, sq)
    g64 = si.to_f64(g)
    assert frob(host(colsum), o.bias_per_sample_grad(g64)) <= TOL
    np.testing.assert_allclose(host(sq), o.bias_sqnorm(g64), rtol=TOL)


# Column sums in strips of 64 columns: one trip of four rows a thread and one row more, both sides of the lines between the
# workgroups' sizes and of eight rows' trips, a strip that is not full, the last small enough call and one beyond; rows that are not
# whole 128-byte lines in 256 strips, in 257 and (the other kernel again) in very many.
@pytest.mark.parametrize("dtype", HALF)
@pytest.mark.parametrize("B,T,p", [
    (8, 128, 768), (8, 129, 768), (2, 256, 1288), (2, 257, 1288), (3, 513, 520), (1, 4097, 328), (1, 2, 65544),
    (4, 256, 6144), (4, 257, 6144), (10, 11, 8192), (10, 11, 8200), (1, 11, 16376), (1, 11, 16392),
])
def test_bias_norm_of_few_strips(dtype, B, T, p):
    test_bias_norm_forms(dtype, B, T, p)


# One call for a step against its three stages, and factors written by the kernels that finish the norms against the
# clip kernels: the same bits.  Stacks whose norms end in every kernel: partial sums of one launch, of several and of two
# kernels; final norms (fp32, short samples, 129 to 256 tokens in whole and ragged widths) of few workgroups and layers, and of
# many in small steps (up to 256 workgroups, 4096 lanes of norms, more layers than a wave's lanes), which form the factors
# themselves, and of larger steps, which do not; more layers than a launch holds.
STEP_STACKS = [
    (si.F32, 3, 9, [(16, 24)] * 3, None),
    (si.F32, 5, 5, [(8, 8)] * 16, None),              # 80 workgroups, 16 layers
    (si.F32, 6, 5, [(8, 8)] * 14, None),              # 84, 14
    (si.F32, 2, 5, [(8, 8)] * 32, None),
    (si.F32, 1, 5, [(8, 8)] * 33, None),
    (si.F32, 2, 5, [(8, 8)] * 70, None),
    (si.F32, 95, 3, [(8, 8)], None),
    (si.F32, 256, 3, [(8, 8)], None),                 # 256 workgroups
    (si.F32, 257, 3, [(8, 8)], None),
    (si.F32, 3, 5, [(8, 8)] * 70, None),              # 210 workgroups, lanes of two layers
    (si.F16, 60, 2, [(64, 64)] * 36, None),           # 3840 lanes of norms: eight samples a lane
    (si.BF16, 65, 2, [(64, 64)] * 36, None),          # 4160
    (si.BF16, 7, 8, [(256, 512)] * 9, None),          # 5.0 MB
    (si.BF16, 7, 8, [(256, 512)] * 11, None),         # 6.1 MB
    (si.BF16, 16, 32, [(16, 8)] * 9, None),           # 512 rows, the most that do
    (si.BF16, 17, 32, [(16, 8)] * 9, None),
    (si.BF16, 5, 21, [(64, 72), (128, 136)], None),
    (si.BF16, 40, 7, [(16, 8)] * 2, None),            # 2 x 10 workgroups of four samples, shared by four each
    (si.F16, 77, 5, [(40, 24)] * 9, None),            # 13 and 26 workgroups a layer
    (si.BF16, 5, 41, [(64, 72), (128, 136)], [0] * 2),               # 33 to 64 tokens
    (si.F16, 31, 64, [(72, 136), (128, 64), (8, 8)], [0] * 3),       # 93 workgroups, 3 layers
    (si.BF16, 2, 130, [(64, 128)] * 3, [0] * 3),
    (si.F16, 31, 256, [(72, 136), (128, 64), (8, 8)], [0] * 3),      # 93, 3
    (si.BF16, 32, 200, [(72, 64)] * 3, [0] * 3),
    (si.F16, 4, 140, [(136, 264), (264, 72)], [0, 1]),
    (si.BF16, 3, 300, [(72, 136), (136, 200), (16, 200), (136, 136)], [0, 1, 1, 0]),
    (si.BF16, 2, 40, [(64 + 8 * (l % 3), 72) for l in range(103)], [l % 2 for l in range(103)]),
]


@pytest.mark.parametrize("dtype,B,T,dims,paths", STEP_STACKS)
@pytest.mark.parametrize("mode", [o.CLIP_STANDARD, o.CLIP_AUTOMATIC])
def test_step_in_one_call(dtype, B, T, dims, paths, mode):
    from paper_2311_11822_amd import binding as dp
    from paper_2311_11822_amd.pipeline import BkPipeline
    w = si.small_workload("step", dtype, B, T, dims, g_std=1.0 if dtype == si.F32 else 1e-2)
    layers = [si.gen_layer(w, l) for l in range(w.L)]
    layers = [(dev(a), dev(g)) for a, g in layers]
    if B > 1:
        for a, g in layers:
            g[0] = 0
    pipe = BkPipeline(layers, paths)
    outputs = [pipe.sqnorm, pipe.C, pipe.norm, pipe.flat]

    def stages(accumulate=0):
        pipe.norms()
        pipe.clip(mode, 0.5, 0.01)
        pipe.grad_noise(0.7, 0.5, 3, 1, 4, pipe.psi - 8, accumulate)
        return [x.clone() for x in outputs]

    def call(counter, accumulate=0):
        dp.dp_private_step_multi(pipe.desc, pipe.dt, pipe.B, mode, 0.5, 0.01, pipe.kept_ptrs if pipe.any_kept else None,
                                 pipe.grad_ptrs, pipe.grad_offsets, accumulate, 4, pipe.psi - 8, 0.7, 3, 1, pipe.sqnorm,
                                 pipe.C, pipe.norm, pipe.ws, counter)

    def check(want, which=slice(None)):
        for got, x in list(zip(outputs, want))[which]:
            assert torch.equal(got.view(torch.int32), x.view(torch.int32))
            got.fill_(123.0)
        assert pipe.counter.item() == 0
    for x in outputs:
        x.fill_(123.0)
    want = stages()
    assert all(torch.isfinite(x).all() for x in want) and (want[3][4:-4] != 0).any()
    for x in outputs:
        x.fill_(123.0)
    for _ in range(2):                                # the count of finished workgroups is back at zero
        pipe.step(mode, 0.5, 0.7, 0.01, 3, 1, 4, pipe.psi - 8)
        check(want)
    call(None)
    check(want)
    pipe.flat.fill_(0.25)
    more = stages(accumulate=1)
    for x in outputs:
        x.fill_(0.25)
    call(pipe.counter, accumulate=1)
    check(more)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(pipe.counter)
    for _ in range(3):
        graph.replay()
        check(want)
        pipe.step(mode, 0.5, 0.7, 0.01, 3, 1, 4, pipe.psi - 8)      # eager work between the replays
        check(want)
    # layer-wise
    R = [0.1 + 0.01 * l for l in range(w.L)]
    pipe.set_groups(list(range(w.L)), R)
    pipe.layerwise_step(mode, 0.01, 0.0, 3, 1, 0, 0)
    C = pipe.C_groups.clone()
    assert torch.isfinite(C).all()
    pipe.C_groups.fill_(123.0)
    pipe.clip_grouped(mode, 0.01)
    assert torch.equal(C.view(torch.int32), pipe.C_groups.view(torch.int32))
    # a NaN in one sample is that sample's norm and factor, in both
    layers[0][0][B - 1, 0, 0] = float("nan") if layers[0][0].dtype != torch.int16 else 0x7FC0
    want = stages()
    assert torch.isnan(want[1][B - 1]) and torch.isfinite(want[1][:B - 1]).all()
    for x in outputs:
        x.fill_(123.0)
    call(pipe.counter)
    check(want, slice(0, 3))


# A step that is refused has touched none of its outputs.
@pytest.mark.parametrize("bad", [
    dict(sigma=-1.0), dict(R=float("inf")), dict(accumulate=2), dict(offset=2 ** 64 - 1), dict(count=2 ** 64 - 1), dict(grads=4),
    dict(ws=None), dict(counter=2),
])
def test_refused_step_touches_nothing(bad):
    from paper_2311_11822_amd import binding as dp
    from paper_2311_11822_amd.pipeline import BkPipeline
    w = si.small_workload("refused", si.BF16, 3, 40, [(72, 136), (16, 24)], g_std=1e-2)
    pipe = BkPipeline([tuple(dev(x) for x in si.gen_layer(w, l)) for l in range(w.L)], [dp.DP_PATH_GHOST, dp.DP_PATH_PEREX])
    outputs = [pipe.sqnorm, pipe.C, pipe.norm, pipe.flat, pipe.kept[1]]
    for x in outputs:
        x.fill_(123.0)
    a = dict(dict(sigma=0.5, R=1.0, accumulate=0, offset=8, count=16, grads=0, ws=pipe.ws, counter=0), **bad)
    grads = [x.data_ptr() for x in pipe.grads]
    grads[1] += a["grads"]
    with pytest.raises(dp.DpError):
        dp.dp_private_step_multi(pipe.desc, pipe.dt, pipe.B, dp.DP_CLIP_STANDARD, a["R"], 0.01, pipe.kept_ptrs, grads,
                                 pipe.grad_offsets, a["accumulate"], a["offset"], a["count"], a["sigma"], 3, 0, pipe.sqnorm,
                                 pipe.C, pipe.norm, a["ws"], pipe.counter.data_ptr() + a["counter"])
    torch.cuda.synchronize()
    for x in outputs:
        assert (x == 123.0).all()
    assert pipe.counter.item() == 0


def test_step_counts_only_where_its_counter_was_cleared(monkeypatch):
    """The cell in which workgroups count must be zero when a step begins: a step on another stream than the one that
    cleared it has nothing that orders the two, and forms the factors in a launch of their own."""
    from paper_2311_11822_amd import binding as dp
    from paper_2311_11822_amd.pipeline import BkPipeline
    w = si.small_workload("cell", si.F32, 4, 8, [(16, 16)])
    layers = [tuple(dev(x) for x in si.gen_layer(w, 0))]
    torch.cuda.synchronize()
    side, other = torch.cuda.Stream(), torch.cuda.Stream()
    with torch.cuda.stream(side):
        pipe = BkPipeline(layers)
    given = []
    step = lambda stream=None: pipe.step(o.CLIP_STANDARD, 0.5, 0.0, 0.01, 0, 0, 0, 0, stream)
    with monkeypatch.context() as m:                      # which cell is passed, nothing enqueued
        m.setattr(dp, "dp_private_step_multi", lambda *args: given.append(args[-2]))
        step()
        step(side)
        step(side.cuda_stream)
        step(other)
        with torch.cuda.stream(other):
            step()
            step(side)
    assert [x is pipe.counter for x in given] == [False, True, True, False, False, True]
    assert all(x is None for x in given if x is not pipe.counter)
    want = None
    for stream in (side, other, torch.cuda.current_stream(), side):
        for x in (pipe.C, pipe.norm, pipe.flat):
            x.fill_(123.0)
        torch.cuda.synchronize()
        step(stream)
        torch.cuda.synchronize()
        got = [x.clone() for x in (pipe.sqnorm, pipe.C, pipe.norm, pipe.flat)]
        want = want or got
        assert all(torch.equal(a, b) for a, b in zip(got, want))
        assert pipe.counter.item() == 0


# Short contractions of many 128 x 128 tiles: three workgroups to a compute unit, three stages.  One k-block, an odd number of
# k-steps, the longest that qualifies; ragged edges; a weight of zero.
@pytest.mark.parametrize("dtype", [si.BF16, si.F16])
@pytest.mark.parametrize("B,T", [(3, 20), (5, 33), (1, 512)])
def test_short_contractions_of_many_tiles(dtype, B, T):
    from paper_2311_11822_amd import binding as dp
    dims = [(1160, 1032)] * 7 + [(1160, 264)]
    dt, tdt = (dp.DP_BF16, torch.bfloat16) if dtype == si.BF16 else (dp.DP_F16, torch.float16)
    gen = torch.Generator(device="cuda").manual_seed(7)
    keep = [tuple((torch.randn((B, T, n), generator=gen, device="cuda") * s).to(tdt) for n, s in ((d, 1.0), (p, 0.01))) for d, p in dims]
    C = torch.rand(B, generator=gen, device="cuda") + 0.1
    if B > 1:
        C[1] = 0.0
    desc = dp.layer_array([(a, g, T, d, p, 0) for (a, g), (d, p) in zip(keep, dims)])
    offs = [sum(d * p for d, p in dims[:l]) for l in range(len(dims))]
    total = sum(d * p for d, p in dims)
    got = [torch.full((d, p), 7.0, device="cuda") for d, p in dims]
    dp.dp_clipped_grad_noise_multi(desc, dt, B, C, got, offs, 0, 1001, total - 2002, 0.5, 1.0, 3, 4)
    for l, ((a, g), (d, p)) in enumerate(zip(keep, dims)):
        alone, clean = torch.empty((d, p), device="cuda"), torch.empty((d, p), device="cuda")
        one = dp.layer_array([(a, g, T, d, p, 0)])
        dp.dp_clipped_grad_noise_multi(one, dt, B, C, [alone], [offs[l]], 0, 1001, total - 2002, 0.5, 1.0, 3, 4)
        assert torch.equal(got[l], alone)                     # whichever tiles the launch takes
        dp.dp_clipped_grad_multi(one, dt, B, C, [clean], 0)
        ref = (a.double() * C.double()[:, None, None]).reshape(B * T, d).t().contiguous() @ g.double().reshape(B * T, p)
        # exact products, sums of up to 512 terms and B re-expressions in fp32: some units of 2^-24 a step
        assert float((clean.double() - ref).norm() / ref.norm()) < 3e-6
    half = [torch.empty((d, p), device="cuda", dtype=tdt) for d, p in dims]
    if T % 32 == 0:
        dp.dp_clipped_grad_noise_multi_h16(desc, dt, B, C, half, offs, 0, 1001, total - 2002, 0.5, 1.0, 3, 4)
        for x, y in zip(half, got):
            assert torch.equal(x.view(torch.int16), y.to(tdt).view(torch.int16))


# Layer-wise pass on either side of the one-kernel form's lines: its longest sample, one token more, a stack that it does
# not take whole, strips of adapters, and per-sample gradients of more than 64 MB beside another layer.
@pytest.mark.parametrize("dtype", [si.BF16, si.F16])
@pytest.mark.parametrize("B,T,dims", [(3, 512, [(128, 96), (64, 64)]), (3, 513, [(128, 96), (64, 64)]),
                                      (9, 200, [(64, 192), (64, 64)]), (5, 130, [(512, 16), (16, 512), (24, 32)]),
                                      (520, 130, [(128, 128), (128, 128), (128, 136)])])
def test_layerwise_either_form(dtype, B, T, dims):
    from paper_2311_11822_amd import binding as dp
    from paper_2311_11822_amd.pipeline import BkPipeline
    tdt = torch.bfloat16 if dtype == si.BF16 else torch.float16
    gen = torch.Generator(device="cuda").manual_seed(11)
    layers = [tuple((torch.randn((B, T, n), generator=gen, device="cuda") * s).to(tdt) for n, s in ((d, 1.0), (p, 0.01)))
              for d, p in dims]
    pipe = BkPipeline(layers, paths=[dp.DP_PATH_PEREX] * len(dims))
    pipe.set_groups(list(range(len(dims))), [0.5] * len(dims))
    pipe.layerwise_step(dp.DP_CLIP_STANDARD, 0.01, 0.0, 1, 0, 0, pipe.psi)
    for l, (a, g) in enumerate(layers):
        each = torch.stack([a[i].double().t().contiguous() @ g[i].double() for i in range(B)])
        sq = each.square().sum((1, 2))
        factor = (0.5 / sq.sqrt()).clamp(max=1.0)
        ref = (each * factor[:, None, None]).sum(0)
        # exact products; sums of T rows and B samples in fp32
        assert float(((pipe.sqnorm[l].double() - sq) / sq).abs().max()) < 1e-5
        assert float((pipe.grads[l].double() - ref).norm() / ref.norm()) < 3e-6


# fp32 norms of stacks whose widths are all multiples of four (either path) and of stacks with another width: the two halves
# of 33 to 64 tokens, one tile, more than two.
@pytest.mark.parametrize("T", [32, 33, 48, 64, 65])
@pytest.mark.parametrize("dims", [[(36, 100), (300, 8), (4, 4)], [(36, 100), (300, 8), (5, 6)]])
def test_f32_norms_by_width(T, dims):
    from paper_2311_11822_amd import binding as dp
    B = 3
    gen = torch.Generator(device="cuda").manual_seed(T)
    keep = [tuple(torch.randn((B, T, n), generator=gen, device="cuda") for n in dim) for dim in dims]
    want = torch.stack([torch.stack([(a[i].double().t() @ g[i].double()).square().sum() for i in range(B)]) for a, g in keep])
    for path in (dp.DP_PATH_GHOST, dp.DP_PATH_PEREX):
        desc = dp.layer_array([(a, g, T, d, p, path) for (a, g), (d, p) in zip(keep, dims)])
        ws = torch.empty(dp.dp_norms_multi_workspace_bytes(desc, dp.DP_F32, B), dtype=torch.uint8, device="cuda")
        got = torch.empty((len(dims), B), device="cuda")
        dp.dp_norms_multi(desc, dp.DP_F32, B, got, ws)
        # sums of up to T^2 products, each of sums of up to 300, in fp32
        assert float(((got.double() - want) / want).abs().max()) < 1e-5


# Accumulating: the weight, the old value and their sum are one rounding, in every tile size.
@pytest.mark.parametrize("dims,T", [([(136, 72)], 200), ([(1024, 1024)] * 2, 300), ([(4096, 4096)], 600), ([(1160, 1032)] * 8, 40)])
def test_accumulate_rounds_once(dims, T):
    from paper_2311_11822_amd import binding as dp
    gen = torch.Generator(device="cuda").manual_seed(5)
    keep = [tuple((torch.randn((1, T, n), generator=gen, device="cuda")).to(torch.bfloat16) for n in dim) for dim in dims]
    desc = dp.layer_array([(a, g, T, d, p, 0) for (a, g), (d, p) in zip(keep, dims)])
    plain = [torch.empty(dim, device="cuda") for dim in dims]
    old = [torch.randn(dim, generator=gen, device="cuda") for dim in dims]
    got = [x.clone() for x in old]
    c = torch.tensor([0.3], device="cuda")
    dp.dp_clipped_grad_multi(desc, dp.DP_BF16, 1, torch.ones(1, device="cuda"), plain, 0)
    dp.dp_clipped_grad_multi(desc, dp.DP_BF16, 1, c, got, 1)
    for x, y, z in zip(got, plain, old):
        assert torch.equal(x, (y.double() * c.double() + z.double()).float())


# Ghost norms of 33 to 95 tokens: up to 64 in pairs of 32-row tiles unless the layer is wide, beyond on large tiles for few
# samples and on 128 x 128 ones for many; the same bits for any number of samples.
@pytest.mark.parametrize("dtype", [si.BF16, si.F16])
@pytest.mark.parametrize("T,d,p", [(33, 136, 120), (47, 8, 520), (64, 64, 128), (64, 4608, 80), (64, 4608, 72), (65, 8, 200), (95, 72, 64)])
def test_ghost_norms_of_33_to_95_tokens(dtype, T, d, p):
    from paper_2311_11822_amd import binding as dp
    dt, tdt = (dp.DP_BF16, torch.bfloat16) if dtype == si.BF16 else (dp.DP_F16, torch.float16)
    gen = torch.Generator(device="cuda").manual_seed(T)
    a = torch.randn((300, T, d), generator=gen, device="cuda").to(tdt)
    g = torch.randn((300, T, p), generator=gen, device="cuda").to(tdt)

    def norms(B):
        desc = dp.layer_array([(a, g, T, d, p, dp.DP_PATH_GHOST)])
        ws = torch.empty(dp.dp_norms_multi_workspace_bytes(desc, dt, B), dtype=torch.uint8, device="cuda")
        out = torch.empty((1, B), device="cuda")
        dp.dp_norms_multi(desc, dt, B, out, ws)
        return out[0]

    many, few = norms(300), norms(50)
    assert torch.equal(many[:50], few)
    want = torch.stack([(a[i].double().t().contiguous() @ g[i].double()).square().sum() for i in range(50)])
    # exact products; sums of up to 4608 columns and T^2 pairs in fp32
    assert float(((few.double() - want) / want).abs().max()) < 1e-5


# A layer's norms and factors in the layer-wise pass are the same bits in either form of it, so that they do not depend on the
# stack: one layer that the one-kernel form cannot take sends few samples to the other.  Every way in which the other
# form's kernels add up (a 128 x 128 tile; 32 rows, 32 columns or 32 x 64 to a wave; several narrow tiles), with and without
# padding beside an infinity.
SQUARES = [(128, 128), (128, 96), (72, 128), (104, 72), (64, 64), (128, 16), (16, 24), (128, 64), (40, 56), (24, 128), (32, 40),
           (8, 72), (40, 72), (64, 128), (48, 104)]


@pytest.mark.parametrize("dtype", [si.BF16, si.F16])
@pytest.mark.parametrize("B,T,dims", [(5, 1, SQUARES), (5, 33, SQUARES), (5, 100, SQUARES), (300, 70, SQUARES[:4]),
                                      (300, 40, SQUARES[4:9]), (5, 100, [(512, 32), (160, 8), (264, 16), (400, 24)]),
                                      (5, 70, [(32, 512), (8, 160), (16, 264), (24, 400)])])
def test_layerwise_norms_do_not_depend_on_the_stack(dtype, B, T, dims):
    from paper_2311_11822_amd import binding as dp
    from paper_2311_11822_amd.pipeline import BkPipeline
    tdt = torch.bfloat16 if dtype == si.BF16 else torch.float16
    gen = torch.Generator(device="cuda").manual_seed(T)
    layers = [tuple((torch.randn((B, T, n), generator=gen, device="cuda") * s).to(tdt) for n, s in ((d, 1.0), (p, 0.01)))
              for d, p in dims + [(128, 136)]]
    for a, g in layers:
        a[0, 0, 0] = g[4, T - 1, -1] = float("inf")
    got = []
    for stack in (layers[:-1], layers):
        pipe = BkPipeline(stack, paths=[dp.DP_PATH_PEREX] * len(stack))
        pipe.set_groups(list(range(pipe.L)), [0.5] * pipe.L)
        pipe.layerwise_step(dp.DP_CLIP_STANDARD, 0.01, 0.0, 1, 0, 0, pipe.psi)
        got.append((pipe.sqnorm[:len(dims)].clone(), pipe.C_groups[:len(dims)].clone()))
        assert all(torch.isfinite(x).all() for x in pipe.grads)
        assert torch.isposinf(pipe.sqnorm[:, [0, 4]]).all() and (pipe.C_groups[:, [0, 4]] == 0).all()
        for l, ((a, g), x) in enumerate(zip(stack, pipe.grads)):
            each = torch.stack([a[i].double().t().contiguous() @ g[i].double() for i in range(B) if i not in (0, 4)])
            factor = torch.cat([pipe.C_groups[l, 1:4], pipe.C_groups[l, 5:]]).double()
            ref = (each * factor[:, None, None]).sum(0)
            assert float((x.double() - ref).norm() / ref.norm()) < 3e-6       # sums of T rows and B samples in fp32
        pipe.norms()
        assert torch.equal(pipe.sqnorm[:len(dims)], got[-1][0])
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])


# Ghost norms of 33 to 64 tokens: waves without columns of their own, and many large samples, which take a compute unit each.
@pytest.mark.parametrize("dtype", [si.BF16, si.F16])
@pytest.mark.parametrize("B,T,d,p", [(70, 40, 24, 16), (70, 64, 104, 8), (70, 33, 8, 112), (1030, 64, 1544, 520)])
def test_ghost_norms_of_33_to_64_tokens_by_width(dtype, B, T, d, p):
    from paper_2311_11822_amd import binding as dp
    dt, tdt = (dp.DP_BF16, torch.bfloat16) if dtype == si.BF16 else (dp.DP_F16, torch.float16)
    gen = torch.Generator(device="cuda").manual_seed(T)
    a = torch.randn((B, T, d), generator=gen, device="cuda").to(tdt)
    g = torch.randn((B, T, p), generator=gen, device="cuda").to(tdt)
    got = []
    for n in (B, 9):
        desc = dp.layer_array([(a[:n], g[:n], T, d, p, dp.DP_PATH_GHOST)])
        ws = torch.empty(dp.dp_norms_multi_workspace_bytes(desc, dt, n), dtype=torch.uint8, device="cuda")
        got.append(torch.empty((1, n), device="cuda"))
        dp.dp_norms_multi(desc, dt, n, got[-1], ws)
    assert torch.equal(got[0][0, :9], got[1][0])
    want = torch.stack([(a[i].double().t().contiguous() @ g[i].double()).square().sum() for i in range(0, B, 10)])
    # exact products; sums of up to 1544 columns and T^2 pairs in fp32
    assert float(((got[0][0, ::10].double() - want) / want).abs().max()) < 1e-5


# Long contractions over ragged rows: up to 2048, 8192 and more rows a launch cuts the same tiles differently.
@pytest.mark.parametrize("B,T", [(2, 1000), (2, 1056), (3, 2752)])
def test_long_contractions_over_ragged_rows(B, T):
    from paper_2311_11822_amd import binding as dp
    d, p = 72, 51000
    gen = torch.Generator(device="cuda").manual_seed(T)
    a, g = (torch.randn((B, T, n), generator=gen, device="cuda").to(torch.bfloat16) for n in (d, p))
    C = torch.rand(B, generator=gen, device="cuda") + 0.1
    got = torch.full((d, p), 7.0, device="cuda")
    dp.dp_clipped_grad(a, g, dp.DP_BF16, B, T, d, p, C, got, 0)
    weighted = (a.double() * C.double()[:, None, None]).reshape(B * T, d).t().contiguous()
    for k in range(0, p, 4096):
        ref = weighted @ g[:, :, k:k + 4096].double().reshape(B * T, -1)
        # exact products; sums of up to 8256 of them in fp32, 16 to a matrix instruction
        assert float((got[:, k:k + 4096].double() - ref).norm() / ref.norm()) < 3e-6
