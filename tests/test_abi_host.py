"""Host-only checks of the C-ABI library (no GPU): it loads, exports every symbol the header
declares, and its pure host functions and argument validation behave as documented."""
import os
import re

import numpy as np
import pytest

import synth_inputs as si
from oracle import bk_oracle as o

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def dp():
    import paper_2311_11822_amd.binding as b
    return b


def declared_functions():
    text = open(os.path.join(ROOT, "include", "dp_bk.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(dp_[a-z0-9_]+)\s*\(", text)))


def test_library_exports_every_declared_symbol(dp):
    names = declared_functions()
    assert {"dp_ghost_norm", "dp_perex_norm", "dp_clip_factors", "dp_clipped_grad", "dp_add_noise"} <= set(names)
    for name in names:
        assert hasattr(dp.lib, name), name
    assert sorted(dp.EXPORTS) == names          # the binding covers the whole header


def test_status_strings(dp):
    seen = {dp.lib.dp_status_string(s) for s in range(5)}
    assert len(seen) == 5 and all(seen)
    assert dp.dp_version() >= 100


def test_path_rule_matches_oracle_reading(dp):
    for w in si.WORKLOADS.values():
        for d, p in w.layers:
            assert dp.dp_choose_path(w.T, d, p) == o.choose_path(w.T, d, p)
    for T, d, p in [(8, 16, 8), (8, 16, 7), (1, 1, 2), (1, 1, 1), (3037000500, 2 ** 31, 2 ** 31), (2 ** 31, 2 ** 31, 2 ** 31)]:
        assert dp.dp_choose_path(T, d, p) == o.choose_path(T, d, p), (T, d, p)


def test_workspace_sizes(dp):
    assert dp.dp_norm_workspace_bytes(0, 1, 16, 256, 768, 2304) >= 16 * 4      # at least one partial per sample
    assert dp.dp_norm_workspace_bytes(0, 1, 0, 256, 768, 2304) == 0
    assert dp.dp_norm_workspace_bytes(0, 1, 1, 256, 12, 8) == 0       # bf16 row not a multiple of 16 B
    assert dp.dp_norm_workspace_bytes(1, 0, 4, 8, 16, 16) > 0
    layers = [(None, None, 256, 768, 768, 0), (None, None, 256, 768, 3072, 1)]
    both = dp.dp_norms_multi_workspace_bytes(layers, 1, 16)
    assert both == sum(dp.dp_norm_workspace_bytes(path, 1, 16, T, d, p) for _, _, T, d, p, path in layers)


# Layer-wise pass: layers that fit one workgroup tile take the one-kernel form, which keeps no per-sample gradients, where it is
# the faster one: many samples, however few layers; not few long samples, nor tall and wide strips of many tokens together.
@pytest.mark.parametrize("B,T,dims,one_kernel", [
    (8192, 128, [(256, 8)] * 2, True), (4096, 128, [(512, 16)] * 16, True), (1024, 1024, [(128, 128)] * 8, True),
    (1024, 256, [(512, 16)] * 80, True), (256, 128, [(128, 128)] * 8, True),
    (8, 2048, [(128, 128)] * 8, False), (1024, 256, [(512, 16), (16, 512)] * 12, False),
    (256, 128, [(192, 32), (32, 192)] * 6, False), (2048, 600, [(32, 32)] * 16, False)])
def test_layerwise_form(dp, B, T, dims, one_kernel):
    layers = [(None, None, T, d, p, dp.DP_PATH_PEREX) for d, p in dims]
    norms = dp.dp_norms_multi_workspace_bytes(layers, dp.DP_BF16, B)
    kept = dp.dp_layerwise_workspace_bytes(layers, dp.DP_BF16, B) - norms
    each = 4 * sum(d * p for d, p in dims)
    assert kept <= 256 * each if one_kernel else kept >= min(B * each, 2 ** 31 - 4 * max(d * p for d, p in dims) * B)


def test_validation_refuses_before_any_launch(dp):
    lib, INV = dp.lib, dp.DP_ERR_INVALID_ARG
    fake = 0x1000                     # never dereferenced: every call below fails validation
    assert lib.dp_ghost_norm(None, fake, 1, 1, 8, 8, 8, fake, fake, 64, None) == INV
    assert lib.dp_perex_norm(fake, fake, 1, 1, 8, 8, 8, None, fake, 64, None) == INV
    assert lib.dp_ghost_norm(fake, fake, 1, 1, 8, 8, 8, fake, None, 0, None) == dp.DP_ERR_WORKSPACE
    assert lib.dp_clip_factors(fake, 0, 1, 0, 1.0, 0.01, fake, None, None) == INV
    assert lib.dp_clip_factors(fake, 1, 1, 0, -1.0, 0.01, fake, None, None) == INV
    assert lib.dp_clipped_grad(fake, fake, 1, 1, 8, 8, 8, fake, None, 0, None) == INV
    assert lib.dp_add_noise(fake, 0, 16, float("nan"), 1.0, 0, 0, None) == INV
    assert lib.dp_add_noise(fake, 0, 16, 0.0, float("inf"), 0, 0, None) == dp.DP_OK   # sigma = 0: no-op
    assert lib.dp_philox_blocks(None, 0, 4, 0, 0, None) == INV
    with pytest.raises(dp.DpError):
        dp.dp_clip_factors(fake, 1, 1, 5, 1.0, 0.01, fake, stream=0)


def test_validation_of_the_later_entry_points(dp):
    import ctypes as C
    lib, INV = dp.lib, dp.DP_ERR_INVALID_ARG
    fake = 0x1000                     # never dereferenced: every call below fails validation
    arr = dp.layer_array([(fake, fake, 8, 8, 8, 0)])
    gp = (C.c_void_p * 1)(fake)
    offs = (C.c_uint64 * 1)(0)
    # fp16 is a storage type like bf16: rows must be multiples of 16 bytes
    assert dp.dp_norm_workspace_bytes(0, dp.DP_F16, 4, 256, 768, 768) == dp.dp_norm_workspace_bytes(0, dp.DP_BF16, 4, 256, 768, 768)
    assert dp.dp_norm_workspace_bytes(0, dp.DP_F16, 1, 256, 12, 8) == 0
    assert dp.dp_norm_workspace_bytes(0, 3, 4, 256, 768, 768) == 0                   # unknown dtype
    # gradients with noise
    assert lib.dp_clipped_grad_noise_multi(arr, 1, 1, 1, fake, gp, None, 0, 0, 16, 1.0, 1.0, 0, 0, None) == INV
    assert lib.dp_clipped_grad_noise_multi(arr, 1, 1, 1, fake, gp, offs, 0, 0, 16, float("nan"), 1.0, 0, 0, None) == INV
    assert lib.dp_clipped_grad_noise_multi(arr, 1, 1, 1, fake, gp, offs, 0, 0, 16, 1.0, 0.0, 0, 0, None) == INV
    assert lib.dp_clipped_grad_noise_multi(arr, 1, 1, 1, fake, gp, offs, 0, 2 ** 64 - 1, 2, 1.0, 1.0, 0, 0, None) == INV
    assert lib.dp_clipped_grad_noise_multi(arr, 1, 1, 0, fake, gp, offs, 0, 0, 16, 1.0, 1.0, 0, 0, None) == INV   # B = 0
    # group-wise clipping
    begin, R = (C.c_int32 * 3)(0, 1, 2), (C.c_float * 2)(1.0, 1.0)
    assert lib.dp_clip_factors_grouped(fake, 2, 4, begin, 2, R, 0, 0.01, None, None, None) == INV
    assert lib.dp_clip_factors_grouped(fake, 2, 4, None, 2, R, 0, 0.01, fake, None, None) == INV
    bad_begin = (C.c_int32 * 3)(0, 2, 1)                                            # not monotone
    assert lib.dp_clip_factors_grouped(fake, 2, 4, bad_begin, 2, R, 0, 0.01, fake, None, None) == INV
    bad_R = (C.c_float * 2)(1.0, -1.0)
    assert lib.dp_clip_factors_grouped(fake, 2, 4, begin, 2, bad_R, 0, 0.01, fake, None, None) == INV
    gol = (C.c_int32 * 1)(3)                                                         # group out of range
    assert lib.dp_clipped_grad_grouped(arr, 1, 1, 1, fake, gol, 2, gp, 0, None) == INV
    assert dp.dp_group_noise_threshold([3.0, 4.0]) == 5.0
    # bias
    assert lib.dp_bias_norm(None, 1, 1, 8, 8, fake, fake, None) == INV
    assert lib.dp_bias_norm(fake, 1, 1, 8, 12, fake, fake, None) == INV             # 16-bit row not 16 B
    assert lib.dp_clipped_bias_grad(fake, 1, 8, None, fake, 0, None) == INV
    assert lib.dp_clipped_bias_grad(fake, 1, 8, fake, fake, 2, None) == INV


# Every refusal of a whole step's gradient half comes before its norms are launched: without a GPU a launch would give
# DP_ERR_HIP, on a GPU the norms would have been overwritten (test_refused_step_touches_nothing).
@pytest.mark.parametrize("keeps", [False, True])
@pytest.mark.parametrize("bad", [
    dict(sigma=-1.0), dict(sigma=float("nan")), dict(sigma=float("inf")), dict(R=float("inf")), dict(R=0.0), dict(accumulate=2),
    dict(shard=(2 ** 64 - 1, 2)), dict(grad=0x1004), dict(grad=None), dict(grads=None), dict(offsets=None), dict(offset=2 ** 64 - 1),
    dict(counter=0x1002), dict(mode=2), dict(stability=-1.0), dict(C=None), dict(sqnorm=None), dict(ws=None),
])
def test_step_refuses_before_any_launch(dp, bad, keeps):
    import ctypes as C
    fake = 0x1000
    layers = dp.layer_array([(fake, fake, 64, 8, 8, dp.DP_PATH_PEREX), (fake, fake, 64, 8, 8, dp.DP_PATH_GHOST)])
    ok = dict(sigma=1.0, R=1.0, accumulate=0, shard=(0, 128), grad=fake, grads=(), offsets=(), offset=64, counter=fake, mode=0,
              stability=0.01, C=fake, sqnorm=fake, ws=fake)
    a = dict(ok, **bad)
    kept = (C.c_void_p * 2)(fake, None) if keeps else None
    grads = (C.c_void_p * 2)(fake, a["grad"]) if a["grads"] is not None else None
    offsets = (C.c_uint64 * 2)(0, a["offset"]) if a["offsets"] is not None else None
    st = dp.lib.dp_private_step_multi(layers, 2, dp.DP_BF16, 4, a["mode"], a["R"], a["stability"], kept, grads, offsets,
                                      a["accumulate"], *a["shard"], a["sigma"], 0, 0, a["sqnorm"], a["C"], None, a["ws"],
                                      1 << 20, a["counter"], None)
    assert st == (dp.DP_ERR_WORKSPACE if bad == dict(ws=None) else dp.DP_ERR_INVALID_ARG)


def test_step_refuses_what_fp32_layers_refuse(dp):
    import ctypes as C
    fake = 0x1000
    grads = (C.c_void_p * 1)(fake)
    step = lambda T, d, kept: dp.lib.dp_private_step_multi(
        dp.layer_array([(fake, fake, T, d, d, dp.DP_PATH_PEREX)]), 1, dp.DP_F32, 1, 0, 1.0, 0.01, kept, grads, None, 0, 0, 0,
        0.0, 0, 0, fake, fake, None, None, 0, None, None)
    assert step(4096, 4096, None) == dp.DP_ERR_UNSUPPORTED                         # more than 2^28 multiply-adds a sample
    assert step(8, 8, (C.c_void_p * 1)(fake)) == dp.DP_ERR_UNSUPPORTED             # kept gradients are for 16-bit layers


# ----------------------------------------------------------------------------
# tile orders of the large-tile kernels: every tile exactly once, for any shape
# ----------------------------------------------------------------------------

GRAD_SHAPES = sorted({(d, p) for w in si.WORKLOADS.values() for d, p in w.layers if d >= 128} |
                     {(136, 264), (4360, 3848), (1800, 1544), (256, 256), (257, 255), (12288, 256), (256, 49152),
                      (4352, 8448), (8704, 4352), (17 * 256, 33 * 256), (70 * 256 - 8, 41 * 256 + 8)})


@pytest.mark.parametrize("d,p", GRAD_SHAPES)
def test_gradient_tile_order_is_a_bijection(dp, d, p):
    r, c = dp.dp_clipped_grad_tile_order(d, p)
    tiles_m, tiles_n = -(-d // 256), -(-p // 256)
    assert len(r) == tiles_m * tiles_n
    assert np.all(r % 256 == 0) and np.all(c % 256 == 0)
    seen = np.zeros((tiles_m, tiles_n), dtype=np.int64)
    np.add.at(seen, (r // 256, c // 256), 1)
    assert np.all(seen == 1)


def test_gradient_tile_order_keeps_patches_together(dp):
    # the 32 tiles one XCD takes in a round (workgroups x, x + 8, ... of a run of 256) form a
    # patch of at most 4 tile rows x 8 tile columns
    r, c = dp.dp_clipped_grad_tile_order(12288, 36864)
    for base in (0, 256, 256 * 13):
        for x in range(8):
            ids = base + x + 8 * np.arange(32)
            rows, cols = np.unique(r[ids] // 256), np.unique(c[ids] // 256)
            assert len(rows) <= 4 and len(cols) <= 8 and len(rows) * len(cols) == 32


@pytest.mark.parametrize("T,B", [(2048, 4), (512, 8), (256, 16), (96, 3), (130, 2), (300, 2), (1024, 3), (1025, 3),
                                 (1152, 2), (2049, 1), (3000, 2), (4096, 2), (5000, 1), (8192, 1), (2304, 5)])
def test_ghost_tile_order_is_a_bijection(dp, T, B):
    sample, r0, c0, slot = dp.dp_ghost_tile_order(T, B)
    nj, ni = -(-T // 128), -(-T // 256)
    tps = sum(nj - 2 * I for I in range(ni))
    assert len(sample) == B * tps
    I, J = r0 // 256, c0 // 128
    assert np.all((sample >= 0) & (sample < B) & (I >= 0) & (I < ni) & (J >= 2 * I) & (J < nj))
    seen = np.zeros((B, ni, nj), dtype=np.int64)
    np.add.at(seen, (sample, I, J), 1)
    want = np.zeros((ni, nj), dtype=np.int64)
    for i in range(ni):
        want[i, 2 * i:] = 1
    assert np.all(seen == want[None])
    # partial-sum slots: each used once, and a sample's slots are contiguous
    assert sorted(slot.tolist()) == list(range(B * tps))
    assert np.all(slot // tps == sample)


def sub_tile_order(n_tail, side):
    """Tiles of a sub-tile launch by the workgroup of their first sub-tile: workgroup b runs on XCD b % 8, each XCD
    takes a contiguous run of each 256 of the side x side sub-tiles of every tile."""
    total = n_tail * side * side
    order = []
    for base in range(0, total, 256):
        part = np.arange(base, min(base + 256, total))
        runs = np.array_split(part, 8)                       # the first len % 8 runs are one longer
        order += [runs[b % 8][b // 8] for b in range(len(part))]
    return [w // (side * side) for w in order if w % (side * side) == 0]


# A launch may be cut whole into 128 x 128 (edges would leave 256 x 256 mostly empty), in its last round, or its last
# tiles into 64 x 64.
@pytest.mark.parametrize("d,p,n_tail,side", [
    (264, 16640, 130, 2), (72, 120000, 469, 2), (136, 70000, 18, 4), (1032, 8200, 0, 4), (4352, 8448, 49, 2), (1800, 1544, 56, 2),
    (256, 256, 1, 4), (8192, 2304, 32, 4), (8192, 2560, 64, 2), (12288, 12288, 0, 4)])
def test_gradient_tile_order_of_cut_tiles(dp, d, p, n_tail, side):
    r, c = dp.dp_clipped_grad_tile_order(d, p)
    tiles_m, tiles_n = -(-d // 256), -(-p // 256)
    assert len(r) == tiles_m * tiles_n and len(set(zip(r.tolist(), c.tolist()))) == len(r)
    # the numbering behind the order: a launch of as many tiles whose first workgroups are all there is
    number = {}
    for q, t in enumerate(grad_tiles_in_number_order(tiles_m, tiles_n)):
        number[t] = q
    got = [number[(y // 256, x // 256)] for y, x in zip(r[len(r) - n_tail:].tolist(), c[len(r) - n_tail:].tolist())]
    assert got == [len(r) - n_tail + t for t in sub_tile_order(n_tail, side)]


# The kernels that a gradient of n square layers takes: joined tiles, one workgroup a tile, tiles that are cut.
@pytest.mark.parametrize("n,side,B,T,want", [
    (8, 2040, 3, 64, (512, 256, 1, 0)), (11, 2040, 64, 64, (704, 256, 1, 0)), (8, 2040, 65, 64, (512, 512, 1, 0)),
    (9, 1016, 4, 160, (144, 144, 0, 0)), (12, 1016, 4, 160, (192, 192, 0, 0)), (9, 1016, 7, 160, (144, 144, 0, 0)),
    (12, 1016, 7, 160, (192, 192, 1, 0)), (16, 1016, 4, 256, (256, 256, 0, 0)), (17, 1024, 4, 256, (256, 256, 1, 16)),
    (12, 1024, 8, 64, (0, 0, 1, 192)), (13, 1024, 8, 64, (208, 208, 0, 0)), (13, 1024, 4, 64, (0, 0, 1, 208)), (8, 2040, 16, 48, (512, 512, 0, 0)),
    (2, 512, 3, 64, (0, 0, 1, 8)), (1, 1536, 5, 64, (0, 0, 1, 36)), (17, 168, 4, 1024, (0, 0, 1, 17)), (16, 168, 4, 1024, (0, 0, 1, 16)),
    (17, 168, 3, 1024, (0, 0, 1, 17)), (17, 224, 4, 1024, (0, 0, 1, 17)), (17, 168, 14, 320, (0, 0, 1, 17)), (17, 168, 11, 384, (0, 0, 1, 17)), (18, 1000, 4, 1024, (256, 256, 1, 32))])
def test_launches_of_a_gradient(dp, n, side, B, T, want):
    plan = dp.dp_clipped_grad_launches([(16, 16, T, side, side, 0)] * n, dp.DP_BF16, B)
    assert (plan["tiles"], plan["workgroups"], plan["whole_blocks"], plan["cut"]) == want
    assert plan["tiles"] + plan["cut"] == n * (-(-side // 256)) ** 2
    small = 16 if side % 32 and T >= 384 and B * T >= 4096 else 32
    assert not plan["cut"] or plan["side"] == (4 if plan["cut"] <= small else 2)


def test_launches_of_a_gradient_refused(dp):
    query = lambda n, T, side, dt: dp.dp_clipped_grad_launches([(16, 16, T, side, side, 0)] * n, dt, 4)
    for n, T, side, dt in [(49, 64, 256, dp.DP_BF16), (1, 8, 256, dp.DP_BF16), (1, 64, 256, dp.DP_F32), (1, 64, 250, dp.DP_BF16),
                           (1, 0, 256, dp.DP_F16)]:
        with pytest.raises(dp.DpError):
            query(n, T, side, dt)


def grad_tiles_in_number_order(tiles_m, tiles_n):
    """Tile numbers of a layer: super-patches of 16 x 16 row by row, in them patches of 4 x 8, in them columns."""
    for sr in range(0, tiles_m, 16):
        for sc in range(0, tiles_n, 16):
            for pr in range(sr, min(sr + 16, tiles_m), 4):
                for pc in range(sc, min(sc + 16, tiles_n), 8):
                    for tn in range(pc, min(pc + 8, sc + 16, tiles_n)):
                        for tm in range(pr, min(pr + 4, sr + 16, tiles_m)):
                            yield tm, tn


@pytest.mark.parametrize("missing", ["_cuda_getCurrentRawStream", "_cuda_getDevice"])
def test_current_stream_without_torch_private_functions(dp, monkeypatch, missing):
    torch = pytest.importorskip("torch")
    from types import SimpleNamespace
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: SimpleNamespace(cuda_stream=77))
    for name in ("_cuda_getCurrentRawStream", "_cuda_getDevice"):
        monkeypatch.setattr(torch._C, name, lambda *a: 78, raising=False)
    assert dp._stream(None) == 78
    monkeypatch.delattr(torch._C, missing)
    assert dp._stream(None) == 77
    assert dp._stream(5) == 5


def test_native_argument_conversion(dp):
    """What the native conversion does not take reaches ctypes and is refused as it always was; statuses raise."""
    import ctypes
    import numpy as np
    with pytest.raises(dp.DpError) as e:
        dp.dp_bias_norm(None, dp.DP_BF16, 4, 8, 64, None, None, stream=0)
    assert e.value.status == dp.DP_ERR_INVALID_ARG and "dp_bias_norm" in str(e.value)
    with pytest.raises(dp.DpError):
        dp.dp_clipped_grad_multi(dp.layer_array([(16, 16, 4, 8, 8, 0)]), dp.DP_BF16, 1, None, [16], stream=0)
    with pytest.raises(ctypes.ArgumentError):
        dp.dp_bias_norm(16, 1.5, 4, 8, 64, 16, 16, stream=0)
    with pytest.raises(ctypes.ArgumentError):
        dp.dp_clip_factors(16, 1, 1, dp.DP_CLIP_STANDARD, "R", 0.01, 16, None, 0)
    with pytest.raises(AttributeError):
        dp.dp_bias_norm(np.zeros(64, dtype=np.float32), dp.DP_F32, 1, 1, 64, 16, 16, stream=0)    # host memory, no data_ptr


def native_calls(dp):
    """Every call with native argument conversion, by arguments that ctypes takes and the library refuses (B = 0)."""
    import ctypes as C
    layers, grads, offs = dp.layer_array([(16, 16, 4, 8, 8, 0)]), (C.c_void_p * 1)(16), (C.c_uint64 * 1)(0)
    return {
        "dp_ghost_norm": dict(a=16, g=16, dt=1, B=0, T=4, d_in=8, d_out=8, sqnorm_out=16, ws=None),
        "dp_perex_norm": dict(a=16, g=16, dt=1, B=0, T=4, d_in=8, d_out=8, sqnorm_out=16, ws=None),
        "dp_clip_factors": dict(sqnorm=16, L=1, B=0, mode=0, R=1.0, stability=0.01, C_out=16, norm_out=None),
        "dp_clipped_grad": dict(a=16, g=16, dt=1, B=0, T=4, d_in=8, d_out=8, Cf=16, grad=16),
        "dp_add_noise": dict(grad_slice=16, global_offset=0, count=4, sigma=-1.0, R=1.0, seed=0, step=0),
        "dp_norms_multi": dict(layers=layers, dt=1, B=0, sqnorm_out=16, ws=None),
        "dp_clipped_grad_multi": dict(layers=layers, dt=1, B=0, Cf=16, grads=grads),
        "dp_clipped_grad_noise_multi": dict(layers=layers, dt=1, B=0, Cf=16, grads=grads, grad_offset=offs, accumulate=0,
                                            shard_offset=0, shard_count=4, sigma=1.0, R=1.0, seed=0, step=0),
        "dp_clipped_grad_noise_multi_h16": dict(layers=layers, dt=1, B=0, Cf=16, grads16=grads, grad_offset=offs, accumulate=0,
                                                shard_offset=0, shard_count=4, sigma=1.0, R=1.0, seed=0, step=0),
        "dp_bias_norm": dict(g=16, dt=1, B=0, T=4, d_out=8, colsum=16, sqnorm_out=16),
        "dp_clipped_bias_grad": dict(colsum=16, B=0, d_out=8, Cf=16, grad_b=16),
        "dp_norms_multi_keep": dict(layers=layers, dt=1, B=0, sqnorm_out=16, kept=grads, ws=None),
        "dp_clipped_grad_kept_multi": dict(layers=layers, dt=1, B=0, Cf=16, kept=grads, grads=grads, grad_offset=offs,
                                           accumulate=0, shard_offset=0, shard_count=4, sigma=1.0, R=1.0, seed=0, step=0),
        "dp_private_step_multi": dict(layers=layers, dt=1, B=0, mode=0, R=1.0, stability=0.01, kept=grads, grads=grads,
                                      grad_offset=offs, accumulate=0, shard_offset=0, shard_count=4, sigma=1.0, seed=0, step=0,
                                      sqnorm_out=16, C_out=16, norm_out=None, ws=None, counter=None),
        "dp_layerwise_clipped_grad": dict(layers=layers, dt=1, B=0, R=[1.0], mode=0, stability=0.01, grads=grads,
                                          grad_offset=offs, accumulate=0, shard_offset=0, shard_count=4, sigma=1.0, seed=0,
                                          step=0, sqnorm_out=16, C_out=16, ws=None),
    }


HOST_ARRAYS = ("layers", "grads", "grads16", "kept", "grad_offset")
DEVICE_POINTERS = ("a", "g", "sqnorm_out", "sqnorm", "C_out", "norm_out", "Cf", "grad", "grad_slice", "colsum", "grad_b", "counter")


def test_arrays_are_taken_where_and_as_ctypes_takes_them(dp):
    """A host array is no device pointer, and its elements are of the prototype's type; nothing is read of one that is not."""
    import ctypes as C
    calls = native_calls(dp)
    assert not dp._pycall or set(calls) == {n for n in dir(dp._pycall) if n.startswith("dp_")}
    wrong = {"layers": [C.c_uint8, C.c_void_p], "grad_offset": [C.c_uint32, C.c_float, C.c_void_p]}
    for name, args in calls.items():
        call = getattr(dp, name)
        with pytest.raises(dp.DpError) as e:
            call(**args, stream=0)
        assert e.value.status == dp.DP_ERR_INVALID_ARG, name
        for key in args:
            if key in HOST_ARRAYS:
                for t in wrong.get(key, [C.c_uint32, C.c_float, C.c_uint64, dp.dp_layer]):
                    with pytest.raises(C.ArgumentError):
                        call(**dict(args, **{key: (t * 1)()}), stream=0)
            if key in DEVICE_POINTERS:
                with pytest.raises(AttributeError):
                    call(**dict(args, **{key: (C.c_float * 64)()}), stream=0)


def test_calls_without_the_native_conversion(dp, monkeypatch):
    """A library that was built without it, or for another Python, is called through ctypes alone."""
    import subprocess
    import sys
    code = ("import sys; sys.modules['paper_2311_11822_amd._pycall'] = None\n"            # its import fails
            "from paper_2311_11822_amd import binding as dp\n"
            "assert dp._pycall is None and dp.dp_version() >= 100\n"
            "try: dp.dp_bias_norm(None, 1, 4, 8, 64, None, None, stream=0)\n"
            "except dp.DpError as e: assert e.status == dp.DP_ERR_INVALID_ARG\n"
            "else: assert False")
    subprocess.run([sys.executable, "-c", code], cwd=ROOT, check=True)
    monkeypatch.setattr(dp, "_pycall", None)
    for name, args in native_calls(dp).items():
        with pytest.raises(dp.DpError) as e:
            getattr(dp, name)(**args, stream=0)
        assert e.value.status == dp.DP_ERR_INVALID_ARG, name
