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
