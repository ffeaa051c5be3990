"""Average pooling without a division: sum * (1 / k), corrected by the remainder, is the correctly rounded quotient."""
import ctypes
import ctypes.util

import numpy as np
import pytest

F = np.float32
_libm = ctypes.CDLL(ctypes.util.find_library("m") or "libm.so.6")
_libm.fmaf.restype = ctypes.c_float
_libm.fmaf.argtypes = [ctypes.c_float] * 3


def corrected(sums, k):
    """What the kernels compute, with the C library's fused multiply-add."""
    inv, kf, fma = F(1.0) / F(k), F(k), _libm.fmaf
    return np.array([fma(fma(-q, kf, s), inv, q) for s, q in zip(sums, (sums * inv).astype(F))], F)


@pytest.mark.parametrize("k", [1, 3, 5, 7, 9, 11, 13, 101, 127, 1001, 65537, 2097151])
def test_correction_gives_the_rounded_quotient(k):
    rng = np.random.default_rng(k)
    sums = (rng.random(6000) * 2.0 ** rng.integers(-148, 1, 6000)).astype(F)          # normal, denormal, zero
    mid = (rng.integers(1 << 23, 1 << 24, 6000) + 0.5) * 2.0 ** rng.integers(-60, -24, 6000)
    near = (mid * k).astype(F)                                                         # quotients next to a tie
    for s in (sums, near, np.nextafter(near, F(0)), np.nextafter(near, F(np.inf)), np.array([0, 2.0 ** -149, 2.0 ** -126, 1.0], F)):
        assert np.array_equal(corrected(s, k).view(np.uint32), (s / F(k)).view(np.uint32))


@pytest.mark.gpu
@pytest.mark.parametrize("kernel", [3, 5, 7, 9, 13, 101])
@pytest.mark.parametrize("n", [1500, 17000])             # pooled in the routing's one launch, and in its first of two
def test_pooled_scores_are_ordered_sums_divided(kernel, n):
    torch = pytest.importorskip("torch")
    from paper_2605_23258_amd import binding as vb
    from paper_2605_23258_amd import pipeline as pl
    H, w, d = 2, 16, 64
    g = torch.Generator(device="cuda").manual_seed(kernel)
    q, k, v = (torch.randn(H, r, d, generator=g, device="cuda") for r in (w, n, n))
    W = torch.randn(H, d, d, generator=g, device="cuda")

    def shape(pool):
        return vb.Shape(n_q_heads=H, n_kv_heads=H, head_dim=d, seq_len=n, window=w, pool_kernel=pool, dtype=vb.VECTOR_F32)
    ws = pl.alloc_workspace(vb.vector_workspace_bytes(shape(1), 100, 50))
    mass, score = (torch.empty(H, n, device="cuda") for _ in range(2))
    vb.vector_score(shape(1), q, k, mass, ws)
    vb.vector_score(shape(kernel), q, k, score, ws)
    out = pl.alloc_outputs(shape(kernel), 100, 50, 50, torch.float32)
    ws_c = pl.alloc_workspace(vb.vector_compress_workspace_bytes(shape(kernel), 100, 50))
    pl.compress_layer(shape(kernel), q, k, v, W, 100, 50, out, ws_c, one_call=True)
    torch.cuda.synchronize()
    m = np.zeros((H, n - w + 2 * (kernel // 2)), F)
    m[:, kernel // 2: kernel // 2 + n - w] = mass.cpu().numpy()[:, : n - w]
    acc = np.zeros((H, n - w), F)
    for j in range(kernel):                                                           # ascending tokens, fp32
        acc = (acc + m[:, j: j + n - w]).astype(F)
    want = (acc / F(kernel)).view(np.uint32)
    for got in (score, out.score):
        assert np.array_equal(got.cpu().numpy()[:, : n - w].view(np.uint32), want)
