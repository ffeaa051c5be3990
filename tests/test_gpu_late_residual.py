"""Rotated keys, and fp32 keys: the residual's products come a tile after the scores.  Each of these kernels, with one and with
several tiles per workgroup, a partial last tile, row indices and position arrays, both pairings, against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import vector_oracle as vo
from paper_2605_23258_amd import binding as vb
from paper_2605_23258_amd import datagen as dg
from paper_2605_23258_amd import pipeline as pl
from parity_util import close

pytestmark = pytest.mark.gpu

# head_dim, query heads per KV head, window: 128, 256 and 512 query rows (fp32 at 128 dims: no more than 256 at a time)
KERNELS = [("bf16", 128, 1, 16), ("bf16", 128, 4, 64), ("bf16", 128, 8, 64), ("bf16", 64, 2, 32), ("bf16", 64, 4, 64), ("bf16", 64, 8, 64),
           ("f32", 64, 1, 16), ("f32", 64, 8, 32), ("f32", 64, 8, 64), ("f32", 128, 1, 16), ("f32", 128, 4, 64)]
# KV heads and tokens: a partial tile, whole tiles, one to five tiles per workgroup
SIZES = [(1, 70), (2, 128), (3, 333), (64, 650), (48, 1100)]


@pytest.mark.parametrize("dtype,d,G,w,rotated", [k + (True,) for k in KERNELS] + [k + (False,) for k in KERNELS if k[0] == "f32"])
@pytest.mark.parametrize("H,n", SIZES)
def test_residual_and_score(dtype, d, G, w, rotated, H, n):
    if H >= 48 and G * w > 256:
        H //= 4
    rng = np.random.default_rng(d + G + w + H + n)
    interleaved = (n + G) % 2 == 1
    store = (lambda a: dg.f32_to_bf16_bits(a.astype(np.float32))) if dtype == "bf16" else (lambda a: a.astype(np.float32))
    wide = dg.widen if dtype == "bf16" else (lambda a: a)
    draw = lambda *s: rng.standard_normal(s)
    q, k, v, W = store(draw(H * G, w, d)), store(draw(H, n, d)), store(draw(H, n, d)), store(draw(H, d, d) / np.sqrt(d))
    inv = dg.rotary_inv_freq(d, 500000.0)
    pos = rng.integers(0, 100000, n).astype(np.int32) if n % 2 else np.arange(n, dtype=np.int32) + 17
    rope, keep = vb.make_rope(inv, pl.to_device(pos) if n % 2 else None, interleaved, 0 if n % 2 else 17)
    shape = vb.Shape(n_q_heads=H * G, n_kv_heads=H, head_dim=d, seq_len=n, window=w, pool_kernel=7, dtype=vb.VECTOR_BF16 if dtype == "bf16" else vb.VECTOR_F32)
    ws = pl.alloc_workspace(vb.vector_workspace_bytes(shape, n // 4, n // 8, 1))
    ws.fill_(0xff)
    score, eps, alone = (torch.full((H, n), -1.0, device="cuda:0") for _ in range(3))
    dev = [pl.to_device(x) for x in (q, k, v, W)]
    if rotated:
        vb.vector_score_residual_rope(shape, *dev, rope, score, eps, ws)
        vb.vector_residual_rope(shape, *dev[1:], rope, alone, ws)
    else:
        vb.vector_score_residual(shape, *dev, score, eps, ws)
        vb.vector_residual(shape, *dev[1:], alone, ws)
    torch.cuda.synchronize()
    del keep
    some = np.unique(np.linspace(0, H - 1, 6).astype(int))               # heads held against the oracle
    ref = vo.residual(wide(k)[some], wide(v)[some], wide(W)[some], **(dict(pos=pos, inv_freq=inv, interleaved=interleaved) if rotated else {}))
    close(eps.cpu().numpy()[some], ref, "residual beside the score")
    close(alone.cpu().numpy()[some], ref, "residual alone")
    rows = (some[:, None] * G + np.arange(G)).ravel()
    ref = vo.score(wide(q)[rows], wide(k)[some], w, 7)
    got = score.cpu().numpy()[some]
    assert np.isposinf(got[:, n - w:]).all()
    close(got[:, :n - w].astype(np.float64) * n, ref[:, :n - w].astype(np.float64) * n, "score")
