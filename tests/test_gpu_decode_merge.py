"""fp32 caches: the merge of the splits, for every number of query heads that takes another way through it, few and many splits,
a segment or both, against the oracle (the bf16 caches' merge: test_gpu_decode_splits.py)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import vector_oracle as vo
from paper_2605_23258_amd import binding as vb
from paper_2605_23258_amd import pipeline as pl
from parity_util import close

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,G", [(64, 1), (64, 8), (64, 10), (64, 16), (128, 1), (128, 2), (128, 3), (128, 5), (128, 12), (128, 16)])
@pytest.mark.parametrize("n_r,n_a", [(2, 0), (0, 3), (70, 40), (3000, 1), (2100, 1900)])
def test_f32(d, G, n_r, n_a):
    rng = np.random.default_rng(d + G + n_r)
    B, H = 2, 2
    draw = lambda *s: rng.standard_normal(s).astype(np.float32)
    q, k_ret, v_ret, k_apx, W = draw(B, H * G, d), draw(B, H, n_r + 2, d), draw(B, H, n_r + 2, d), draw(B, H, max(n_a, 1), d), draw(H, d, d) / np.float32(np.sqrt(d))
    k_ret[:, :, n_r:], v_ret[:, :, n_r:] = 1e30, -1e30        # beyond the live length
    k_ret[0, 0, :n_r // 2] *= 4                               # one split's reference far above the others'
    lens = np.array([n_r, n_r // 2], dtype=np.int32)
    dev = [pl.to_device(x) for x in (k_ret, v_ret, k_apx, W, lens)]
    cache = vb.Cache(batch=B, n_q_heads=H * G, n_kv_heads=H, head_dim=d, dtype=vb.VECTOR_F32, cap_retain=n_r + 2, n_approx=n_a)
    cache.k_ret, cache.v_ret, cache.k_apx, cache.W, cache.len_retain = (t.data_ptr() for t in dev)
    shape = vb.Shape(n_q_heads=H * G, n_kv_heads=H, head_dim=d, seq_len=max(n_r + 2, 64), window=1, pool_kernel=1, dtype=vb.VECTOR_F32)
    ws = pl.alloc_workspace(vb.vector_workspace_bytes(shape, n_a, n_a, B))
    ws.fill_(0xff)
    out = torch.full((B, H * G, d), 7.0, dtype=torch.float32, device="cuda:0")
    scale = 1.0 / np.sqrt(d)
    vb.vector_decode_attn(cache, pl.to_device(q), scale, out, ws)
    torch.cuda.synchronize()
    ref = vo.decode_attn(q, k_ret, v_ret, lens, k_apx[:, :, :n_a], W, scale)
    close(out.cpu().numpy(), ref, f"d {d} G {G} rows {n_r} + {n_a}")
