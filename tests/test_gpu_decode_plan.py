"""Decode over sequences of different lengths, cut by a plan that the launch makes from the live lengths: ranges that begin and end at
any granule of 32 rows and cross sequences, segments and sequences without rows, one long among many short ones, as many
sequences as a plan takes and one more; and a step with its token, in blocks with room and full ones.  The largest capacity that
a call states steers whether it is worth a plan: these state one that is."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import vector_oracle as vo
from paper_2605_23258_amd import binding as vb
from paper_2605_23258_amd import datagen as dg
from paper_2605_23258_amd import pipeline as pl
from parity_util import close
from test_gpu_decode_splits import run

pytestmark = pytest.mark.gpu

STEER = 1 << 20           # rows: 8192 steps, more than a plan asks for with one (sequence, KV head)


@pytest.mark.parametrize("H,lens,apxs", [
    (1, [2500, 1], [0, 0]), (2, [0, 0], [2500, 31]), (3, [0, 3000, 0, 0], [0, 0, 2000, 0]), (1, [30000, 33], [32, 9000]),
    (2, [1023, 1024, 1025, 31, 32, 33], [1025, 1024, 1023, 33, 32, 31]),
    (8, [2000 - 61 * b for b in range(24)], [1500 - 47 * b for b in range(24)]),
    (1, [5000] + [(37 * b) % 300 for b in range(63)], [1, 4000] + [(53 * b) % 200 for b in range(62)]),
    (1, [5000] + [(37 * b) % 300 for b in range(64)], [(53 * b) % 200 for b in range(65)]),
])
@pytest.mark.parametrize("rope", [False, True])
def test_lengths(H, lens, apxs, rope):
    run(128, 4, H, lens, apxs, ragged=True, rope=rope, seed=len(lens) + H, steer=STEER)


@pytest.mark.parametrize("d,G", [(64, 4), (64, 16), (128, 1), (128, 16)])
def test_other_shapes(d, G):
    run(d, G, 3, [2100, 0, 700, 1], [77, 1, 2000, 0], ragged=True, rope=d == 128 and G == 16, seed=d + G, steer=STEER)


@pytest.mark.parametrize("d", [64, 128])
def test_step(d):
    """The token of every sequence: row len of its block, of a full block nowhere; a sequence with nothing else; the lengths afterwards."""
    rng = np.random.default_rng(d)
    store = lambda a: dg.f32_to_bf16_bits(np.asarray(a, np.float32))
    H, G, lens, caps, apxs = 2, 4, [2047, 0, 640, 31, 100], [2100, 3, 640, 40, 101], [300, 0, 1500, 0, 64]
    B, Hq, scale = len(lens), H * G, 1.0 / np.sqrt(d)
    q, W = store(rng.standard_normal((B, Hq, d))), store(rng.standard_normal((H, d, d)) / np.sqrt(d))
    k, v = ([store(rng.standard_normal((H, c, d))) for c in caps] for _ in range(2))
    k_apx = [store(rng.standard_normal((H, n, d))) for n in apxs]
    k_new, v_new = store(rng.standard_normal((B, H, d))), store(rng.standard_normal((B, H, d)))
    flat = lambda rows: pl.to_device(np.concatenate([r.reshape(-1, d) for r in rows]))
    starts = lambda n: np.concatenate([[0], np.cumsum([H * x for x in n])[:-1]]).astype(np.int64)
    keep = [flat(k), flat(v), flat(k_apx), pl.to_device(W), pl.to_device(np.array(lens, np.int32))]
    keep += [pl.to_device(a) for a in (np.array(caps, np.int32), np.array(apxs, np.int32), starts(caps), starts(apxs))]
    cache = vb.Cache(batch=B, n_q_heads=Hq, n_kv_heads=H, head_dim=d, dtype=vb.VECTOR_BF16, cap_retain=STEER, n_approx=max(apxs))
    cache.k_ret, cache.v_ret, cache.k_apx, cache.W, cache.len_retain = (t.data_ptr() for t in keep[:5])
    cache.cap_retain_seq, cache.n_approx_seq, cache.ret_row_start, cache.apx_row_start = (t.data_ptr() for t in keep[5:])
    shape = vb.Shape(n_q_heads=Hq, n_kv_heads=H, head_dim=d, seq_len=max(caps), window=1, pool_kernel=1, dtype=vb.VECTOR_BF16)
    ws = pl.alloc_workspace(vb.vector_workspace_bytes(shape, max(apxs), max(apxs), B))
    ws.fill_(0xff)
    out = torch.full((B, Hq, d), 7.0, dtype=torch.float32, device="cuda:0")
    vb.vector_decode_step(cache, pl.to_device(q), pl.to_device(k_new), pl.to_device(v_new), scale, out, ws, flags=vb.VECTOR_DECODE_OUT_F32)
    torch.cuda.synchronize()
    for b, n in enumerate(lens):
        rows = [np.concatenate([x[b][:, :n], new[b][:, None]], axis=1) for x, new in ((k, k_new), (v, v_new))]
        ref = vo.decode_attn(dg.widen(q[b:b + 1]), dg.widen(rows[0])[None], dg.widen(rows[1])[None], np.array([n + 1]), dg.widen(k_apx[b])[None],
                             dg.widen(W), scale)[0]
        close(out[b].cpu().numpy(), ref, f"sequence {b}")
        if n < caps[b]:
            k[b][:, n], v[b][:, n] = k_new[b], v_new[b]
    assert np.array_equal(pl.to_host(keep[0]), np.concatenate([r.reshape(-1, d) for r in k]))
    assert np.array_equal(pl.to_host(keep[1]), np.concatenate([r.reshape(-1, d) for r in v]))
    assert np.array_equal(keep[4].cpu().numpy(), np.minimum(np.array(lens) + 1, caps))


@pytest.mark.parametrize("retained", [True, False])
def test_segment_that_the_call_leaves_out(retained):
    """A capacity of 0 for the batch leaves the segment out whatever the sequences' own counts say, and its rows need no memory."""
    rng = np.random.default_rng(retained)
    store = lambda a: dg.f32_to_bf16_bits(np.asarray(a, np.float32))
    d, H, G, rows, other = 128, 2, 4, [2300, 700, 1], [40, 300, 90]
    B, Hq, scale = len(rows), H * G, 1.0 / np.sqrt(d)
    q, W = store(rng.standard_normal((B, Hq, d))), store(rng.standard_normal((H, d, d)) / np.sqrt(d))
    k, v = ([store(rng.standard_normal((H, n, d))) for n in rows] for _ in range(2))
    flat = lambda x: pl.to_device(np.concatenate([r.reshape(-1, d) for r in x]))
    starts = lambda n: pl.to_device(np.concatenate([[0], np.cumsum([H * x for x in n])[:-1]]).astype(np.int64))
    i32 = lambda x: pl.to_device(np.array(x, np.int32))
    ret, apx = (rows, other) if retained else (other, rows)
    keep = [flat(k), flat(v), pl.to_device(W), i32(ret), i32(ret), i32(apx), starts(ret), starts(apx)]
    cache = vb.Cache(batch=B, n_q_heads=Hq, n_kv_heads=H, head_dim=d, dtype=vb.VECTOR_BF16, cap_retain=STEER if retained else 0, n_approx=0 if retained else STEER)
    cache.len_retain, cache.cap_retain_seq, cache.n_approx_seq, cache.ret_row_start, cache.apx_row_start = (t.data_ptr() for t in keep[3:])
    if retained:
        cache.k_ret, cache.v_ret = keep[0].data_ptr(), keep[1].data_ptr()
    else:
        cache.k_apx, cache.W = keep[0].data_ptr(), keep[2].data_ptr()
    shape = vb.Shape(n_q_heads=Hq, n_kv_heads=H, head_dim=d, seq_len=max(rows), window=1, pool_kernel=1, dtype=vb.VECTOR_BF16)
    ws = pl.alloc_workspace(vb.vector_workspace_bytes(shape, max(rows), max(rows), B))
    ws.fill_(0xff)
    out = torch.full((B, Hq, d), 7.0, dtype=torch.float32, device="cuda:0")
    vb.vector_decode_attn(cache, pl.to_device(q), scale, out, ws, flags=vb.VECTOR_DECODE_OUT_F32)
    torch.cuda.synchronize()
    none = np.zeros((1, H, 0, d))
    for b, n in enumerate(rows):
        kb, vbt = dg.widen(k[b])[None], dg.widen(v[b])[None]
        ref = vo.decode_attn(dg.widen(q[b:b + 1]), kb if retained else none, vbt if retained else none, np.array([n if retained else 0]),
                             none if retained else kb, dg.widen(W), scale)[0]
        close(out[b].cpu().numpy(), ref, f"sequence {b}")
