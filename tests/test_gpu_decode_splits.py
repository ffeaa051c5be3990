"""How decode attention shares out the cache: every number of query heads per KV head that has a kernel, few and many
pieces per segment, sequences of very different lengths (in one uniform block each, or in blocks of their own), empty
segments and sequences, live lengths on the edges of the 128-row steps, against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import vector_oracle as vo
from paper_2605_23258_amd import binding as vb
from paper_2605_23258_amd import datagen as dg
from paper_2605_23258_amd import pipeline as pl
from parity_util import close

pytestmark = pytest.mark.gpu

THETA = 10000.0


def run(d, G, H, lens, apxs, ragged, rope=False, literal=False, seed=0):
    """One attention over sequences of lens[b] retained and apxs[b] approximated rows; `ragged`: blocks of their own."""
    rng = np.random.default_rng(seed)
    store = lambda a: dg.f32_to_bf16_bits(a.astype(np.float32))
    B, Hq = len(lens), H * G
    if not ragged:
        assert len(set(apxs)) == 1
    caps = [n + 3 + b % 2 for b, n in enumerate(lens)] if ragged else [max(lens) + 5] * B
    q, W = store(rng.standard_normal((B, Hq, d))), store(rng.standard_normal((H, d, d)) / np.sqrt(d))
    k_ret, v_ret = ([store(rng.standard_normal((H, c, d))) for c in caps] for _ in range(2))
    k_apx = [store(rng.standard_normal((H, n, d))) for n in apxs]
    for b, n in enumerate(lens):                 # rows beyond the live length must never reach the result
        k_ret[b][:, n:] = store(np.full((1,), 1e30))[0]
        v_ret[b][:, n:] = store(np.full((1,), -1e30))[0]
    pos = [rng.integers(0, 100000, (H, n)).astype(np.int32) for n in apxs]
    scale, inv = 1.0 / np.sqrt(d), dg.rotary_inv_freq(d, THETA)
    flat = lambda rows: pl.to_device(np.concatenate([r.reshape(-1, d) for r in rows] + [np.zeros((1, d), np.uint16)]))
    keep = [flat(k_ret), flat(v_ret), flat(k_apx), pl.to_device(W), pl.to_device(np.array(lens, dtype=np.int32))]
    cache = vb.Cache(batch=B, n_q_heads=Hq, n_kv_heads=H, head_dim=d, dtype=vb.VECTOR_BF16, cap_retain=max(caps), n_approx=max(apxs))
    cache.k_ret, cache.v_ret, cache.k_apx, cache.W, cache.len_retain = (t.data_ptr() for t in keep)
    if ragged:
        starts = lambda n: np.concatenate([[0], np.cumsum([H * x for x in n])[:-1]]).astype(np.int64)
        keep += [pl.to_device(a) for a in (np.array(caps, np.int32), np.array(apxs, np.int32), starts(caps), starts(apxs))]
        cache.cap_retain_seq, cache.n_approx_seq, cache.ret_row_start, cache.apx_row_start = (t.data_ptr() for t in keep[5:])
    shape = vb.Shape(n_q_heads=Hq, n_kv_heads=H, head_dim=d, seq_len=max(max(caps), 64), window=1, pool_kernel=1, dtype=vb.VECTOR_BF16)
    ws = pl.alloc_workspace(vb.vector_workspace_bytes(shape, max(apxs), max(apxs), B))
    ws.fill_(0xff)                               # not a number, wherever something is read that was not written
    out = torch.full((B, Hq, d), 7.0, dtype=torch.float32, device="cuda:0")
    flags = vb.VECTOR_DECODE_OUT_F32 | (vb.VECTOR_DECODE_LITERAL if literal else 0)
    qd = pl.to_device(q)
    if rope:
        rp, k = vb.make_rope(inv, pl.to_device(np.concatenate([x.reshape(-1) for x in pos] + [np.zeros(1, np.int32)])))
        vb.vector_decode_attn_rope(cache, rp, qd, scale, out, ws, flags=flags)
    else:
        vb.vector_decode_attn(cache, qd, scale, out, ws, flags=flags)
    torch.cuda.synchronize()
    for b in range(B):
        kw = dict(pos_apx=pos[b][None], inv_freq=inv) if rope else {}
        if lens[b] + apxs[b] == 0:
            ref = np.zeros((1, Hq, d))
        else:
            ref = vo.decode_attn(dg.widen(q[b:b + 1]), dg.widen(k_ret[b][None]), dg.widen(v_ret[b][None]), np.array([lens[b]]),
                                 dg.widen(k_apx[b][None]), dg.widen(W), scale, **kw)
        got = out[b:b + 1].cpu().numpy()
        if rope and lens[b] + apxs[b] > 0 and apxs[b]:
            # a key that is turned back is rounded to bf16 (2^-9 of each element at most) before W is applied; the weights
            # of the rows sum to one, so the result moves by no more than the worst row does
            turned = np.abs(vo.rope_unrotate(dg.widen(k_apx[b]), pos[b], inv, False))
            worst = 2.0 ** -9 * np.einsum("htd,hdj->htj", turned, np.abs(dg.widen(W))).max(axis=1).repeat(G, axis=0)[None]
            got = np.where(np.abs(got - ref) <= worst, ref, got)
        close(got, ref, f"sequence {b}")


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("G", [1, 2, 3, 4, 5, 6, 7, 8, 10, 12, 16])
def test_query_heads(G, d):
    run(d, G, 2, [700, 129], [260, 260], ragged=False, seed=G)


@pytest.mark.parametrize("lens,apxs", [
    ([1], [0]), ([0], [1]), ([0, 0, 5], [0, 0, 0]), ([127, 128, 129, 0], [128] * 4), ([20000], [7000]), ([3, 9000], [33, 33]),
    ([40] * 70, [31] * 70), ([256 * i for i in range(12)], [1000] * 12), ([2000], [0]), ([0], [2000]),
])
@pytest.mark.parametrize("kind", ["plain", "rope", "literal"])
def test_lengths(lens, apxs, kind):
    run(128, 4, 2, lens, apxs, ragged=False, rope=kind == "rope", literal=kind == "literal", seed=len(lens))


@pytest.mark.parametrize("lens,apxs", [
    ([5, 9000, 1, 700], [0, 10, 3000, 129]), ([0, 0, 300], [0, 500, 0]), ([1600 - 60 * b for b in range(24)], [1600 - 61 * b for b in range(24)]),
    ([(37 * b) % 300 for b in range(130)], [(53 * b) % 200 for b in range(130)]),
])
@pytest.mark.parametrize("kind", ["plain", "rope", "literal"])
def test_unequal_blocks(lens, apxs, kind):
    run(128, 4, 3 if len(lens) < 100 else 1, lens, apxs, ragged=True, rope=kind == "rope", literal=kind == "literal", seed=len(lens))


@pytest.mark.parametrize("d,G", [(64, 8), (64, 1), (128, 16)])
def test_unequal_blocks_other_shapes(d, G):
    run(d, G, 1, [5, 4000, 0, 900], [77, 1, 2000, 0], ragged=True, seed=d + G)
