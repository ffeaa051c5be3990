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
from parity_util import ATOL, RTOL, close

pytestmark = pytest.mark.gpu

THETA = 10000.0


def reference(q, k_ret, v_ret, k_apx, W, scale, pos=None, inv=None):
    """q [Hq, d], rows [H, n, d], all bf16: one attention over exact and rebuilt rows.  With positions, a key that is turned
    back is a bf16 operand of the product with W, like the keys of a cache without rotary embedding."""
    lin = dg.widen(k_apx) if pos is None else dg.widen(dg.f32_to_bf16_bits(vo.rope_unrotate(dg.widen(k_apx), pos, inv, False).astype(np.float32)))
    keys = np.concatenate([dg.widen(k_ret), dg.widen(k_apx)], axis=1)
    vals = np.concatenate([dg.widen(v_ret), np.matmul(lin.astype(np.float64), np.asarray(W, np.float64))], axis=1)
    none = np.zeros((1, keys.shape[0], 0, keys.shape[2]))
    if keys.shape[1] == 0:
        return np.zeros(q.shape)
    return vo.decode_attn(dg.widen(q)[None], keys[None], vals[None], np.array([keys.shape[1]]), none, np.zeros_like(W), scale)[0]


def told_apart(ref, wrong):
    return (np.abs(wrong - ref) > ATOL + RTOL * np.abs(ref)).any()


def check(got, q, k_ret, v_ret, k_apx, W, scale, what, pos=None, inv=None):
    """The bar of `close`; and with positions, unless they are hardly any of the rows, that it would not let a step pass that
    lost the approximated values or was one position off."""
    W = dg.widen(W)
    ref = reference(q, k_ret, v_ret, k_apx, W, scale, pos, inv)
    close(got, ref, what)
    if pos is not None and 50 * k_apx.shape[1] >= max(k_ret.shape[1], 1):
        assert told_apart(ref, reference(q, k_ret, v_ret, k_apx, np.zeros_like(W), scale, pos, inv)), f"{what}: blind to W"
        assert told_apart(ref, reference(q, k_ret, v_ret, k_apx, W, scale, pos + 1, inv)), f"{what}: blind to the positions"


def run(d, G, H, lens, apxs, ragged, rope=False, literal=False, seed=0, steer=0):
    """One attention over sequences of lens[b] retained and apxs[b] approximated rows; `ragged`: blocks of their own, with at least
    `steer` as the largest capacity, which there only steers how the work is split."""
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
    cache = vb.Cache(batch=B, n_q_heads=Hq, n_kv_heads=H, head_dim=d, dtype=vb.VECTOR_BF16, cap_retain=max(max(caps), steer), n_approx=max(apxs))
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
        check(out[b].cpu().numpy(), q[b], k_ret[b][:, :lens[b]], v_ret[b][:, :lens[b]], k_apx[b], W, scale, f"sequence {b}",
              *((pos[b], inv) if rope else ()))


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


def run_paged(d, G, H, lens, n_apx, block_rows, blocks_per_seq, rope, seed):
    """A step with its token over paged retained blocks; lens[b] up to the capacity, at which the token has no row to go to.
    Only live blocks have a place of their own in the pool."""
    rng = np.random.default_rng(seed)
    store = lambda a: dg.f32_to_bf16_bits(a.astype(np.float32))
    B, Hq, cap = len(lens), H * G, block_rows * blocks_per_seq
    live = [min(blocks_per_seq, n // block_rows + 1) for n in lens]         # with the token's
    ids = iter(rng.permutation(H * sum(live)) + 1)                           # block 0: of nobody, never read
    table = np.zeros((B, H, blocks_per_seq), np.int32)
    k_pool = store(np.full((H * sum(live) + 1, block_rows, d), 1e30))
    v_pool = store(np.full(k_pool.shape, -1e30))
    k_lin, v_lin = ([store(rng.standard_normal((H, n, d))) for n in lens] for _ in range(2))
    for b, n in enumerate(lens):
        for h in range(H):
            for j in range(live[b]):
                table[b, h, j] = next(ids)
                rows = slice(j * block_rows, min(n, (j + 1) * block_rows))
                for pool, lin in ((k_pool, k_lin), (v_pool, v_lin)):
                    pool[table[b, h, j], :max(0, rows.stop - rows.start)] = lin[b][h, rows]
    k_apx, pos = store(rng.standard_normal((B, H, n_apx, d))), rng.integers(0, 100000, (B, H, n_apx)).astype(np.int32)
    q, W = store(rng.standard_normal((B, Hq, d))), store(rng.standard_normal((H, d, d)) / np.sqrt(d))
    k_new, v_new = store(rng.standard_normal((B, H, d))), store(rng.standard_normal((B, H, d)))
    scale, inv = 1.0 / np.sqrt(d), dg.rotary_inv_freq(d, THETA)
    t = dict(len=pl.to_device(np.array(lens, np.int32)), k=pl.to_device(k_pool), v=pl.to_device(v_pool), k_apx=pl.to_device(k_apx),
             W=pl.to_device(W), table=pl.to_device(table))
    cache = vb.Cache(batch=B, n_q_heads=Hq, n_kv_heads=H, head_dim=d, dtype=vb.VECTOR_BF16, cap_retain=cap, n_approx=n_apx)
    cache.len_retain, cache.k_ret, cache.v_ret, cache.k_apx, cache.W = (t[x].data_ptr() for x in ("len", "k", "v", "k_apx", "W"))
    cache.ret_block_table, cache.ret_block_rows, cache.ret_blocks_per_seq = t["table"].data_ptr(), block_rows, blocks_per_seq
    shape = vb.Shape(n_q_heads=Hq, n_kv_heads=H, head_dim=d, seq_len=max(cap, 64), window=1, pool_kernel=1, dtype=vb.VECTOR_BF16)
    ws = pl.alloc_workspace(vb.vector_workspace_bytes(shape, n_apx, n_apx, B))
    ws.fill_(0xff)
    out = torch.full((B, Hq, d), 7.0, dtype=torch.float32, device="cuda:0")
    args = [pl.to_device(x) for x in (q, k_new, v_new)] + [scale, out, ws]
    if rope:
        rp, keep = vb.make_rope(inv, pl.to_device(pos))
        vb.vector_decode_step_rope(cache, rp, *args, flags=vb.VECTOR_DECODE_OUT_F32)
    else:
        vb.vector_decode_step(cache, *args, flags=vb.VECTOR_DECODE_OUT_F32)
    torch.cuda.synchronize()
    for b, n in enumerate(lens):
        with_token = [np.concatenate([x[b], new[b][:, None]], axis=1) for x, new in ((k_lin, k_new), (v_lin, v_new))]
        if n in (0, 1, cap) or b % 16 == 0 or len(lens) < 16:
            check(out[b].cpu().numpy(), q[b], *with_token, k_apx[b], W, scale, f"sequence {b}", *((pos[b], inv) if rope else ()))
        for h in range(H):
            if n < cap:
                k_pool[table[b, h, n // block_rows], n % block_rows] = k_new[b, h]
                v_pool[table[b, h, n // block_rows], n % block_rows] = v_new[b, h]
    assert np.array_equal(pl.to_host(t["k"]), k_pool) and np.array_equal(pl.to_host(t["v"]), v_pool)       # the token's rows, and no others
    assert np.array_equal(t["len"].cpu().numpy(), np.minimum(np.array(lens) + 1, cap))


@pytest.mark.parametrize("rope", [False, True])
@pytest.mark.parametrize("block_rows", [16, 32, 64])
@pytest.mark.parametrize("d,G", [(64, 4), (128, 8)])
def test_paged_step(d, G, block_rows, rope):
    n = 6 * block_rows
    run_paged(d, G, 2, [n, 0, 1, n - 1, n - block_rows, 2 * block_rows + 5, 31], 300, block_rows, 6, rope, seed=d + block_rows)


@pytest.mark.parametrize("rope", [False, True])
@pytest.mark.parametrize("d", [64, 128])
def test_paged_step_over_more_blocks_than_lanes(d, rope):
    """768 (sequence, head) pairs leave two workgroups to a retained segment: 100 blocks of 32 rows, more than one register holds."""
    run_paged(d, 4, 4, [6400, 6399, 6000] + [(7 * b) % 50 for b in range(189)], 40, 32, 200, rope, seed=d)
