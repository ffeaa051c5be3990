"""More query rows per KV head than the passes hold at once (512; fp32 at d = 128: 256): the query heads go through the
pair of passes a group at a time, each group adding its share to the column mass and only the first carrying the
residual.  Through the compression call with and without the window's log-sum-exp, on plain and on rotated keys, for
one prompt, for equal ones (stacked heads) and for unequal ones (taken one by one), and the limits of one head's window."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import vector_oracle as vo
from paper_2605_23258_amd import binding as vb
from paper_2605_23258_amd import datagen as dg
from paper_2605_23258_amd import pipeline as pl
import workloads as wl
from parity_util import close
from test_gpu_lse import window_lse

pytestmark = pytest.mark.gpu

THETA = 500000.0
CASES = {
    # dtype, d, KV heads, query heads per KV head, window, tokens: groups
    "bf16_9x64": ("bf16", 128, 2, 9, 64, 1500),            # 8 + 1 heads
    "bf16_20x60_long": ("bf16", 128, 1, 20, 60, 17003),    # 8 + 8 + 4; beyond the length of one routing launch
    "bf16_d64_17x32": ("bf16", 64, 2, 17, 32, 900),        # 16 + 1
    "f32_d128_5x60": ("f32", 128, 1, 5, 60, 700),          # 4 + 1
    "f32_d64_11x48": ("f32", 64, 2, 11, 48, 700),          # 10 + 1
}


def _layer(name, layer=0, **kw):
    dtype, d, H, G, w, n = CASES[name]
    cfg = dg.scaled(dg.CONFIGS["cfg2" if dtype == "bf16" else "cfg1"], head_dim=d, n_kv_heads=H, n_q_heads=H * G, seq_len=n, window=w,
                    cal_tokens=512)
    return cfg, wl.make_layer(cfg, layer, **kw)


@pytest.mark.parametrize("rotated", [False, True], ids=["plain", "rotated"])
@pytest.mark.parametrize("with_lse", [False, True], ids=["two_passes", "lse"])
@pytest.mark.parametrize("name", list(CASES))
def test_compress_in_groups(name, with_lse, rotated):
    cfg, li = _layer(name, **(dict(rope_theta=THETA, rope_interleaved=False, pos_offset=9) if rotated else {}))
    shape, n, w = pl.shape_of(cfg), cfg.seq_len, cfg.window
    n_r, n_a, n_p = cfg.counts()
    keep = []
    rope = None
    if rotated:
        rope, k = vb.make_rope(li.extra["inv_freq"], None, False, 9)
        keep.append(k)
    lse = pl.to_device(window_lse(li.q_win, li.k)) if with_lse else None
    out = pl.alloc_outputs(shape, n_p, n_a, n_r, torch.bfloat16 if cfg.dtype == "bf16" else torch.float32)
    ws = pl.alloc_workspace(vb.vector_compress_workspace_bytes(shape, n_p, n_a))
    dev = {x: pl.to_device(getattr(li, x)) for x in ("q_win", "k", "v", "w_cal")}
    vb.vector_compress_ex(shape, vb.make_options(rope, lse) if rotated or with_lse else None, dev["q_win"], dev["k"], dev["v"], dev["w_cal"], n_p, n_a,
                          out.score, out.eps, out.tier, out.idx_retain, out.idx_approx, out.k_ret, out.v_ret, out.k_apx, n_r, ws)
    torch.cuda.synchronize()
    score, eps = out.score.cpu().numpy(), out.eps.cpu().numpy()
    ref = vo.score(dg.widen(li.q_win), dg.widen(li.k), w, cfg.pool_kernel, cfg.pool_mode)
    turned = dict(pos=li.extra["pos"], inv_freq=li.extra["inv_freq"], interleaved=False) if rotated else {}
    assert np.isposinf(score[:, n - w:]).all()
    close(score[:, : n - w].astype(np.float64) * n, ref[:, : n - w].astype(np.float64) * n, "n*score")
    close(eps, vo.residual(dg.widen(li.k), dg.widen(li.v), dg.widen(li.w_cal), **turned), "eps")
    tier, idx_r, idx_a = vo.route(score, eps, n_p, n_a)
    assert np.array_equal(out.tier.cpu().numpy(), tier)
    assert np.array_equal(out.idx_retain.cpu().numpy(), idx_r) and np.array_equal(out.idx_approx.cpu().numpy(), idx_a)
    rk, rv, ra = vo.compact(li.k, li.v, idx_r, idx_a)
    assert np.array_equal(pl.to_host(out.k_ret), rk) and np.array_equal(pl.to_host(out.v_ret), rv) and np.array_equal(pl.to_host(out.k_apx), ra)


@pytest.mark.parametrize("lens", [(900, 900, 900), (700, 1100, 450)], ids=["equal", "unequal"])
@pytest.mark.parametrize("name", ["bf16_9x64", "f32_d128_5x60"])
def test_batches_in_groups_equal_one_call_per_prompt(name, lens):
    dtype, d, H, G, w, _ = CASES[name]
    cfg, _ = _layer(name)
    layers = [wl.make_layer(dg.scaled(cfg, seq_len=n), b) for b, n in enumerate(lens)]
    counts = [vo.budget_counts_frac(n, cfg.f_retain, cfg.f_approx) for n in lens]
    n_pool, n_approx = [c[0] for c in counts], [c[1] for c in counts]
    n_ret = [p - a for p, a in counts]
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    W = pl.to_device(layers[0].w_cal)
    shape = pl.shape_of(cfg, seq_len=1)
    batch, keep = vb.make_batch(lens, n_pool, n_approx, n_ret)
    ws = pl.alloc_workspace(vb.vector_compress_batch_workspace_bytes(shape, batch))
    f = lambda m, t, v: torch.full((H * m,), v, dtype=t, device="cuda:0")
    T, R, A = sum(lens), sum(n_ret), sum(n_approx)
    got = dict(score=f(T, torch.float32, -1.0), eps=f(T, torch.float32, -1.0), tier=f(T, torch.uint8, 9), ir=f(R, torch.int32, -1),
               ia=f(A, torch.int32, -1))
    rows = [torch.zeros((H * m, d), dtype=tdt, device="cuda:0") for m in (R, R, A)]
    vb.vector_compress_batch(shape, batch, pl.to_device(np.stack([li.q_win for li in layers])), pl.to_device(np.concatenate([li.k for li in layers], axis=1)),
                             pl.to_device(np.concatenate([li.v for li in layers], axis=1)), W, got["score"], got["eps"], got["tier"], got["ir"], got["ia"],
                             *rows, ws)
    t0 = 0
    for b, li in enumerate(layers):
        n = lens[b]
        s1 = pl.shape_of(cfg, seq_len=n)
        one = pl.alloc_outputs(s1, n_pool[b], n_approx[b], n_ret[b], tdt)
        ws1 = pl.alloc_workspace(vb.vector_compress_workspace_bytes(s1, n_pool[b], n_approx[b]))
        pl.compress_layer(s1, pl.to_device(li.q_win), pl.to_device(li.k), pl.to_device(li.v), W, n_pool[b], n_approx[b], one, ws1, one_call=True)
        torch.cuda.synchronize()
        for x in ("score", "eps", "tier"):
            assert torch.equal(got[x][H * t0: H * (t0 + n)].view(H, n), getattr(one, x)), (x, b)
        ref = vo.score(dg.widen(li.q_win), dg.widen(li.k), w, cfg.pool_kernel, cfg.pool_mode)
        close(one.score.cpu().numpy()[:, : n - w].astype(np.float64) * n, ref[:, : n - w].astype(np.float64) * n, f"n*score of prompt {b}")
        t0 += n
    del keep


@pytest.mark.parametrize("dtype,d,most", [("bf16", 128, 288), ("bf16", 64, 384), ("f32", 128, 256), ("f32", 64, 288)])
def test_window_of_one_head(dtype, d, most):
    """The longest window of a query head, a shorter one that fills no whole unit of 32 rows, and one too long."""
    for window in (most, most - 95, most + 1):
        cfg = dg.scaled(dg.CONFIGS["cfg2" if dtype == "bf16" else "cfg1"], head_dim=d, n_kv_heads=1, n_q_heads=2, seq_len=900, window=window,
                        cal_tokens=512)
        li = wl.make_layer(cfg, 1)
        shape = pl.shape_of(cfg)
        dev = {x: pl.to_device(getattr(li, x)) for x in ("q_win", "k", "v", "w_cal")}
        score, eps = (torch.full((1, 900), -1.0, device="cuda:0") for _ in range(2))
        ws = pl.alloc_workspace(vb.vector_workspace_bytes(shape, 300, 100, 1))
        call = lambda: vb.vector_score_residual(shape, dev["q_win"], dev["k"], dev["v"], dev["w_cal"], score, eps, ws)
        if window > most:
            with pytest.raises(vb.VectorError) as ei:
                call()
            assert ei.value.code == vb.VECTOR_ERR_SHAPE
            torch.cuda.synchronize()
            assert (score == -1.0).all() and (eps == -1.0).all()
            continue
        call()
        torch.cuda.synchronize()
        ref = vo.score(dg.widen(li.q_win), dg.widen(li.k), window, cfg.pool_kernel)
        m = 900 - window
        close(score.cpu().numpy()[:, :m].astype(np.float64) * 900, ref[:, :m].astype(np.float64) * 900, f"n*score (window {window})")
        close(eps.cpu().numpy(), vo.residual(dg.widen(li.k), dg.widen(li.v), dg.widen(li.w_cal)), f"eps (window {window})")
