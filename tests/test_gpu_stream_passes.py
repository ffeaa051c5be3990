"""The two streaming passes of the scorer at the edges of their tiles, rings and row units: heads of one to seven
tiles, one row more or less than a unit count holds, and the largest row block that goes through at once."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import vector_oracle as vo
from paper_2605_23258_amd import binding as vb
from paper_2605_23258_amd import datagen as dg
import workloads as wl
from paper_2605_23258_amd import pipeline as pl

pytestmark = pytest.mark.gpu

# dtype, d, query heads per KV head, window, tokens
CASES = [
    ("bf16", 128, 4, 32, 64), ("bf16", 128, 4, 32, 65), ("bf16", 128, 4, 32, 255), ("bf16", 128, 4, 32, 16449),
    ("bf16", 128, 1, 1, 129), ("bf16", 128, 3, 43, 449), ("bf16", 128, 8, 32, 321), ("bf16", 128, 9, 57, 450), ("bf16", 128, 8, 64, 20000),
    ("bf16", 64, 4, 32, 128), ("bf16", 64, 4, 33, 385), ("bf16", 64, 16, 32, 897),
    ("f32", 128, 4, 32, 33), ("f32", 128, 4, 33, 223), ("f32", 128, 8, 32, 1500),
    ("f32", 64, 4, 32, 65), ("f32", 64, 8, 32, 447), ("f32", 64, 8, 64, 700),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "%s-d%d-g%d-w%d-n%d" % c)
def test_scores_and_residuals_against_the_oracle(case):
    dtype, d, group, window, n = case
    base = dg.CONFIGS["cfg2" if dtype == "bf16" else "cfg1"]
    cfg = dg.scaled(base, head_dim=d, n_kv_heads=2, n_q_heads=2 * group, seq_len=n, window=window, pool_kernel=3, cal_tokens=512, heavy_frac=0.05)
    li = wl.make_layer(cfg, 3)
    shape = pl.shape_of(cfg)
    dev = {k: pl.to_device(getattr(li, k)) for k in ("q_win", "k", "v", "w_cal")}
    ws = pl.alloc_workspace(vb.vector_workspace_bytes(shape, 1, 0, 1))
    score, eps = (torch.full((2, n), -7.0, device="cuda") for _ in range(2))
    vb.vector_score_residual(shape, dev["q_win"], dev["k"], dev["v"], dev["w_cal"], score, eps, ws)
    alone = torch.full((2, n), -7.0, device="cuda")
    vb.vector_score(shape, dev["q_win"], dev["k"], alone, ws)
    torch.cuda.synchronize()
    assert torch.equal(score, alone)
    wide = {k: dg.widen(getattr(li, k)) for k in ("q_win", "k", "v", "w_cal")}
    got, ref = score.cpu().numpy().astype(np.float64), vo.score(wide["q_win"], wide["k"], window, 3).astype(np.float64)
    assert np.isposinf(got[:, n - window:]).all()
    np.testing.assert_allclose(got[:, : n - window] * n, ref[:, : n - window] * n, rtol=2e-3, atol=1e-3)
    np.testing.assert_allclose(eps.cpu().numpy(), vo.residual(wide["k"], wide["v"], wide["w_cal"]), rtol=2e-3, atol=1e-3)
