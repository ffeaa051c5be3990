"""Routing of a whole head in one launch: lengths around the blocks, the waves' runs and the line to the
launches for longer heads, with distinct scores, many ties, plateaus and single values, against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import vector_oracle as vo
from paper_2605_23258_amd import binding as vb
from paper_2605_23258_amd import pipeline as pl

pytestmark = pytest.mark.gpu

KINDS = {
    "distinct": lambda rng, sh: rng.standard_normal(sh),
    "three_values": lambda rng, sh: rng.integers(0, 3, sh),
    "plateau": lambda rng, sh: np.where(rng.random(sh) < 0.6, 0.0, np.exp(4 * rng.standard_normal(sh))),
    "one_value": lambda rng, sh: np.full(sh, 0.25),
    "outliers": lambda rng, sh: np.where(rng.random(sh) < 0.01, np.inf, 1.0 + 1e-6 * rng.random(sh)),
}


@pytest.mark.parametrize("n,heads", [(1, 1), (2, 3), (5, 1), (255, 2), (256, 1), (257, 3), (2047, 2), (2048, 1), (2049, 2), (4100, 40),
                                     (16384, 2), (16385, 3), (24575, 1), (24576, 2), (24577, 1)])
@pytest.mark.parametrize("kind", list(KINDS))
def test_route_at_block_edges(n, heads, kind):
    rng = np.random.default_rng(n * 31 + heads)
    score = KINDS[kind](rng, (heads, n)).astype(np.float32)
    eps = np.abs(KINDS["distinct" if kind == "three_values" else kind](rng, (heads, n))).astype(np.float32)
    shape = vb.Shape(n_q_heads=heads, n_kv_heads=heads, head_dim=64, seq_len=n, window=1, pool_kernel=1, dtype=vb.VECTOR_F32)
    for n_p, n_a in {(n, n), (n, 0), (1, 1), (max(n // 3, 1), n // 7), (max(n - 1, 1), n // 2), (max(n // 2, 1), max(n // 2, 1) - (n > 3))}:
        ws = pl.alloc_workspace(vb.vector_workspace_bytes(shape, n_p, n_a, 1))
        tier = torch.full((heads, n), 9, dtype=torch.uint8, device="cuda:0")
        i_r = torch.full((heads, max(n_p - n_a, 1)), -1, dtype=torch.int32, device="cuda:0")
        i_a = torch.full((heads, max(n_a, 1)), -1, dtype=torch.int32, device="cuda:0")
        vb.vector_route(heads, n, pl.to_device(score), pl.to_device(eps), n_p, n_a, tier, i_r if n_p > n_a else None, i_a if n_a else None, ws)
        torch.cuda.synchronize()
        o_tier, o_r, o_a = vo.route(score, eps, n_p, n_a)
        assert np.array_equal(tier.cpu().numpy(), o_tier)
        if n_p > n_a:
            assert np.array_equal(i_r.cpu().numpy(), o_r)
        if n_a:
            assert np.array_equal(i_a.cpu().numpy(), o_a)
