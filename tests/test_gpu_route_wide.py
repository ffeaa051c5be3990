"""Routing with workgroups of sixteen waves: lengths around their blocks and parts that begin in one block and end in the
next, lists of 9 to 32 chunks (both chunk lengths), thresholds in the outermost bins; and the pooled scores, bit for bit,
for every way the windows are read."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2605_23258_amd import binding as vb
from paper_2605_23258_amd import pipeline as pl
import test_gpu_route_head as rh

pytestmark = pytest.mark.gpu


# heads that make the parts 1, 2, 3, 5 and 11 units of 256 tokens, so that some lie across a block's end
@pytest.mark.parametrize("n,heads", [(4095, 8), (4097, 8), (8191, 25), (8193, 23), (12289, 8), (12289, 40), (16383, 64), (16384, 43)])
@pytest.mark.parametrize("kind", ["distinct", "plateau"])
def test_one_launch(n, heads, kind):
    rh.test_route_at_block_edges(n, heads, kind)


@pytest.mark.parametrize("n,heads", [(18431, 3), (32769, 2), (34817, 1), (65536, 2), (65537, 1), (131072, 1)])
@pytest.mark.parametrize("kind", ["distinct", "outliers"])
def test_two_launches(n, heads, kind):
    rh.test_route_at_block_edges(n, heads, kind)


@pytest.mark.parametrize("mode", [vb.VECTOR_POOL_AVG, vb.VECTOR_POOL_MAX], ids=["avg", "max"])
@pytest.mark.parametrize("kernel", [1, 3, 9, 11, 17, 19])
@pytest.mark.parametrize("n", [61, 2049, 20011, 70001])
def test_pooled_scores(n, kernel, mode):
    heads, window, d = 2, 20, 64
    g = torch.Generator(device="cuda").manual_seed(n + kernel)
    q, k = (torch.randn(heads, m, d, generator=g, device="cuda") for m in (window, n))

    def score(kern):
        shape = vb.Shape(n_q_heads=heads, n_kv_heads=heads, head_dim=d, seq_len=n, window=window, pool_kernel=kern, dtype=vb.VECTOR_F32,
                         pool_mode=mode)
        out = torch.full((heads, n), -1.0, device="cuda")
        vb.vector_score(shape, q, k, out, pl.alloc_workspace(vb.vector_workspace_bytes(shape, 1, 0, 1)))
        torch.cuda.synchronize()
        return out.cpu().numpy()

    mass, got, prefix, half = score(1), score(kernel), n - window, kernel // 2
    padded = np.zeros((heads, prefix + 2 * half), dtype=np.float32)
    padded[:, half:half + prefix] = mass[:, :prefix]
    acc = np.zeros((heads, prefix), dtype=np.float32)
    for i in range(kernel):                      # ascending tokens, in fp32
        acc = np.maximum(acc, padded[:, i:i + prefix]) if mode == vb.VECTOR_POOL_MAX else acc + padded[:, i:i + prefix]
    assert np.array_equal(got[:, :prefix], acc if mode == vb.VECTOR_POOL_MAX else acc / np.float32(kernel))
    assert np.isposinf(got[:, prefix:]).all()
