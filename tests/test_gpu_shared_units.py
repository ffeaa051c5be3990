"""Query rows that two waves of a workgroup share: each fetches half of a unit's rows and adds up half of its chunks' sums.
One head, so that tokens make as many chunks as there are tiles: 1 to 5, around 32 (what is read at once) and all 256; rows that
fill one unit, end inside one, or are 128."""
import math

import pytest

torch = pytest.importorskip("torch")

from paper_2605_23258_amd import binding as vb
from paper_2605_23258_amd import pipeline as pl

pytestmark = pytest.mark.gpu

# dtype, d, query heads, window, tokens
CASES = [("bf16", 128, 4, 32, n) for n in (64, 65, 129, 200, 300, 2047, 2113, 16384, 16500)]
CASES += [("bf16", 128, 1, 1, 130), ("bf16", 128, 3, 11, 2113), ("bf16", 64, 4, 32, 129), ("bf16", 64, 4, 32, 4225), ("bf16", 64, 2, 17, 700)]
CASES += [("f32", 128, 4, 32, n) for n in (33, 97, 1057)] + [("f32", 64, 4, 32, n) for n in (129, 2113)]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "%s-d%d-g%d-w%d-n%d" % c)
def test_mass_against_64_bits(case):
    dtype, d, G, w, n = case
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device="cuda").manual_seed(n)
    q, k = torch.randn(G, w, d, generator=g, device="cuda").to(dt), torch.randn(1, n, d, generator=g, device="cuda").to(dt)
    shape = vb.Shape(n_q_heads=G, n_kv_heads=1, head_dim=d, seq_len=n, window=w, pool_kernel=1, dtype=vb.VECTOR_BF16 if dtype == "bf16" else vb.VECTOR_F32)
    score = torch.full((1, n), -7.0, device="cuda")
    vb.vector_score(shape, q, k, score, pl.alloc_workspace(vb.vector_workspace_bytes(shape, 1, 0, 1)))
    logits = (q.double().cpu().view(G * w, d) @ k[0].double().cpu().t()) / math.sqrt(d)
    seen = torch.arange(n)[None, :] <= (n - w + torch.arange(w))[:, None]
    p = torch.softmax(logits.view(G, w, n).masked_fill(~seen, float("-inf")), dim=-1).mean(dim=(0, 1))
    # logits of up to 6 in 32 bits: 128 roundings of 2^-24 of their largest term, and as much again from the exponentials
    torch.testing.assert_close(score[0, : n - w].double().cpu(), p[: n - w], rtol=2e-5, atol=1e-12)
