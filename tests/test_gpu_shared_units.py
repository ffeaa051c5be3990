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


def rows_apart(case):
    return "g%d-w%d-%s%s%s" % (case[0], case[1], "x".join(map(str, case[2])), "-rope" if case[3] else "", "-lse" if case[4] else "")


# 64 dims, whose query rows lie in the place of the sums until the first tile's barrier: query heads, window, tokens of the prompts,
# rotated keys, log-sum-exp given; one to several tiles of 128 tokens per workgroup, partial ones, prompts of equal and unequal length
@pytest.mark.parametrize("case", [(G, w, n, rope, lse) for G, w, n in [(1, 16, (70,)), (4, 32, (129,)), (2, 17, (700,)), (4, 32, (4225,)), (3, 40, (300, 300)), (1, 16, (1401, 640)),
                                                                       (4, 32, (5000, 129, 260))]
                                  for rope in (False, True) for lse in (False, True)] + [(4, 32, (40000,), False, True)], ids=rows_apart)
def test_rows_in_the_place_of_the_sums(case):
    G, w, lens, rope, lse = case
    d, H, B, T = 64, 2, len(lens), sum(lens)
    g = torch.Generator(device="cuda").manual_seed(T + G)
    rnd = lambda *sh: torch.randn(*sh, generator=g, device="cuda").bfloat16()
    q, k, v, W = rnd(B, H * G, w, d), rnd(H, T, d), rnd(H, T, d), (rnd(H, d, d).float() / 8).bfloat16()
    half = d // 2
    inv = 500000.0 ** (-torch.arange(half, dtype=torch.float64) / half)
    wide = lambda x: x.double().cpu()
    mass, eps, lse_rows = [], [], []
    for b, n in enumerate(lens):
        t0 = sum(lens[:b])
        kb, vbt = wide(k[:, t0:t0 + n]), wide(v[:, t0:t0 + n])
        logits = torch.matmul(wide(q[b]).view(H, G * w, d), kb.transpose(1, 2).contiguous()).view(H, G, w, n) / math.sqrt(d)
        logits = logits.masked_fill(torch.arange(n) > n - w + torch.arange(w)[:, None], float("-inf"))
        lse_rows.append(torch.logsumexp(logits, dim=-1).view(H * G, w))
        mass.append(torch.softmax(logits, dim=-1).mean(dim=(1, 2)))
        if rope:
            angle = torch.arange(n, dtype=torch.float64)[:, None] * inv
            c, s = torch.cos(angle), torch.sin(angle)
            kb = torch.cat((kb[..., :half] * c + kb[..., half:] * s, kb[..., half:] * c - kb[..., :half] * s), dim=-1)
        eps.append(((vbt - torch.matmul(kb, wide(W))) ** 2).sum(-1))
    shape = vb.Shape(n_q_heads=H * G, n_kv_heads=H, head_dim=d, seq_len=lens[0], window=w, pool_kernel=1, dtype=vb.VECTOR_BF16)
    rp, keep = vb.make_rope(inv.numpy()) if rope else (None, None)
    given = torch.stack(lse_rows).float().cuda() if lse else None
    options = vb.make_options(rp, given) if rope or lse else None
    pools, none = [n // 2 for n in lens], [0] * B
    batch, keep_batch = vb.make_batch(lens, pools, none, pools)
    R = sum(pools)
    out = [torch.full((H * T,), -7.0, device="cuda") for _ in range(2)]
    rest = [torch.empty(H * T, dtype=torch.uint8, device="cuda"), torch.empty(H * R, dtype=torch.int32, device="cuda"), torch.empty(1, dtype=torch.int32, device="cuda")]
    rest += [torch.empty(H * R, d, dtype=torch.bfloat16, device="cuda") for _ in range(2)] + [torch.empty(1, d, dtype=torch.bfloat16, device="cuda")]
    ws = pl.alloc_workspace(vb.vector_compress_batch_workspace_bytes(shape, batch))
    vb.vector_compress_batch_ex(shape, batch, options, q, k, v, W, *out, *rest, ws)
    torch.cuda.synchronize()
    for b, n in enumerate(lens):
        score, residual = (x[H * sum(lens[:b]):H * sum(lens[:b + 1])].view(H, n).double().cpu() for x in out)
        # logits of up to 6 in 32 bits, 64 roundings of 2^-24 of their largest term, and the given sums' own; residuals of 64 terms, keys turned back to 2^-16
        torch.testing.assert_close(score[:, :n - w], mass[b][:, :n - w], rtol=2e-5, atol=1e-12)
        torch.testing.assert_close(residual, eps[b], rtol=2e-4 if rope else 2e-5, atol=1e-4)
