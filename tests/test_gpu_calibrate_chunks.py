"""The value map's chunks of tokens: whole and cut tiles, the tiles' sums added to a total, one chunk per head and several, the
longest ones, heads that do not divide the CUs."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import vector_oracle as vo
from paper_2605_23258_amd import binding as vb
from paper_2605_23258_amd import datagen as dg
from paper_2605_23258_amd import pipeline as pl

pytestmark = pytest.mark.gpu

# (head dim, heads, tokens, chunks per head): tiles of 128 tokens for d = 128, 256 for d = 64
SIZES = [
    (128, 1, 128, 1), (128, 1, 129, 1), (128, 1, 257, 2),           # chunks of 256 tokens, the last one with a single token
    (128, 256, 511, 1), (128, 256, 512, 1), (128, 256, 513, 1),     # four tiles less a token, four, a fifth of one token
    (128, 256, 2048, 1), (128, 256, 2049, 2),                       # the longest chunk, and two where one would be longer
    (128, 300, 1290, 2),                                            # more heads than CUs: six tiles, and five with a cut one
    (128, 130, 2088, 3),                                            # two rounds: six tiles twice, and five with a cut one
    (64, 1, 64, 1), (64, 1, 255, 1), (64, 1, 257, 2),               # the tile's second half empty, cut, and a second tile of one token
    (64, 256, 1023, 1), (64, 256, 1025, 1), (64, 256, 2049, 2),     # one chunk per head around four tiles; two chunks
    (64, 33, 5000, 7),                                              # seven chunks of three tiles, the last one shorter
]


@pytest.mark.parametrize("d,heads,m,chunks", SIZES)
def test_chunks_of_tokens(d, heads, m, chunks):
    rng = np.random.default_rng(d + heads + m)
    k = rng.standard_normal((heads, m, d), dtype=np.float32)
    w = rng.standard_normal((heads, d, d), dtype=np.float32) / np.float32(np.sqrt(d))
    v = np.matmul(k, w) + 0.1 * rng.standard_normal((heads, m, d), dtype=np.float32)
    kb, vbf = torch.from_numpy(k).bfloat16(), torch.from_numpy(v).bfloat16()
    shape = pl.shape_of(dg.scaled(dg.CONFIGS["cfg2"], seq_len=m, head_dim=d, n_kv_heads=heads, n_q_heads=heads))
    # the workspace: two d x d products per chunk in fp32, and the sums' 16 x 16 tiles in fp64
    nb = d // 16
    tiles = nb * (nb + 1) // 2 + nb * nb
    assert vb.vector_calibrate_workspace_bytes(shape) == heads * (chunks * 2 * d * d * 4 + tiles * 256 * 8)
    W = torch.full((heads, d, d), float("nan"), dtype=torch.bfloat16, device="cuda:0")
    ws = pl.alloc_workspace(vb.vector_calibrate_workspace_bytes(shape))
    vb.vector_calibrate(shape, kb.cuda(), vbf.cuda(), W, ws)
    torch.cuda.synchronize()
    got = W.double().cpu().numpy()
    # The fp32 sums: eight additions to an accumulator, each off by 2^-23 of it at most, and at most 16 accumulators in a total, by
    # 2^-24: below `sums` of the sum of the products' magnitudes.  W is stored in bf16: eight bits, half a unit is up to 2^-8 of an element.
    sums = 2.0 ** -24 * (2 * 8 + 16)
    for h in sorted({0, heads // 2, heads - 1}):
        kd, vd = kb[h].double().numpy(), vbf[h].double().numpy()
        gram, cross = kd.T @ kd, kd.T @ vd
        # the normal equations themselves, whatever their conditioning
        slack = 2.0 ** -8 * np.abs(gram) @ np.abs(got[h]) + sums * (np.abs(kd.T) @ (np.abs(kd) @ np.abs(got[h]) + np.abs(vd)))
        off = np.abs(gram @ got[h] - cross)
        assert (off <= slack).all(), f"head {h}: {off.flat[(off - slack).argmax()]:.3e} of {slack.flat[(off - slack).argmax()]:.3e}"
        if m >= 4 * d:
            # and the map: the sums' errors times the condition number (at most 9 for these keys) and the norm of W (at most 3)
            ref = vo.ols_fit(kd[None], vd[None])[0]
            bound = 2.0 ** -8 * np.abs(ref) + sums * 2 * np.linalg.cond(gram) * 3 + 1e-6
            err = np.abs(got[h] - ref)
            assert (err <= bound).all(), f"head {h}: max err {err.max():.3e}, bound {bound.flat[err.argmax()]:.3e}"


# (head dim, heads, tokens, chunk): fp32 sums of many tokens.  With 256 heads a chunk is as long as one may be, with 8 heads of
# 12000 tokens as short as a workgroup per CU makes it.
LONG_SUMS = [(128, 256, 32768, 1024), (64, 256, 32768, 1024), (128, 8, 12000, 256), (64, 8, 12000, 256), (64, 96, 32768, 1024)]


@pytest.mark.parametrize("d,heads,m,chunk", LONG_SUMS)
def test_sums_are_as_good_as_those_of_short_chunks(d, heads, m, chunk):
    """Keys that are nearly one direction: the map magnifies what the fp32 sums lose (by 1 / spread^2, 6e4), far beyond its own
    rounding to bf16.  It may be off by as much as sums over chunks of `chunk` tokens would make it, 16 tokens at a time
    into one accumulator that rounds to nearest, the chunks added in 64 bits."""
    g = torch.Generator(device="cuda").manual_seed(d + heads)
    spread = 2.0 ** -8
    k, v = (torch.empty((heads, m, d), dtype=torch.bfloat16, device="cuda") for _ in range(2))
    for h in range(heads):
        size = 0.5 + 0.5 * torch.rand(m, 1, generator=g, device="cuda")
        k[h] = (size * (1 + spread * torch.randn(m, d, generator=g, device="cuda"))).bfloat16()
        v[h] = (k[h].float() @ (torch.randn(d, d, generator=g, device="cuda") / d ** 0.5)).bfloat16()
    shape = pl.shape_of(dg.scaled(dg.CONFIGS["cfg2"], seq_len=m, head_dim=d, n_kv_heads=heads, n_q_heads=heads))
    W = torch.full((heads, d, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    vb.vector_calibrate(shape, k, v, W, pl.alloc_workspace(vb.vector_calibrate_workspace_bytes(shape)))
    torch.cuda.synchronize()
    # root mean square of the relative error of a sum of equal terms: the k-th of a chunk's K additions rounds at k / K of the chunk,
    # by 2^-24 / sqrt(3); the chunks' errors are independent
    K, M = chunk / 16, m / 16
    rel = 2.0 ** -24 / 3 ** 0.5 * K / (3 * M) ** 0.5
    rng = np.random.default_rng(m)
    got, off, magnified = W.double().cpu().numpy(), 0.0, 0.0
    some = sorted({0, heads // 2, heads - 1})
    for h in some:
        kd, vd = k[h].double().cpu().numpy(), v[h].double().cpu().numpy()
        gram, cross = kd.T @ kd, kd.T @ vd
        ref = np.linalg.solve(gram, cross)
        off += ((got[h] - ref) ** 2).mean() / len(some)
        # what errors of that size do to the map
        e = np.tril(rng.standard_normal((d, d)))
        e = (e + np.tril(e, -1).T) * rel * gram
        c = rng.standard_normal((d, d)) * rel * np.abs(cross)
        magnified += (np.linalg.solve(gram, c - e @ ref) ** 2).mean() / len(some)
    stored = (2.0 ** -8) ** 2 * (got[some] ** 2).mean()          # half a unit of bf16 per element, at most
    assert off <= magnified + stored, f"rms {off ** 0.5:.2e}, of the sums {magnified ** 0.5:.2e}, of bf16 {stored ** 0.5:.2e}"
