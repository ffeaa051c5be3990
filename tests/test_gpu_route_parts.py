"""Single-launch routing: how a batch's tokens are shared out over workgroups (parts that begin and end inside a block of
tokens, parts of several blocks, prompts shorter than one part), and every kernel width that it pools itself."""
import pytest

torch = pytest.importorskip("torch")

import test_gpu_batch as tb

pytestmark = pytest.mark.gpu

POOLS = {"pool_%s_%d" % (mode, kernel): ("cfg2", dict(n_kv_heads=2, n_q_heads=4, window=16, pool_kernel=kernel, pool_mode=mode), (700, 4101), (0, 1))
         for mode in ("avg", "max") for kernel in (1, 3, 5, 7, 9, 11, 13, 15, 17)}
# beyond: pooled by a launch of their own, routed by two
WIDER = {
    "pool_19_short": ("cfg2", dict(n_kv_heads=2, n_q_heads=8, window=32, pool_kernel=19), (700, 2048, 6100, 32), (5, 0, 1, 0)),
    "pool_19_more_prompts_than_arguments_hold": ("cfg1", dict(n_kv_heads=1, n_q_heads=2, window=20, pool_kernel=19), tuple(70 + 131 * i for i in range(20)),
                                                 tuple(i % 3 for i in range(20))),
}
PARTS = {
    # 24 heads: parts of 4 units of 256 tokens, four blocks of 4096 tokens a head
    "parts_across_blocks": ("cfg2", dict(n_kv_heads=8, n_q_heads=8, window=16, head_dim=64), (12289, 16384, 300), (0, 1, 0)),
    # one part per head, of two blocks of 2048 tokens
    "parts_whole_heads": ("cfg2", dict(n_kv_heads=64, n_q_heads=64, window=16, head_dim=64), (4000, 2049, 700, 64, 3000), (0, 0, 2, 0, 1)),
}
tb.BATCHES.update(POOLS)
tb.BATCHES.update(PARTS)
tb.BATCHES.update(WIDER)


@pytest.mark.parametrize("name", list(PARTS) + list(POOLS) + ["pool_19_short"])
def test_equals_one_call_per_prompt(name):
    tb.test_compress_batch_equals_one_call_per_sequence(name)


@pytest.mark.parametrize("name", list(POOLS) + list(WIDER))
def test_pooling_against_the_oracle(name):
    tb.test_compress_batch_against_the_oracle_sequence_by_sequence(name)
