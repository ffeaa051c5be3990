"""Batches of unequal prompts whose routing takes two launches: prompts beyond the length of one, or a pooling kernel beyond the
widest that one launch forms.  Their parameter blocks are kernel arguments, or a table when there are many."""
import pytest

torch = pytest.importorskip("torch")

import test_gpu_batch as tb

pytestmark = pytest.mark.gpu

TWO_LAUNCHES = {
    "long_bf16_three": ("cfg2", dict(n_kv_heads=2, n_q_heads=8, window=32), (17000, 4100, 20011), (3, 0, 1)),
    # pools for 16, 32 and 64 register slots per thread, and one that exceeds them
    "long_bf16_wide_pool": ("cfg2", dict(n_kv_heads=1, n_q_heads=2, window=16), (40000, 17001, 70000), (0, 2, 0), ((12000, 6000), (17001, 100), (60000, 59000))),
    "long_f32_max_pool_kernel_11": ("cfg1", dict(n_kv_heads=2, n_q_heads=4, window=20, pool_kernel=11, pool_mode="max"), (1500, 18000), (0, 5)),
    "pool_19_short": ("cfg2", dict(n_kv_heads=2, n_q_heads=8, window=32, pool_kernel=19), (700, 2048, 6100, 32), (5, 0, 1, 0)),
    "pool_19_more_prompts_than_arguments_hold": ("cfg1", dict(n_kv_heads=1, n_q_heads=2, window=20, pool_kernel=19), tuple(70 + 131 * i for i in range(20)),
                                                 tuple(i % 3 for i in range(20))),
}


@pytest.mark.parametrize("name", list(TWO_LAUNCHES))
def test_against_the_oracle(name):
    tb.against_the_oracle(tb.RaggedBatch(TWO_LAUNCHES[name]), name)


@pytest.mark.parametrize("name", list(TWO_LAUNCHES))
def test_equals_one_call_per_prompt(name):
    tb.equals_one_call_per_sequence(tb.RaggedBatch(TWO_LAUNCHES[name]))


def test_equal_scores():
    """Queries of zero: every prefix token of a prompt has the same score, up to the last bits, and what two launches
    select is what one call per prompt selects."""
    rb = tb.RaggedBatch(("cfg2", dict(n_kv_heads=2, n_q_heads=8, window=32, pool_kernel=1), (33000, 16500, 5000), (0, 1, 0)))
    rb.q_win[:] = 0
    for li in rb.layers:
        li.q_win[:] = 0
    tb.equals_one_call_per_sequence(rb)
