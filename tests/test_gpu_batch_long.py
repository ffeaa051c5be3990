"""Batches of unequal prompts whose routing takes two launches, prompts beyond the length of one, and wide pooling kernels.  Their parameter blocks are kernel arguments, or a table when there are many."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import test_gpu_batch as tb

pytestmark = pytest.mark.gpu

TWO_LAUNCHES = {
    "long_bf16_three": ("cfg2", dict(n_kv_heads=2, n_q_heads=8, window=32), (17000, 4100, 20011), (3, 0, 1)),
    # pools for 16, 32 and 64 register slots per thread, and one that exceeds them
    "long_bf16_wide_pool": ("cfg2", dict(n_kv_heads=1, n_q_heads=2, window=16), (40000, 17001, 70000), (0, 2, 0), ((12000, 6000), (17001, 100), (60000, 59000))),
    "long_f32_max_pool_kernel_11": ("cfg1", dict(n_kv_heads=2, n_q_heads=4, window=20, pool_kernel=11, pool_mode="max"), (1500, 18000), (0, 5)),
    "kernel_13_short": ("cfg2", dict(n_kv_heads=2, n_q_heads=8, window=32, pool_kernel=13), (700, 2048, 6100, 32), (5, 0, 1, 0)),
    "kernel_13_more_prompts_than_arguments_hold": ("cfg1", dict(n_kv_heads=1, n_q_heads=2, window=20, pool_kernel=13), tuple(70 + 131 * i for i in range(20)),
                                                   tuple(i % 3 for i in range(20))),
}
tb.BATCHES.update(TWO_LAUNCHES)


@pytest.mark.parametrize("name", list(TWO_LAUNCHES))
def test_against_the_oracle(name):
    tb.test_compress_batch_against_the_oracle_sequence_by_sequence(name)


@pytest.mark.parametrize("name", [x for x in TWO_LAUNCHES if TWO_LAUNCHES[x][0] == "cfg2"])
def test_equals_one_call_per_prompt(name):
    tb.test_compress_batch_equals_one_call_per_sequence(name)


def test_equal_scores():
    """Queries of zero: every prefix token of a prompt has the same score, up to the last bits, and what two launches
    select is what one call per prompt selects."""
    tb.BATCHES["long_flat"] = ("cfg2", dict(n_kv_heads=2, n_q_heads=8, window=32, pool_kernel=1), (33000, 16500, 5000), (0, 1, 0))
    make = tb.RaggedBatch.__init__

    def flat(self, name):
        make(self, name)
        self.q_win[:] = 0
        for li in self.layers:
            li.q_win[:] = 0
    tb.RaggedBatch.__init__ = flat
    try:
        tb.test_compress_batch_equals_one_call_per_sequence("long_flat")
    finally:
        tb.RaggedBatch.__init__ = make
