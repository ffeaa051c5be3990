"""Batches of unequal prompts: how the passes' workgroups are dealt out.  Fewer workgroups than XCDs, numbers of heads and of
workgroups that eight does not divide, as many prompts as one launch takes, chunks of several tiles."""
import pytest

torch = pytest.importorskip("torch")

import test_gpu_batch as tb

pytestmark = pytest.mark.gpu

CASES = {
    "wgs_two": ("cfg2", dict(n_kv_heads=1, n_q_heads=4, window=16), (40, 64), (0, 1)),
    "wgs_three_heads": ("cfg2", dict(n_kv_heads=3, n_q_heads=6, window=32), (1000, 130, 4100, 64, 2049), (0, 1, 0, 2, 0)),
    "wgs_five_heads_512_rows": ("cfg2", dict(n_kv_heads=5, n_q_heads=40, window=64), (700, 3333, 90), (1, 0, 0)),
    "wgs_sixty_four_prompts": ("cfg2", dict(n_kv_heads=2, n_q_heads=4, window=16, head_dim=64), tuple(100 + 37 * ((11 * i) % 64) for i in range(64)), (0,) * 64),
}


@pytest.mark.parametrize("name", list(CASES))
def test_equals_one_call_per_prompt(name):
    tb.equals_one_call_per_sequence(tb.RaggedBatch(CASES[name]))


def test_against_the_oracle():
    tb.against_the_oracle(tb.RaggedBatch(CASES["wgs_three_heads"]), "wgs_three_heads")
