"""Single-launch routing: how a batch's tokens are shared out over workgroups (parts that begin in one block of tokens and end in
the next, parts of several blocks, prompts shorter than one part), and every kernel width that it pools itself."""
import pytest

torch = pytest.importorskip("torch")

import test_gpu_batch as tb

pytestmark = pytest.mark.gpu

POOLS = {"pool_%s_%d" % (mode, kernel): ("cfg2", dict(n_kv_heads=2, n_q_heads=4, window=16, pool_kernel=kernel, pool_mode=mode), (700, 4101), (0, 1))
         for mode in ("avg", "max") for kernel in (1, 3, 5, 7, 9, 11, 13, 15, 17)}
POOLS.update({
    "kernel_13_short": ("cfg2", dict(n_kv_heads=2, n_q_heads=8, window=32, pool_kernel=13), (700, 2048, 6100, 32), (5, 0, 1, 0)),
    "kernel_13_more_prompts_than_arguments_hold": ("cfg1", dict(n_kv_heads=1, n_q_heads=2, window=20, pool_kernel=13), tuple(70 + 131 * i for i in range(20)),
                                                   tuple(i % 3 for i in range(20))),
})
PARTS = {
    # 24 heads: parts of 4 units of 256 tokens, up to four blocks of 4096 tokens a head
    "parts_inside_blocks": ("cfg2", dict(n_kv_heads=8, n_q_heads=8, window=16, head_dim=64), (12289, 16384, 300), (0, 1, 0)),
    # one part per head, of two blocks of 2048 tokens
    "parts_whole_heads": ("cfg2", dict(n_kv_heads=64, n_q_heads=64, window=16, head_dim=64), (4000, 2049, 700, 64, 3000), (0, 0, 2, 0, 1)),
}
# parts of 6 units, some from one block into the next: one block's end and two; sixteen waves (blocks of 16 units) and eight (8)
ACROSS = {
    "across_blocks_of_4096": ("cfg2", dict(n_kv_heads=8, n_q_heads=8, window=16, head_dim=64), (8192, 2048, 5121, 7000, 3333, 6144, 4097, 2900), (0, 0, 2, 0, 1, 0, 0, 3)),
    "across_two_ends": ("cfg2", dict(n_kv_heads=12, n_q_heads=12, window=16, head_dim=64), (8192, 16384, 5000), (0, 1, 0)),
    "across_blocks_of_2048": ("cfg2", dict(n_kv_heads=17, n_q_heads=17, window=16, head_dim=64), (4096, 2300, 3500, 1000, 2700, 3100), (0, 0, 1, 0, 2, 0)),
}
ALL = {**POOLS, **PARTS, **ACROSS}


def parts_across(lens, heads):
    """(prompt, first unit, last unit) of the parts that begin inside one block and end in another: units per part as few as give
    no more than 256 workgroups."""
    units = [-(-n // 256) for n in lens]
    per_part = next(u for u in range(1, 65) if u >= max(units) or sum(-(-x // u) for x in units) * heads <= 256)
    block = 8 if max(lens) <= 4096 else 16
    return [(b, u, min(u + per_part, units[b]) - 1) for b in range(len(lens)) for u in range(0, units[b], per_part)
            if u % block and u // block != (min(u + per_part, units[b]) - 1) // block]


def test_which_cases_have_parts_across_blocks():
    for name, case in {**PARTS, **ACROSS}.items():
        across = parts_across(case[2], case[1]["n_kv_heads"])
        assert len(across) >= 2 if name in ACROSS else not across, name


@pytest.mark.parametrize("name", list(ALL))
def test_equals_one_call_per_prompt(name):
    tb.equals_one_call_per_sequence(tb.RaggedBatch(ALL[name]))


@pytest.mark.parametrize("name", list(POOLS) + list(ACROSS))
def test_against_the_oracle(name):
    tb.against_the_oracle(tb.RaggedBatch(ALL[name]), name)
