"""Decode launches whose pieces of approximated rows apply W themselves, and those that leave it to the merge: as many workgroups as
the first may have and one sequence more, the most query heads that it takes and more, pieces of one row, and a retained
segment or a sequence without rows beside them."""
import pytest

pytest.importorskip("torch")

from test_gpu_decode_splits import run, run_paged

pytestmark = pytest.mark.gpu


# one step of rows in either segment and eight KV heads: two workgroups each, 256 of them with 16 sequences
@pytest.mark.parametrize("sequences", [16, 17])
@pytest.mark.parametrize("d,G", [(64, 1), (64, 8), (128, 1), (128, 8), (128, 10)])
def test_most_workgroups(d, G, sequences):
    run(d, G, 8, [100 - b for b in range(sequences)], [97] * sequences, ragged=False, seed=d + G + sequences)


@pytest.mark.parametrize("lens,n_apx", [([0], 1), ([1], 33), ([300], 128), ([0, 129], 129), ([5], 1000)])
@pytest.mark.parametrize("d,G", [(64, 5), (128, 7)])
def test_pieces(d, G, lens, n_apx):
    run(d, G, 3, lens, [n_apx] * len(lens), ragged=False, seed=n_apx + d)


@pytest.mark.parametrize("d", [64, 128])
def test_paged(d):
    run_paged(d, 8, 2, [70, 0, 31], 150, 16, 8, False, d)
