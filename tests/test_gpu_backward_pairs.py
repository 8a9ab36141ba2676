"""The gradient of a bf16 batch where two waves share a unit or a tile: one to nine units of 32 rows a KV head (halves of eight
with none, some and all of four), calls of one to nine tiles (fewer than the ring holds, not a multiple of four), a split of the
rows' walk or none; fp64 gradients and the bar of test_gpu_backward_precision."""
import pytest

from tests.test_gpu_backward_precision import run_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h_q,h_kv,n_q", [(1, 1, 1), (2, 2, 40), (3, 1, 33), (4, 2, 70), (8, 2, 31), (5, 1, 32), (9, 1, 20)])
@pytest.mark.parametrize("lens", [[9], [33], [32, 32], [5, 70, 32], [40, 100, 61]])
def test_units_and_tiles(h_q, h_kv, n_q, lens):
    n = len(lens)
    run_case(lens + [n_q], [([(m, 11 * m) for m in range(n)], n, 500, n_q)], h_q, h_kv)


def test_two_calls_over_the_same_messages():
    run_case([64, 3, 290, 45, 80], [([(0, 5), (2, 90), (1, 0)], 3, 700, 45), ([(2, 3), (0, 400), (0, 9)], 4, 512, 80)], 6, 2)


# (8 units in workgroups of 4; units that the workgroups do not share evenly; a call whose rows are the last of a longer message; own
#  tiles behind the parents' last group of four, and in it)
@pytest.mark.parametrize("lens,calls", [
    ([200, 43, 31], [([(0, 0)], 1, 200, 43), ([(0, 5), (0, 300)], 2, 600, 31)]),
    ([96, 330], [([(0, 0)], 1, 100, 330)]),
    ([128, 420], [([(0, 7)], 1, 140, 100)]),
    ([330], [([], 0, 0, 330)]),
])
def test_units_split_over_workgroups(lens, calls):
    run_case(lens, calls, 8, 2)
