"""A workspace asked for once, for the longest tours and the most scenarios of a
pool, is enough for every shorter or smaller call on it (no GPU needed): the
path that a call takes depends on both, and some paths need more room."""
import pytest

from paper_2602_05179_amd import binding


@pytest.fixture(autouse=True)
def _automatic():
    binding.set_schedule(0)
    binding.tune_clear()
    yield
    binding.set_schedule(0)


@pytest.mark.parametrize("T", (1, 2, 3, 8, 40))
@pytest.mark.parametrize("N", (20, 255, 256, 257, 300, 320, 321, 400, 1000, 2000, 2400))
def test_enough_for_smaller_calls(T, N):
    lens = sorted({1, 2, max(1, N // 2 - 1), N // 2, N // 2 + 1, N - 1, N} - {0})
    scen = (1, 64, 65, 1000, 20_000, 40_000, 70_000, 400_000)
    size = {(m, S): binding.workspace_bytes(T, m, N, S, 150) for m in lens for S in scen}
    for m in lens:
        for S in scen:
            for m2 in (x for x in lens if x <= m):
                for S2 in (x for x in scen if x <= S):
                    assert size[m, S] >= size[m2, S2], (T, N, m, S, m2, S2)


def test_room_for_the_copy_of_a_shorter_tour():
    N, S = 300, 20_000  # whole-pool tours stay in LDS here, half of the pool takes the tour-ordered copy
    assert binding.eval_path(1, N, N, S, 150) == binding.PATH_TILES
    assert binding.eval_path(1, N // 2 - 1, N, S, 150) == binding.PATH_ORDERED
    assert binding.workspace_bytes(1, N, N, S, 150) >= S * N
