"""GPU parity of the value table on tours over part of the pool, whose demands
are gathered instead of staged as whole rows, against the CPU oracle: both
sides of the line, byte and int16 demands, demands past a byte and negative
ones off the tour, ragged half tiles.  And its time on a short tour in a large
pool."""
import sys

import numpy as np
import pytest

import oracle
from paper_2602_05179_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def binding():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_05179_amd import binding as b
    return b


def _device(*arrays):
    return [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in arrays]


def _check(binding, tour, dist, dem, Q, label):
    print("[case] %s n=%d N=%d S=%d Q=%d" % (label, tour.size, dist.shape[0] - 1, dem.shape[0], Q), flush=True)
    sys.stdout.flush()
    V, status = binding.split_values_device(*_device(tour, dist, dem), Q)
    got = V.cpu().numpy()
    assert int(status.item()) == 0, label
    for s in range(dem.shape[0]):
        vals, _ = oracle.split_values(tour, dist, dem[s, tour - 1], Q)
        want = [binding.SPLIT_INF if v is None else v for v in vals[1:]]
        assert np.array_equal(got[:, s], want), "%s scenario %d" % (label, s)


@pytest.mark.parametrize("S", (70, 128, 97))
@pytest.mark.parametrize("Q", (60, 300))
@pytest.mark.parametrize("n,N", ((1, 3), (1, 257), (2, 300), (42, 257), (43, 257), (31, 400), (64, 384), (64, 383), (100, 900), (150, 900),
                                 (20, 2559), (20, 2560), (20, 2561)))
def test_values_part_of_the_pool(binding, n, N, Q, S):
    rng = np.random.default_rng(n + N + Q + S)
    dist = W.dist_round(W.coords(rng, N))
    tour = W.random_tour(rng, N)[:n]
    dem = rng.integers(1, 15, size=(S, N)).astype(np.int16)
    off = np.setdiff1d(np.arange(1, N + 1), tour)
    dem[7, off[0] - 1] = 999  # off the tour
    _check(binding, tour, dist, dem, Q, "bytes")
    dem[3, tour[n // 2] - 1] = Q + 1
    dem[65:, tour[0] - 1] = 256
    dem[9, off[-1] - 1] = -4
    _check(binding, tour, dist, dem, Q, "no split in some, int16, a negative demand off the tour")


def test_values_time_of_a_short_tour(binding):
    """Five customers of 2000, S = 5e4: 98 us with whole rows staged, 13 without."""
    rng = np.random.default_rng(1)
    n, N, S, Q = 5, 2000, 50_000, 60
    dist = W.dist_round(W.coords(rng, N))
    tour, d = _device(W.random_tour(rng, N)[:n], dist)
    dem = torch.randint(1, 21, (S, N), device="cuda", dtype=torch.int16)
    V, st = torch.empty((n, S), dtype=torch.int32, device="cuda"), torch.empty(1, dtype=torch.int32, device="cuda")
    ws = torch.empty(binding.values_workspace_bytes(n, N, S), dtype=torch.uint8, device="cuda")
    best = 1e9
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(50):
            binding.split_values_device(tour, d, dem, Q, V=V, status=st, workspace=ws)
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) / 50 * 1e3)
    assert best < 60, best
