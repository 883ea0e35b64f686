"""GPU parity of the value table's tile kernel against the CPU oracle: tour
lengths around the ring lengths with both rings, scenarios without a split in
byte and int16 tiles, a ragged last half tile, and the calls the general
kernel keeps (demands not 16-byte aligned, pools past the LDS)."""
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


def _check(binding, tour, dist, dem, Q, label, dem_dev=None):
    print("[case] %s n=%d N=%d S=%d Q=%d" % (label, tour.size, dist.shape[0] - 1, dem.shape[0], Q), flush=True)
    sys.stdout.flush()
    t, d = (torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (tour, dist))
    q = torch.from_numpy(np.ascontiguousarray(dem)).cuda() if dem_dev is None else dem_dev
    V, status = binding.split_values_device(t, d, q, Q)
    got = V.cpu().numpy()
    assert int(status.item()) == 0, label
    for s in range(dem.shape[0]):
        vals, _ = oracle.split_values(tour, dist, dem[s, tour - 1], Q)
        want = [binding.SPLIT_INF if v is None else v for v in vals[1:]]
        assert np.array_equal(got[:, s], want), "%s scenario %d" % (label, s)


@pytest.mark.parametrize("Q", (60, 300))
@pytest.mark.parametrize("n", (1, 2, 6, 7, 8, 31, 32, 33, 63, 64, 65, 100))
def test_values_tiles(binding, n, Q):
    rng = np.random.default_rng(n + Q)
    N, S = n + 1, 70
    dist = W.dist_round(W.coords(rng, N))
    tour = W.random_tour(rng, N)[:n]
    dem = rng.integers(1, 15, size=(S, N)).astype(np.int16)
    _check(binding, tour, dist, dem, Q, "bytes")
    dem[3, tour[n // 2] - 1] = 200  # above 60
    dem[65:, tour[0] - 1] = 61
    _check(binding, tour, dist, dem, Q, "no split in some, bytes")
    dem[10, tour[-1] - 1] = 400
    dem[40, tour[n // 3] - 1] = 301
    _check(binding, tour, dist, dem, Q, "no split in some, int16")


def test_values_general_kernel(binding):
    rng = np.random.default_rng(9)
    N, n, S, Q = 21, 20, 70, 50
    dist = W.dist_round(W.coords(rng, N))
    tour = W.random_tour(rng, N)[:n]
    dem = rng.integers(1, 15, size=(S, N)).astype(np.int16)
    flat = torch.zeros(S * N + 1, dtype=torch.int16, device="cuda")
    flat[1:] = torch.from_numpy(dem.reshape(-1)).cuda()
    shifted = flat[1:].view(S, N)
    assert shifted.data_ptr() % 16 == 2
    _check(binding, tour, dist, dem, Q, "demands not aligned", dem_dev=shifted)
    N = 2600
    dist = W.dist_round(W.coords(rng, N))
    dem = rng.integers(1, 15, size=(S, N)).astype(np.int16)
    _check(binding, W.random_tour(rng, N)[:n], dist, dem, Q, "pool past the LDS")


@pytest.mark.parametrize("wide", (False, True))
@pytest.mark.parametrize("n", (1, 2, 3, 7, 8, 20, 31, 32, 33, 64, 100))
def test_values_ends_at_the_last_row(binding, n, wide):
    """Windows of one to three customers keep the stack shallow, so nothing but
    the end of the tour sends the recursion out of its usual path at position
    n: the rows after the table's last one keep what they held."""
    rng = np.random.default_rng(n)
    N, S, Q, spare = n + 1, 70, 600 if wide else 30, 160
    dist = W.dist_round(W.coords(rng, N))
    tour = W.random_tour(rng, N)[:n]
    lo, hi = (200, 301) if wide else (10, 16)
    dem = rng.integers(lo, hi, size=(S, N)).astype(np.int16)
    print("[case] last row n=%d wide=%s" % (n, wide), flush=True)
    rows = torch.full((n + spare, S), -7, dtype=torch.int32, device="cuda")
    t, d, q = (torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (tour, dist, dem))
    _, status = binding.split_values_device(t, d, q, Q, V=rows[:n])
    got = rows.cpu().numpy()
    assert int(status.item()) == 0
    assert (got[n:] == -7).all()
    for s in range(S):
        vals, _ = oracle.split_values(tour, dist, dem[s, tour - 1], Q)
        want = [binding.SPLIT_INF if v is None else v for v in vals[1:]]
        assert np.array_equal(got[:n, s], want), s
