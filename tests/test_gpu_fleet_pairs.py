"""GPU parity of the hard fleet bound against the CPU oracle where two waves
share a tile (one counts routes, the other runs the passes) and where one wave
runs both: calls on either side of the line between them, tiles in LDS and
the tour-ordered copy, both rings, fleets that answer every tile, some or none,
windows past the ring, demands past a byte, captured calls.  And the time of a
small call whose counting pass answers nothing."""
import os

import numpy as np
import pytest

import oracle
from paper_2602_05179_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

THREADS = max(1, min(16, len(os.sched_getaffinity(0))))
INF32 = np.iinfo(np.int32).max


@pytest.fixture(scope="module")
def binding():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_05179_amd import binding as b
    return b


def _device(*arrays):
    return [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in arrays]


def _want(tour, dist, dem, Q, K):
    r = oracle.split_variant(tour, dist, dem, Q, beta=-1, K=K, nthreads=THREADS)
    return np.where(r == oracle.INF64, INF32, r).astype(np.int32)


def _check(binding, tour, dist, dem, Q, K, label):
    print("[case] %s n=%d N=%d S=%d Q=%d K=%d" % (label, tour.size, dist.shape[0] - 1, dem.shape[0], Q, K), flush=True)
    out = binding.split_variant_device(*_device(tour, dist, dem), Q, beta=-1, K=K)
    got = out.costs.cpu().numpy()
    assert int(out.status.cpu()[0]) == 0
    assert np.array_equal(got, _want(tour, dist, dem, Q, K)), label


# 1024 and 1536 tiles are the lines (ring 64 or tour-ordered; ring 32 in LDS)
@pytest.mark.parametrize("Q,S", ((60, 64 * 1536), (60, 64 * 1536 + 1), (250, 64 * 1024 - 5), (250, 64 * 1024 + 70)))
def test_fleet_at_the_line(binding, Q, S):
    rng = np.random.default_rng(Q + S)
    n = 24
    dist = W.dist_round(W.coords(rng, n))
    tour = W.random_tour(rng, n)
    dem = rng.integers(1, 12 if Q == 60 else 40, size=(S, n)).astype(np.int16)
    least = dem.sum(1).max() / Q
    for ratio in (1.0, 1.41, 1.7):
        _check(binding, tour, dist, dem, Q, max(1, int(np.ceil(ratio * least))), "ratio %.2f" % ratio)


@pytest.mark.parametrize("path", (1, 2))  # tiles in LDS, tour-ordered copy
@pytest.mark.parametrize("Q", (60, 250))
@pytest.mark.parametrize("n,N", ((1, 1), (16, 16), (17, 17), (33, 40), (64, 130), (100, 100), (200, 200)))
def test_fleet_pairs(binding, n, N, Q, path):
    rng = np.random.default_rng(n + Q + path)
    S = 64 * 5 + 9
    dist = W.dist_round(W.coords(rng, N))
    tour = W.random_tour(rng, N)[:n]
    dem = rng.integers(1, 12 if Q == 60 else 30, size=(S, N)).astype(np.int16)
    dem[64:128] = np.maximum(1, dem[64:128] // 4)  # one tile of light loads: answered where others are not
    least = dem[:, tour - 1].sum(1).max() / Q
    binding.set_variant_path(path)
    try:
        for ratio in (0.9, 1.2, 1.38, 1.42, 1.5, 2.5):
            _check(binding, tour, dist, dem, Q, max(1, int(np.ceil(ratio * least))), "ratio %.2f" % ratio)
        dem[3, tour[n // 2] - 1] = Q + 1  # no split
        dem[200, tour[0] - 1] = 300  # past a byte: its tile is redone
        _check(binding, tour, dist, dem, Q, max(1, int(np.ceil(1.6 * least))), "no split, redone tile")
    finally:
        binding.set_variant_path(0)


@pytest.mark.parametrize("Q", (90, 210))
def test_fleet_windows_past_the_ring(binding, Q):
    """Vehicles of 45 to 100 stops: the counting pass leaves its ring in some
    tiles, and the passes do."""
    rng = np.random.default_rng(Q)
    n, S = 120, 64 * 4 + 3
    dist = W.dist_round(W.coords(rng, n))
    tour = W.random_tour(rng, n)
    dem = rng.integers(1, 4, size=(S, n)).astype(np.int16)
    dem[:128] *= 8
    least = dem.sum(1).max() / Q
    for K in (max(1, int(np.ceil(least))), int(np.ceil(1.5 * least)), n):
        _check(binding, tour, dist, dem, Q, K, "long windows")


def test_fleet_pairs_captured(binding):
    rng = np.random.default_rng(12)
    n, S, Q, K = 60, 64 * 20, 60, 12
    dist = W.dist_round(W.coords(rng, n))
    tour = W.random_tour(rng, n)
    dem = rng.integers(1, 12, size=(S, n)).astype(np.int16)
    dem[: S // 2] = np.maximum(1, dem[: S // 2] // 2)
    t, d, q = _device(tour, dist, dem)
    out = binding.split_variant_device(t, d, q, Q, beta=-1, K=K)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        binding.split_variant_device(t, d, q, Q, beta=-1, K=K, out=out, workspace=out.workspace)
    for turn in range(4):
        out.costs.fill_(-1)
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(out.costs.cpu().numpy(), _want(tour, dist, dem, Q, K)), turn
        dem = np.roll(dem, 7, axis=0)  # the next replay sees other demands
        q.copy_(torch.from_numpy(dem))


def test_fleet_time_of_a_pass_in_vain(binding):
    """n = 40, S = 5000, Q = 80, K = 9 on a random tour, where most tiles hold a
    scenario that takes ten routes: 45.3 us for the passes alone, 53.2 with the
    counting pass before them."""
    rng = np.random.default_rng(1)
    n, S, Q, K = 40, 5000, 80, 9
    dist = W.dist_round(W.coords(rng, n))
    mu = rng.integers(1, 21, size=n)
    t, d, q = _device(W.random_tour(rng, n), dist, W.demands_normal(rng, S, mu))
    out = binding.split_variant_device(t, d, q, Q, beta=-1, K=K)
    best = 1e9
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        torch.cuda.synchronize()
        a.record()
        for _ in range(100):
            binding.split_variant_device(t, d, q, Q, beta=-1, K=K, out=out, workspace=out.workspace)
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) * 10)
    assert best < 49, best
