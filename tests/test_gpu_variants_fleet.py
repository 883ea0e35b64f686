"""GPU parity of the fleet bound's one-pass answer against the CPU oracle: K
on both sides of the line where it is tried (vehicles that hold 7/5 of the
largest load in a tile), tiles in which only some scenarios keep to K, equal
costs with different numbers of routes, scenarios without a split, tiles
redone, and costs too large to carry the count; whole rows, gathered rows and
the tour-ordered copy, tour lengths around the ring lengths."""
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


def _check(binding, tour, dist, dem, Q, K, label):
    print("[case] %s n=%d N=%d S=%d Q=%d K=%d" % (label, tour.size, dist.shape[0] - 1, dem.shape[0], Q, K), flush=True)
    t, d, q = (torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (tour, dist, dem))
    out = binding.split_variant_device(t, d, q, Q, beta=-1, K=K)
    got = out.costs.cpu().numpy()
    assert int(out.status.cpu()[0]) == 0
    r = oracle.split_variant(tour, dist, dem, Q, beta=-1, K=K, nthreads=THREADS)
    want = np.where(r == oracle.INF64, INF32, r).astype(np.int32)
    assert np.array_equal(got, want), label


# n, N: whole rows, a tour in a pool twice its size (gathered), long rows
# (tour-ordered copy)
SHAPES = [(1, 1), (2, 2), (7, 7), (31, 31), (32, 33), (33, 33), (63, 64), (64, 64), (65, 65), (100, 100),
          (40, 90), (129, 300), (390, 400)]


@pytest.mark.parametrize("Q", (60, 250))  # both rings
@pytest.mark.parametrize("n,N", SHAPES)
def test_fleet_one_pass(binding, n, N, Q):
    rng = np.random.default_rng(7 * n + Q)
    S = 64 * 3 + 13
    dist = W.dist_round(W.coords(rng, N))
    tour = W.random_tour(rng, N)[:n]
    dem = rng.integers(1, 12 if Q == 60 else 30, size=(S, N)).astype(np.int16)
    least = dem[:, tour - 1].sum(1).max() / Q
    for ratio in (1.0, 1.25, 1.39, 1.41, 1.6, 3.0):
        _check(binding, tour, dist, dem, Q, max(1, int(np.ceil(ratio * least))), "ratio %.2f" % ratio)
    dem[5, tour[n // 2] - 1] = Q + 1  # no split
    dem[70, tour[0] - 1] = 300  # past a byte: its tile is redone
    _check(binding, tour, dist, dem, Q, max(1, int(np.ceil(1.6 * least))), "no split, redone tile")


def test_fleet_one_pass_ties_and_scale(binding):
    rng = np.random.default_rng(3)
    n, S, Q = 90, 200, 60
    tour = W.random_tour(rng, n)
    dem = rng.integers(1, 12, size=(S, n)).astype(np.int16)
    least = int(np.ceil(dem.sum(1).max() / Q))
    # a return to the depot costs nothing: the same cost with few or many routes
    flat = np.zeros((n + 1, n + 1), np.int32)
    for K in (least, int(1.45 * least) + 1, 2 * least):
        _check(binding, tour, flat, dem, Q, K, "equal costs")
    near = W.dist_round(W.coords(rng, n))
    for scale in (1, 30, 1000):  # the count fits, fits by the table only or not, does not fit
        _check(binding, tour, (near * scale).astype(np.int32), dem, Q, int(1.6 * least), "costs x %d" % scale)
