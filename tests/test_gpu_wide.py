"""GPU parity for demands past a byte (int16 tiles staged half at a time)
against the CPU oracle: odd pools, ragged last tiles on either side of half a
tile, several tours per workgroup, the largest demands and capacities, and a
negative demand on and off the tour.  Bit-exact costs and sums."""
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


def _run(binding, tours, lens, dist, dem, Q, label):
    print("[case] %s N=%d S=%d Q=%d" % (label, dist.shape[0] - 1, dem.shape[0], Q), flush=True)
    sys.stdout.flush()
    t, l, d, q = (torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (tours, lens, dist, dem))
    out = binding.split_eval_device(t, l, d, q, Q, max_len=int(lens.max()))
    return out.costs.cpu().numpy(), out.sums.cpu().numpy()


def _same(binding, tours, lens, dist, dem, Q, label):
    costs, sums = _run(binding, tours, lens, dist, dem, Q, label)
    ref = oracle.split_eval(tours, lens, dist, dem, Q)
    assert np.array_equal(costs, ref["costs"]), label
    assert np.array_equal(sums, ref["sums"]), label


# path 0: the one-launch form where it fits; 1: the general kernels
@pytest.mark.parametrize("path", (0, 1))
@pytest.mark.parametrize("n,N,S", [(1, 1, 1), (2, 3, 31), (7, 9, 32), (20, 21, 33), (33, 40, 65), (100, 101, 160),
                                   (150, 150, 129)])
def test_wide_demands(binding, n, N, S, path):
    rng = np.random.default_rng(n * 1000 + S)
    dist = W.dist_round(W.coords(rng, N))
    tour = W.random_tour(rng, N)[:n]
    lens = np.array([n], np.int32)
    fine = W.demands_normal(rng, S, rng.integers(1, 401, size=N))
    mixed = rng.integers(0, 20, size=(S, N)).astype(np.int16)
    mixed[S // 2, tour[0] - 1] = 256
    huge = rng.integers(30000, 32768, size=(S, N)).astype(np.int16)
    binding.set_schedule(32, 3, 4, 3, waves=0, path=path)
    try:
        _same(binding, tour, lens, dist, fine, 3000, "fine units")
        _same(binding, tour, lens, dist, mixed, 300, "one demand past a byte")
        _same(binding, tour, lens, dist, huge, 32767, "the largest demands")
        _same(binding, tour, lens, dist, huge, 2**31 - 1, "no capacity bound")
    finally:
        binding.set_schedule(0)


def test_wide_batch(binding):
    """Four and more tours per workgroup share the half tiles; one is empty."""
    rng = np.random.default_rng(5)
    N, S = 260, 100
    dist = W.dist_round(W.coords(rng, N))
    dem = W.demands_normal(rng, S, rng.integers(1, 301, size=N))
    tours = [W.random_tour(rng, N)[:k] for k in (40, 260, 0, 77, 130, 5)]
    lens = np.array([t.size for t in tours], np.int32)
    _same(binding, np.concatenate(tours).astype(np.int32), lens, dist, dem, 2500, "batch")


def test_negative_demand_in_a_wide_tile(binding):
    rng = np.random.default_rng(6)
    N, n, S, Q = 30, 25, 100, 2000
    dist = W.dist_round(W.coords(rng, N))
    dem = W.demands_normal(rng, S, rng.integers(100, 301, size=N))
    tour = np.arange(1, n + 1, dtype=np.int32)
    lens = np.array([n], np.int32)
    off = dem.copy()
    off[40, N - 1] = -5  # not on the tour
    for path in (0, 1):
        binding.set_schedule(32, 3, 4, 3, waves=0, path=path)
        try:
            costs, _ = _run(binding, tour, lens, dist, off, Q, "negative off the tour")
            clean = off.copy()
            clean[40, N - 1] = 5
            assert np.array_equal(costs, oracle.split_eval(tour, lens, dist, clean, Q)["costs"])
            on = dem.copy()
            on[70, tour[3] - 1] = -1
            costs, sums = _run(binding, tour, lens, dist, on, Q, "negative on the tour")
            assert sums[0] == binding.SPLIT_SUM_INVALID and (costs == binding.SPLIT_INF).all()
        finally:
            binding.set_schedule(0)
