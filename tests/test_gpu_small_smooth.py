"""GPU parity of the one-launch evaluation on structured tours, which it gives
to the window scan or to the pruned stack by their routes' length, against the
CPU oracle: nearest-neighbour tours, routes on both sides of six stops in all or
some of the scenarios, windows past the ring, demands past a byte, ragged
tiles.  Bit-exact costs and sums.  And its time: such a tour costs a small call
no more than it does with the window scan forced on it."""
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


def _near_tour(dist, n):
    left, cur, out = set(range(1, n + 1)), 0, []
    while left:
        cur = min(left, key=lambda c: (dist[cur, c], c))
        left.remove(cur)
        out.append(cur)
    return np.array(out, np.int32)


def _device(*arrays):
    return [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in arrays]


@pytest.mark.parametrize("ring", (32, 64))
@pytest.mark.parametrize("n,S", ((1, 70), (4, 70), (5, 70), (15, 65), (16, 64), (17, 700), (63, 131), (100, 600), (250, 500)))
def test_one_launch_structured_tours(binding, n, S, ring):
    rng = np.random.default_rng(n)
    N = min(n + 3, 256)
    dist = W.dist_round(W.coords(rng, N))
    tour, lens = _near_tour(dist, n), np.array([n], np.int32)
    even = rng.integers(1, 12, size=(S, N)).astype(np.int16)
    mixed = even.copy()
    mixed[::2] = np.maximum(1, mixed[::2] // 6)  # long routes in every other scenario
    wide = even.copy()
    wide[S // 2, tour[-1] - 1] = 300
    binding.set_schedule(ring, 3, 4, 3, waves=0, path=0)
    try:
        for label, dem, Q in (("short routes", even, 25), ("long routes", even, 90), ("both", mixed, 40),
                              ("windows past the ring", even, 6 * n), ("past a byte", wide, 90)):
            print("[case] %s n=%d N=%d S=%d Q=%d ring=%d" % (label, n, N, S, Q, ring), flush=True)
            sys.stdout.flush()
            assert binding.eval_path(1, n, N, S, Q) == binding.PATH_ONE_LAUNCH
            ref = oracle.split_eval(tour, lens, dist, dem, Q)
            t, l, d, q = _device(tour, lens, dist, dem)
            out = binding.split_eval_device(t, l, d, q, Q, max_len=n)
            assert np.array_equal(out.costs.cpu().numpy(), ref["costs"]), label
            assert np.array_equal(out.sums.cpu().numpy(), ref["sums"]), label
    finally:
        binding.set_schedule(0)


def test_one_launch_time_on_structured_tours(binding):
    """n = 200, S = 500, 14 stops a route: 61 us on the stack, 42 on the scan."""
    rng = np.random.default_rng(4)
    n, S, Q = 200, 500, 150
    dist = W.dist_round(W.coords(rng, n))
    tour, lens = _near_tour(dist, n), np.array([n], np.int32)
    t, l, d, q = _device(tour, lens, dist, W.demands_normal(rng, S, rng.integers(1, 21, size=n)))
    best = {}
    try:
        for _ in range(3):
            for variant in ((32, 3, 4, 3), (32, 8, 3, 3)):
                binding.set_schedule(*variant, waves=0, path=0)
                out = binding.split_eval_device(t, l, d, q, Q, max_len=n)
                a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                torch.cuda.synchronize()
                a.record()
                for _ in range(100):
                    binding.split_eval_device(t, l, d, q, Q, max_len=n, out=out, workspace=out.workspace)
                b.record()
                torch.cuda.synchronize()
                best[variant] = min(best.get(variant, 1e9), a.elapsed_time(b))
    finally:
        binding.set_schedule(0)
    assert best[(32, 3, 4, 3)] < 1.2 * best[(32, 8, 3, 3)], best
