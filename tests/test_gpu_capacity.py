"""GPU parity at capacities up to the largest int32, with demands of a byte,
against the CPU oracle: the value table, every path of the evaluation, route
recovery, the hard fleet bound and served requests, on costs where a later predecessor is as cheap as the first or cheaper (all zero,
all equal, no triangle inequality), so that the route from the first customer
is not the only one that counts.  Bit-exact."""
import sys

import numpy as np
import pytest

import oracle
from paper_2602_05179_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

TOP = 2**31 - 1
S = 70


@pytest.fixture(scope="module")
def binding():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_05179_amd import binding as b
    return b


def _cases(n):
    rng = np.random.default_rng(n)
    N = n + 1
    tour = W.random_tour(rng, N)[:n]
    dem = rng.integers(0, 256, size=(S, N)).astype(np.int16)
    zero = np.zeros((N + 1, N + 1), np.int32)
    free = rng.integers(0, 1000, size=zero.shape).astype(np.int32)
    for cost, dist in (("zero", zero), ("equal", zero + 9), ("no triangle inequality", free),
                       ("rounded", W.dist_round(W.coords(rng, N)))):
        for Q in (TOP, TOP - 200 * n, 255 * n, 255 * n - 1):
            print("[case] %s n=%d Q=%d" % (cost, n, Q), flush=True)
            sys.stdout.flush()
            yield "%s, Q = %d" % (cost, Q), tour, dist, dem, Q


@pytest.mark.parametrize("n", (1, 2, 3, 20, 31))
def test_values_at_any_capacity(binding, n):
    for label, tour, dist, dem, Q in _cases(n):
        t, d, q = (torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (tour, dist, dem))
        V, status = binding.split_values_device(t, d, q, Q)
        got = V.cpu().numpy()
        assert int(status.item()) == 0, label
        for s in range(S):
            vals, _ = oracle.split_values(tour, dist, dem[s, tour - 1], Q)
            assert np.array_equal(got[:, s], vals[1:]), "%s, scenario %d" % (label, s)


# path 0: the one-launch form; 1: tiles in LDS; 2: the tour-ordered copy
@pytest.mark.parametrize("variant", ((32, 3, 4, 3), (64, 3, 4, 3), (32, 8, 3, 3), (64, 16, 4, 4)))
@pytest.mark.parametrize("path", (0, 1, 2))
@pytest.mark.parametrize("n", (1, 2, 3, 20, 31))
def test_evaluation_at_any_capacity(binding, n, path, variant):
    lens = np.array([n], np.int32)
    binding.set_schedule(*variant, waves=0, path=path)
    try:
        for label, tour, dist, dem, Q in _cases(n):
            t, l, d, q = (torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (tour, lens, dist, dem))
            out = binding.split_eval_device(t, l, d, q, Q, max_len=n)
            ref = oracle.split_eval(tour, lens, dist, dem, Q)
            assert np.array_equal(out.costs.cpu().numpy(), ref["costs"]), label
            assert np.array_equal(out.sums.cpu().numpy(), ref["sums"]), label
    finally:
        binding.set_schedule(0)


# a capacity as large as any load leaves every split open: demands past a byte too
def _wide(dem):
    dem = dem.copy()
    dem[64:, ::2] = 32767
    return dem


@pytest.mark.parametrize("wide", (False, True))
@pytest.mark.parametrize("n", (1, 2, 3, 20, 31))
def test_routes_at_any_capacity(binding, n, wide):
    try:
        for label, tour, dist, dem, Q in _cases(n):
            dem = _wide(dem) if wide else dem
            if Q < dem.max():
                continue
            t, d, q = (torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (tour, dist, dem))
            ref = oracle.split_routes(tour, dist, dem, Q)
            for variant in binding.ROUTE_VARIANTS:
                binding.set_route_variant(*variant)
                out = binding.split_routes_device(t, d, q, Q)
                got = out.host()
                assert np.array_equal(got["costs"], ref["costs"]), (label, variant)
                assert np.array_equal(got["nroutes"], ref["nroutes"]), (label, variant)
                assert np.array_equal(got["pred"].T, ref["pred"]), (label, variant)
    finally:
        binding.set_route_variant(0)


@pytest.mark.parametrize("wide", (False, True))
@pytest.mark.parametrize("K", (0, 1, 3))
@pytest.mark.parametrize("n", (1, 2, 3, 20, 31))
def test_fleet_at_any_capacity(binding, n, K, wide):
    for label, tour, dist, dem, Q in _cases(n):
        dem = _wide(dem) if wide else dem
        if Q < dem.max():
            continue
        t, d, q = (torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (tour, dist, dem))
        out = binding.split_variant_device(t, d, q, Q, beta=-1, K=K)
        ref = oracle.split_variant(tour, dist, dem, Q, beta=-1, K=K)
        ref = np.where(ref == oracle.INF64, np.iinfo(np.int32).max, ref)
        assert int(out.status.cpu()[0]) == 0, label
        assert np.array_equal(out.costs.cpu().numpy(), ref), label


@pytest.mark.parametrize("N", (31, 300))  # staged in LDS; the tour-ordered copy
def test_served_at_any_capacity(binding, N):
    srv = binding.Server(1 << 30, max_len=64)
    try:
        for label, tour, dist, dem, Q in _cases(N - 1):
            iid = srv.add_instance(dist, dem)
            for part in (tour[:1], tour[:2], tour[:20], tour[:31]):
                lens = np.array([part.size], np.int32)
                res = srv.wait(srv.submit(iid, part, Q, S, want_costs=True))
                ref = oracle.split_eval(part, lens, dist, dem, Q)
                assert np.array_equal(res["costs"], ref["costs"][0]), label
                assert res["sum"] == ref["sums"][0], label
    finally:
        srv.close()
