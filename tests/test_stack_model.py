"""The pruned-stack recursion's machine code on a host model of a wave
(stack_model.py), against the definition: both rings, every demand source and
the value table, tours in which almost everything or nothing is removed, ties,
scenarios without a split, windows past the ring, ragged waves, and the largest
capacity.  Every table read, demand read and row store is bounds-checked, every
load has to be waited for, and the code has to end."""
import shutil

import numpy as np
import pytest

import stack_model as M

pytestmark = pytest.mark.skipif(any(shutil.which(t) is None for t in M.TOOLS), reason="LLVM tools not available")

INF = 1 << 30
VARIANTS = [(r, s, o) for r in (32, 64) for s, o in (("LDS", "NONE"), ("LDS16", "NONE"), ("STREAM", "NONE"), ("LDS", "VALUES"),
                                                      ("LDS16", "VALUES"))]


@pytest.fixture(scope="module", params=VARIANTS, ids=lambda p: "%d-%s-%s" % p)
def variant(request, tmp_path_factory):
    ring, src, out = request.param
    code = M.assemble(M.source(ring, src, out), str(tmp_path_factory.mktemp("stack")))
    # the size that the header tells the compiler to count for the block
    assert code[-1][0] < {32: 32768, 64: 106496}[ring]
    return ring, src, out, code


def _near(dist, n):
    left, cur, out = set(range(1, n + 1)), 0, []
    while left:
        cur = min(left, key=lambda c: (dist[cur, c], c))
        left.remove(cur)
        out.append(cur)
    return np.array(out)


def _cases(wide):
    k = 40 if wide else 1
    for n, lanes in ((1, 64), (2, 1), (3, 64), (4, 37), (5, 64), (8, 33), (33, 64), (70, 64)):
        rng = np.random.default_rng(n)
        xy = rng.integers(0, 1001, size=(n + 1, 2))
        dist = np.rint(np.hypot(*(xy[:, None] - xy[None]).transpose(2, 0, 1))).astype(np.int64)
        dem = rng.integers(1, 12, size=(64, n)) * k
        near, random = _near(dist, n), 1 + rng.permutation(n)
        yield "random", lanes, random, dist, dem, 60 * k
        yield "one customer a route", lanes, random, dist, dem, 11 * k
        yield "near", lanes, near, dist, dem, 100 * k
        yield "ties", lanes, random, np.full_like(dist, 7), dem, 40 * k
        yield "free", lanes, random, np.zeros_like(dist), dem, 90 * k
        yield "no triangle inequality", lanes, random, rng.integers(0, 1000, size=dist.shape), dem, 70 * k
        some = dem.copy()
        some[5 % lanes, n // 2] = 61 * k
        some[lanes // 2 :, 0] = 200 if not wide else 32767
        yield "no split in some", lanes, random, dist, some, 60 * k
        if n > 8:
            yield "long windows", lanes, near, dist, dem, 6 * n * k
            yield "one route", lanes, random, dist, dem, 20 * n * k
        if n == 33:
            yield "any capacity", lanes, random, np.zeros_like(dist), dem, min(2**31 - 1, n * (32767 if wide else 255))
    for n in (31, 32, 33, 63, 64, 65, 100):  # potentials that only grow: nothing is ever removed
        dist = np.full((n + 1, n + 1), 500)
        for j in range(1, n):
            dist[j, j + 1] = 300 - 2 * j
        one = np.full((64, n), 3 * k)
        one[7] = k  # in one scenario a vehicle takes the whole tour
        yield "all kept", 64, 1 + np.arange(n), dist, one, n * k
    rng = np.random.default_rng(200)  # as long as the chip's tiles, vehicles of 24 stops
    n = 200
    xy = rng.integers(0, 1001, size=(n + 1, 2))
    dist = np.rint(np.hypot(*(xy[:, None] - xy[None]).transpose(2, 0, 1))).astype(np.int64)
    yield "random, n = 200", 64, 1 + rng.permutation(n), dist, rng.integers(1, 21, size=(64, n)) * k, 250 * k


def _tables(tour, dist):
    """c_j (0 at n), f_0, b_j of the potential form."""
    n = tour.size
    arc = np.array([0] + [dist[tour[j - 1], tour[j]] for j in range(1, n)]).cumsum()
    a = dist[0, tour] - arc
    b = arc + dist[tour, 0]
    c = np.append(b[:-1] + a[1:], 0)
    return c, int(a[0]), b


def _reference(dem, Q, c, f0):
    """m_j [n + 1, 64] by the definition, and the longest window in positions."""
    n = dem.shape[1]
    load = np.concatenate([np.zeros((64, 1), np.int64), dem.cumsum(1)], 1)
    f = np.full((64, n + 1), INF)
    f[:, 0] = f0
    m, longest = np.full((n + 1, 64), INF), 0
    for j in range(1, n + 1):
        fits = load[:, j : j + 1] - load[:, :j] <= Q
        longest = max(longest, int(fits.sum(1).max()))
        m[j] = np.where(fits, f[:, :j], INF).min(1)
        if j < n:
            f[:, j] = np.where(m[j] >= INF // 2, INF, m[j] + c[j - 1])
    return m, longest


def test_stack_code(variant):
    ring, src, out, code = variant
    wide = src == "LDS16"
    for label, lanes, tour, dist, dem, Q in _cases(wide):
        n = tour.size
        c, f0, b = _tables(tour, dist)
        m, longest = _reference(dem, Q, c, f0)
        tab = np.zeros((n + 4, 2), np.int32)  # three entries after position n, and no more
        tab[1 : n + 1, 0], tab[1 : n + 1, 1] = tour - 1, c
        rows = np.zeros((64, n), np.int64)
        rows[:, tour - 1] = dem
        lds = rows.astype(np.int16 if wide else np.uint8).tobytes()
        groups = (n - 1) // 4 + 3
        flat = np.zeros((64, 4 * groups), np.uint8)
        flat[:, :n] = dem.clip(0, 255)
        perm = np.ascontiguousarray(flat.view(np.uint32).T).reshape(-1)
        table = np.full((n, 64), -7, np.int32)
        ab = np.stack([np.zeros(n, np.int32), b.astype(np.int32)], 1)
        w = M.Wave(code, lanes, lds, tab, ab if out == "VALUES" else None, perm, table[: max(n - 1, 0)])
        for name, val in (("tab", M.TAB), ("n", n), ("f0", f0 & 0xFFFFFFFF), ("Q", Q), ("base", M.PERM & 0xFFFFFFFF),
                          ("baseh", M.PERM >> 32), ("out", M.OUT & 0xFFFFFFFF), ("outh", M.OUT >> 32), ("step", 256), ("steph", 0),
                          ("ab", M.AB - 20)):
            w.ws(M.OPERANDS[name], val)
        lane = np.arange(64, dtype=np.uint32)
        for name, val in (("row", 4 * lane if src == "STREAM" else lane * np.uint32(n * (2 if wide else 1))), ("col", 4 * lane)):
            i = int(M.OPERANDS[name][1:])
            w.v[i], w.vdef[i] = val, True
        where = "%s, n = %d, %d lanes, Q = %d" % (label, n, lanes, Q)
        try:
            w.run(400 + n * (100 + 8 * min(longest, ring)))
        except M.Fault as e:
            raise AssertionError("%s: %s" % (where, e))
        assert w.exec == (1 << lanes) - 1, where
        on = slice(0, lanes)
        over = w.v[1][on] != 0
        if longest < ring:
            assert not over.any(), where
        if label == "all kept":
            assert over.any() == (n >= ring), where
        if over.any():  # the caller recomputes the tile
            continue
        got, want = w.v[0][on].view(np.int32).astype(np.int64), m[n][on]
        split = want < INF // 2
        assert np.array_equal(got[split], want[split]) and (got[~split] >= INF // 2).all(), where
        if out == "VALUES":
            assert (table[n - 1] == -7).all() and (table[:, lanes:] == -7).all(), where
            for j in range(1, n):
                ok = m[j][on] < INF // 2
                assert np.array_equal(table[j - 1][on][ok], (m[j] + b[j - 1])[on][ok]), (where, j)
                assert (table[j - 1][on][~ok] >= INF).all(), (where, j)
