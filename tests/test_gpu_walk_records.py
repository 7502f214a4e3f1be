"""Walks over near records (at most six neighbours, at most eight diagonals per matrix), and
walks handed over to single-walk waves: every record bit for bit the oracle's, at the edges
where the record format changes and on walks long enough to be handed over."""
import numpy as np
import pytest

import oracle as O
from paper_math_0609672_amd import workloads as W
from test_gpu_parity import DEV, compare_walks, np_, srw, torch  # noqa: F401

pytestmark = pytest.mark.gpu


def banded(n, offsets, seed, ground_frac=0.02):
    """Edges i .. i + d for every offset d, each kept with probability 0.9 (0.2 past the
    third), at most six per node, on top of a path."""
    rng = np.random.default_rng(seed)
    eu, ev = [np.arange(n - 1)], [np.arange(1, n)]
    deg = np.full(n, 2)
    for k, d in enumerate(offsets):
        for i in np.flatnonzero(rng.random(n - d) < (0.9 if k < 2 else 0.2)):
            if deg[i] < 6 and deg[i + d] < 6:
                deg[i] += 1
                deg[i + d] += 1
                eu.append([i])
                ev.append([i + d])
    eu, ev = np.concatenate(eu), np.concatenate(ev)
    exc = np.zeros(n)
    at = rng.choice(n, max(1, int(ground_frac * n)), replace=False)
    exc[at] = rng.uniform(0.1, 1.0, at.size)
    return W.assemble(n, eu, ev, rng.uniform(0.1, 10.0, eu.size), exc)


# one diagonal pair fewer than, as many as and one more than a near record's list holds;
# a node of seven neighbours; two nodes; a thin 3D grid
EDGES = {
    "six_diagonals": banded(3001, (7, 40), 1),
    "eight_diagonals": banded(3001, (7, 40, 333), 2),
    "ten_diagonals": banded(3001, (7, 40, 333, 1500), 3),
    "two_nodes": W.from_dense(np.array([[2.0, -1.0], [-1.0, 1.5]])),
    "star_of_seven": W.assemble(2000, np.concatenate([np.arange(1999), np.full(5, 1000)]),
                                np.concatenate([np.arange(1, 2000), 1000 + np.arange(2, 7)]),
                                np.ones(2004), np.where(np.arange(2000) % 97 == 77, 0.5, 0.0)),
    "wide_band": W.grid((7, 3, 61), ground_frac=0.01, seed=4),
}


@pytest.mark.parametrize("name", list(EDGES))
def test_record_formats_bit_exact(srw, name):  # noqa: F811
    compare_walks(srw, EDGES[name], 70, 9)


# one weakly grounded node: the walks of the lowest ranks run for tens of thousands of
# steps, so they are handed over from bulk waves (near, line and bucketed records)
def weak(eu, ev, n, g):
    exc = np.zeros(n)
    exc[n // 3] = 2.0 * g.sum() / 2e4  # a walk that ends at ground only takes about 2e4 steps
    return W.assemble(n, eu, ev, g, exc)


def long_walks(kind):
    rng = np.random.default_rng(5)
    if kind == "grid":
        eu, ev = W.grid_edges((40, 37))
        return weak(eu, ev, 40 * 37, rng.uniform(0.5, 1.5, eu.size))
    A = W.random_graph(1500, 1800 if kind == "sparse" else 9000, seed=8)  # degrees to 7 and to 25
    r = np.repeat(np.arange(A.n), np.diff(A.rowptr))
    up = r < A.col
    return weak(r[up], A.col[up].astype(np.int64), A.n, -A.val[up])


@pytest.mark.parametrize("kind", ["grid", "sparse", "wide"])
@pytest.mark.parametrize("walk_waves", [0, 4, 12])
def test_handed_over_walks_bit_exact(srw, kind, walk_waves):  # noqa: F811
    F, t = compare_walks(srw, long_walks(kind), 24, 3, walk_waves=walk_waves)
    assert int(F.records()["length"].max()) > 5000  # far past the age at which walks move


@pytest.mark.parametrize("kind", ["grid", "wide"])
def test_step_cap_of_handed_over_walks(srw, kind):  # noqa: F811
    """A cap equal to the longest walk passes; one step less fails the build."""
    A = long_walks(kind)
    M = srw.Matrix.from_host(A, DEV)
    F = srw.build_factor(M, 24, 0.0, 3, keep=2)
    longest = int(F.records()["length"].max())
    full = np_(F.export()["yval"])
    F = srw.build_factor(M, 24, 0.0, 3, max_steps=longest)
    assert np.array_equal(np_(F.export()["yval"]), full)
    with pytest.raises(srw.SrwError) as e:
        srw.build_factor(M, 24, 0.0, 3, max_steps=longest - 1)
    assert e.value.status == srw.E_WALK_LIMIT


@pytest.mark.parametrize("count", [3, 256, 257])  # near records up to 256 matrices
def test_batches_at_the_list_limit(srw, count):  # noqa: F811
    mats = [W.grid((3 + i % 5, 4 + i % 3), seed=i, ground_frac=0.1) for i in range(count)]
    F = srw.build_factor_batched([srw.Matrix.from_host(A, DEV) for A in mats], 20, 0.0, list(range(count)))
    got = {k: np_(v) for k, v in F.export().items()}
    off = 0
    for i, A in enumerate(mats):
        ref = O.build_factor(A, 20, 0.0, i)
        a, b = got["yptr"][off], got["yptr"][off + A.n]
        assert np.array_equal(got["ycol"][a:b] - off, ref.ycol)
        assert np.array_equal(got["yval"][a:b], ref.yval)
        off += A.n
