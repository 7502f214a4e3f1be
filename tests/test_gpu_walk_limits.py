"""The walk kernel at the limits of its record formats and of its queues: every walk is the
oracle's, bit for bit, on either side of a limit."""
import threading

import numpy as np
import pytest

import oracle as O
from paper_math_0609672_amd import workloads as W
from test_gpu_parity import DEV, compare_walks, np_, srw, torch  # noqa: F401

pytestmark = pytest.mark.gpu


def factor_bit_exact(srw, A, walks, seed, **kw):  # noqa: F811
    F = srw.build_factor(srw.Matrix.from_host(A, DEV), walks, 0.0, seed, **kw)
    got = {k: np_(v) for k, v in F.export().items()}
    ref = O.build_factor(A, walks, 0.0, seed)
    for k in ("rank", "yptr", "ycol", "yval", "d"):
        assert np.array_equal(got[k], getattr(ref, k)), k
    return F


def wide_circulant(n):
    """Node v joined to v +- 1 .. 12: twelve neighbours of little weight between twelve of
    much, half of every diagonal excess (walks end soon).  Four or five of the light ones
    meet one of the 64 equal draw ranges, eight one of 32: a record has 64 bucket lines, its
    first line and three more."""
    off = np.concatenate([np.arange(-12, 0), [0], np.arange(1, 13)])
    w = np.where(off == 0, 1.0, np.where(abs(off) <= 6, -0.004, -0.0375))
    col = (np.arange(n, dtype=np.int32)[:, None] + off.astype(np.int32)) % n
    val = np.broadcast_to(w, col.shape).copy()
    for v in list(range(12)) + list(range(n - 12, n)):  # rows that wrap round
        o = np.argsort(col[v])
        col[v], val[v] = col[v][o], val[v][o]
    return W.CSR(n, np.arange(n + 1, dtype=np.int64) * 25, col.reshape(-1), val.reshape(-1))


def record_lines(A, v):
    """Lines of node v's record: with k in 3..6 the first for which each of 2^k equal draw
    ranges meets at most six entries, 2^k bucket lines; the first line; eight entries a line."""
    p = slice(A.rowptr[v], A.rowptr[v + 1])
    off = A.col[p] != v
    c = np.cumsum(-A.val[p][off]) / A.val[p][~off][0]
    deg = int(off.sum())
    if deg <= 6:
        return 1
    lo = np.concatenate([[0.0], c[:-1]])
    for k in range(3, 7) if deg <= 64 else ():
        first = np.arange(2 ** k)[:, None] / 2 ** k
        if ((lo < first + 0.5 ** k) & (c > first)).sum(1).max() <= 6:
            return 2 ** k + 1 + (deg + 7) // 8
    return 1 + (deg + 7) // 8


# 68 lines a node: start records' lines, which follow the walk records', end below the 2^27
# lines that an entry's line word can name (900,000) or pass them (1,040,000)
@pytest.mark.parametrize("n", [900_000, 1_040_000])
def test_start_records_past_the_line_mask(srw, n):  # noqa: F811
    A = wide_circulant(n)
    assert record_lines(A, n // 2) == 68
    assert (2 * 68 * n > 2 ** 27) == (n > 1_000_000) and 68 * n < 2 ** 27
    factor_bit_exact(srw, A, 2, 3)


def chorded_path(n, hub):
    """A path whose nodes are joined in random pairs (narrow records on many diagonals); with
    hub, node 5 is joined to six more (a record with bucket lines)."""
    rng = np.random.default_rng(n)
    p = rng.permutation(np.arange(20, n))
    p = np.sort(p[: p.size // 2 * 2].reshape(-1, 2), axis=1)
    p = p[p[:, 1] > p[:, 0] + 1]
    far = n - 10 * np.arange(1, 7) if hub else np.zeros(0, np.int64)
    eu = np.concatenate([np.arange(n - 1), p[:, 0], np.full(far.size, 5)])
    ev = np.concatenate([np.arange(1, n), p[:, 1], far])
    exc = np.where(np.arange(n) % 40 == 0, 0.5, 0.0)
    return W.assemble(n, eu, ev, np.ones(eu.size), exc)


# 1,280 lines are 160 KiB with their start records: all of a workgroup's LDS, of which the
# kernel needs a little for itself
@pytest.mark.parametrize("lines", [1279, 1280, 1281])
@pytest.mark.parametrize("kind", ["near", "lines", "buckets"])
def test_tables_at_the_size_of_the_lds(srw, kind, lines):  # noqa: F811
    if kind == "near":
        A = W.grid((lines,), ground_frac=0.05, seed=2)
    else:
        hub = kind == "buckets"
        A = chorded_path(lines - 9 if hub else lines, hub)
        assert record_lines(A, 5) == (10 if hub else 1)
        assert np.unique(A.col - np.repeat(np.arange(A.n), np.diff(A.rowptr))).size > 9
    assert sum(record_lines(A, v) for v in range(A.n)) == lines
    F = factor_bit_exact(srw, A, 40, 7)
    assert F.stats()["walk_lds"] == (lines <= (1280 if kind == "near" else 1279))


@pytest.mark.parametrize("walk_waves", [0, 24, 64])
def test_as_many_bulk_waves_as_the_chip_holds(srw, walk_waves):  # noqa: F811
    """20,000 chunks: from 24 waves to a CU on the first workgroups alone fill the chip."""
    compare_walks(srw, W.grid((160, 125), ground_frac=0.01, seed=6), 24, 4, walk_waves=walk_waves)


def test_builds_at_once(srw):  # noqa: F811
    """Builds of several threads and streams share the chip; three of them hold a table of more
    than half a CU's LDS in every workgroup."""
    mats = [W.random_graph(900, 1100, seed=4), W.random_graph(90, 420, seed=2), W.grid((160, 125), seed=3),
            W.random_graph(1000, 1200, seed=4)]
    for i in (0, 1, 3):
        lines = sum(record_lines(mats[i], v) for v in range(mats[i].n))
        assert 640 < lines < 1280
    refs = [O.build_factor(A, 200, 0.0, i) for i, A in enumerate(mats)]
    bad = []

    def work(i):
        try:
            s = torch.cuda.Stream(device=DEV)
            with torch.cuda.stream(s):
                M = srw.Matrix.from_host(mats[i], DEV)
                for _ in range(8):
                    F = srw.build_factor(M, 200, 0.0, i, stream=s)
                    got = {k: np_(v) for k, v in F.export().items()}
                    if F.stats()["walk_lds"] != (i != 2):
                        bad.append((i, "walk_lds"))
                    for k in ("ycol", "yval", "d"):
                        if not np.array_equal(got[k], getattr(refs[i], k)):
                            bad.append((i, k))
                    F.free()
        except Exception as e:  # noqa: BLE001
            bad.append((i, e))

    ts = [threading.Thread(target=work, args=(i,)) for i in range(len(mats))]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad


@pytest.mark.parametrize("max_steps", [2 ** 32 - 256, 2 ** 32, 2 ** 64 - 1])
def test_step_caps_past_32_bits(srw, max_steps):  # noqa: F811
    """Walks of both kinds of wave under the largest caps."""
    factor_bit_exact(srw, W.grid((40, 37), ground_frac=0.001, seed=8), 24, 3, max_steps=max_steps)
