"""The triangular solves past the dense head in two launches (a wave per row over the chain,
16, 32 or 64 lanes per row over the rest, by the factor's mean row length), against the oracle,
at the smallest size that takes two launches, and where the chain rows are solved by blocks
with the blocks' inverses: 131,072 rows or more past the head, blocks deep enough."""
import numpy as np
import pytest

import oracle as O
from paper_math_0609672_amd import workloads as W
from test_gpu_parity import DEV, np_, srw, torch  # noqa: F401

pytestmark = pytest.mark.gpu

# mean row length below 28, between 28 and 56, above 56 (ragged sizes: odd, no multiple of
# 16, 64 or 256); then one row fewer than, and as many as, two launches need
CASES = {
    "short_rows": ((53, 51, 52), 64, 1e-2, (0, 28)),
    "middle_rows": ((53, 51, 52), 256, 1e-4, (28, 56)),
    "long_rows": ((53, 51, 52), 1024, 0.0, (56, 1e9)),
    "one_launch": ((135167,), 16, 1e-3, (0, 28)),
    "two_launches": ((135168,), 16, 1e-3, (0, 28)),
}


@pytest.mark.parametrize("name", list(CASES))
def test_apply_matches_oracle(srw, name):  # noqa: F811
    """1e-12 in FP64 and 1e-5 with the FP32 factor, as for every other factor: sums in
    another order of rows of at most a few hundred entries whose absolute sum is at most 1."""
    dims, walks, drop, (lo, hi) = CASES[name]
    A = W.grid(dims, ground_frac=0.02, seed=3)
    ref = O.build_factor(A, walks, drop, 7, threads=8)
    assert lo * A.n <= ref.ycol.size <= hi * A.n
    M = srw.Matrix.from_host(A, DEV)
    r = W.rhs(A.n, seed=5)
    z = O.apply(ref, r)
    for precision, tol in (("fp64", 1e-12), ("fp32", 1e-5)):
        F = srw.build_factor(M, walks, drop, 7, precision=precision)
        for _ in range(2):
            got = np_(srw.apply(F, torch.as_tensor(r, device=DEV)))
            assert np.linalg.norm(got - z) <= tol * np.linalg.norm(z), precision
        F.free()


# the chain plan over the last row, on matrices of no geometry (whose blocks have to be made
# smaller with longer rows), and on long chains (few grounded nodes)
PLANS = {
    "plan_takes_all_rows": (W.grid((48, 64, 44), ground_frac=0.02, seed=3), 256, 1e-4),
    "random_graph": (W.random_graph(140000, 420000, seed=7, ground_frac=0.01), 64, 1e-3),
    "smaller_blocks": (W.random_graph(140000, 1120000, seed=7, ground_frac=0.01), 64, 1e-3),
    "long_chains": (W.grid((53, 51, 52), ground_frac=0.0005, seed=3), 256, 1e-4),
}


@pytest.mark.parametrize("name", list(PLANS))
def test_chain_plan_matches_oracle(srw, name):  # noqa: F811
    """The bound of every apply test (1e-12, 1e-5 with the FP32 factor); the application
    without allocations and a second factor of the same seed give the same bits."""
    A, walks, drop = PLANS[name]
    ref = O.build_factor(A, walks, drop, 7, threads=8)
    M = srw.Matrix.from_host(A, DEV)
    r = W.rhs(A.n, seed=5)
    rt = torch.as_tensor(r, device=DEV)
    z = O.apply(ref, r)
    for precision, tol in (("fp64", 1e-12), ("fp32", 1e-5)):
        F = srw.build_factor(M, walks, drop, 7, precision=precision)
        G = srw.build_factor(M, walks, drop, 7, precision=precision)
        got = np_(srw.apply(F, rt))
        assert np.linalg.norm(got - z) <= tol * np.linalg.norm(z), precision
        assert np.array_equal(np_(srw.apply_noalloc(F, rt)), got)
        assert np.array_equal(np_(srw.apply(G, rt)), got)
        F.free()
        G.free()


def test_chain_plan_of_two_games(srw):  # noqa: F811
    """The plans of the two games' factors (no dense head), preconditioning BiCGSTAB: the
    oracle's first iterates to 1e-10, as in the tests of smaller sizes."""
    A = W.grid_asym((53, 51, 52), ground_frac=0.0005, seed=3)
    ref = O.build_factor_ldu(A, 64, 1e-3, 7)
    M = srw.Matrix.from_host(A, DEV)
    F = srw.build_factor_ldu(M, 64, 1e-3, 7)
    b = W.rhs(A.n, seed=5)
    for k in (1, 2):
        _, x, _, _ = srw.bicgstab_solve(M, F, torch.as_tensor(b, device=DEV), 0.0, k)
        _, rx, _, _ = O.bicgstab(A, ref, b, 0.0, k)
        assert np.linalg.norm(np_(x) - rx) <= 1e-10 * np.linalg.norm(rx)
    F.free()


# orders that are not the library's random one: one launch over all rows, lanes by row length
@pytest.mark.parametrize("walks,drop,lo,hi", [(16, 1e-2, 0, 28), (64, 1e-3, 28, 56), (1024, 0.0, 56, 1e9)])
@pytest.mark.parametrize("precision,tol", [("fp64", 1e-12), ("fp32", 1e-5)])
def test_natural_order_matches_oracle(srw, walks, drop, lo, hi, precision, tol):  # noqa: F811
    """Chains through all rows, without and behind a dense head: the bound of every apply test."""
    A = W.grid((17, 19, 21), ground_frac=0.005, seed=3)
    ref = O.build_factor(A, walks, drop, 7, rk=np.arange(A.n, dtype=np.int32), threads=8)
    assert lo * A.n < ref.ycol.size <= hi * A.n
    r = W.rhs(A.n, seed=5)
    z = O.apply(ref, r)
    M = srw.Matrix.from_host(A, DEV)
    for head in (-1, 512, 0):
        F = srw.build_factor(M, walks, drop, 7, rank="natural", precision=precision, head_rows=head)
        got = np_(srw.apply(F, torch.as_tensor(r, device=DEV)))
        assert np.linalg.norm(got - z) <= tol * np.linalg.norm(z), head
        F.free()


@pytest.mark.parametrize("order", ["natural", "given"])
def test_two_games_in_given_orders(srw, order):  # noqa: F811
    """As many rows as the random order's plan is tried for: no plan, the oracle's iterates."""
    A = W.grid_asym((53, 51, 52), ground_frac=0.05, seed=3)
    rk = np.arange(A.n, dtype=np.int32)
    if order == "given":
        rk = np.random.default_rng(2).permutation(rk).astype(np.int32)
    ref = O.build_factor_ldu(A, 16, 1e-2, 7, rk=rk)
    M = srw.Matrix.from_host(A, DEV)
    F = srw.build_factor_ldu(M, 16, 1e-2, 7, rank="natural" if order == "natural" else torch.as_tensor(rk, device=DEV))
    b = W.rhs(A.n, seed=5)
    for k in (1, 2):
        _, x, _, _ = srw.bicgstab_solve(M, F, torch.as_tensor(b, device=DEV), 0.0, k)
        _, rx, _, _ = O.bicgstab(A, ref, b, 0.0, k)
        assert np.linalg.norm(np_(x) - rx) <= 1e-10 * np.linalg.norm(rx)
    F.free()


@pytest.mark.parametrize("walks", [64, 256])
def test_two_games_on_either_side_of_the_plan(srw, walks):  # noqa: F811
    """Chain rows of 8.8 entries (one launch) and of 18.7 (the plan): the oracle's iterates."""
    A = W.grid_asym((53, 51, 52), ground_frac=0.0005, seed=3)
    ref = O.build_factor_ldu(A, walks, 1e-3, 7, threads=8)
    M = srw.Matrix.from_host(A, DEV)
    b = W.rhs(A.n, seed=5)
    F = srw.build_factor_ldu(M, walks, 1e-3, 7)
    for k in (1, 2):
        _, x, _, _ = srw.bicgstab_solve(M, F, torch.as_tensor(b, device=DEV), 0.0, k)
        _, rx, _, _ = O.bicgstab(A, ref, b, 0.0, k)
        assert np.linalg.norm(np_(x) - rx) <= 1e-10 * np.linalg.norm(rx)
    F.free()


def substitute(ref, r, dtype):
    """Y^T w = r, Y z = D^-1 w row by row in the given type, the factor's values in FP32."""
    order = np.argsort(ref.rank)
    nnz = np.arange(ref.ycol.size, dtype=np.int64)
    val, d = ref.yval.astype(np.float32), ref.d.astype(np.float32).astype(dtype)
    at = np.argsort(ref.ycol, kind="stable")
    tptr = np.concatenate([[0], np.cumsum(np.bincount(ref.ycol, minlength=ref.n))])
    trow = np.searchsorted(ref.yptr, nnz[at], side="right") - 1
    val, tval = val.astype(dtype), val[at].astype(dtype)
    w, z, r = np.zeros(ref.n, dtype), np.zeros(ref.n, dtype), r.astype(dtype)
    for i in order[::-1]:
        p = slice(tptr[i], tptr[i + 1])
        w[i] = r[i] - np.dot(tval[p], w[trow[p]])
    for i in order:
        p = slice(ref.yptr[i], ref.yptr[i + 1])
        z[i] = w[i] / d[i] - np.dot(val[p], z[ref.ycol[p]])
    return z


def test_plan_of_fp32_factors_loses_nothing(srw):  # noqa: F811
    """The plan's rows are rounded to FP32 as often again as a substitution's.  Their sums in
    64 bits make up for that: over four solves the mean error against 64 bits is no larger
    than that of a substitution in FP32, but for half of it as room for the few solves."""
    A, walks, drop = PLANS["long_chains"]
    M = srw.Matrix.from_host(A, DEV)
    here, plain = [], []
    for seed in (7, 8):
        ref = O.build_factor(A, walks, drop, seed, threads=8)
        F = srw.build_factor(M, walks, drop, seed, precision="fp32")
        for k in range(2):
            r = W.rhs(A.n, seed=10 * seed + k)
            exact = substitute(ref, r, np.float64)
            got = np_(srw.apply(F, torch.as_tensor(r, device=DEV)))
            size = np.linalg.norm(exact)
            here.append(np.linalg.norm(got - exact) / size)
            plain.append(np.linalg.norm(substitute(ref, r, np.float32) - exact) / size)
        F.free()
    print("mean errors", np.mean(here), np.mean(plain))
    assert np.mean(here) <= 1.5 * np.mean(plain)
