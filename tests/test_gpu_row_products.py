"""The solvers' products with the matrix, 256 rows and 2,048 entries at a time: rows that span
several such tiles, empty-handed last threads, and sizes around a workgroup's rows."""
import numpy as np
import pytest

import oracle as O
from paper_math_0609672_amd import workloads as W
from test_gpu_parity import DEV, np_, srw, torch  # noqa: F401

pytestmark = pytest.mark.gpu


def hub(n, at, fan):
    """A path with one node joined to `fan` others, every fifth node grounded."""
    rng = np.random.default_rng(n + fan)
    far = rng.choice(np.setdiff1d(np.arange(n), [at - 1, at, at + 1]), fan, replace=False)
    eu = np.concatenate([np.arange(n - 1), np.full(fan, at)])
    ev = np.concatenate([np.arange(1, n), far])
    return W.assemble(n, eu, ev, rng.uniform(0.5, 2.0, eu.size), np.where(np.arange(n) % 5 == 0, 1.0, 0.0))


CASES = {
    "two_rows": W.from_dense(np.array([[2.0, -1.0], [-1.0, 1.5]])),
    "255": W.grid((255,), ground_frac=0.1, seed=1),
    "256": W.grid((256,), ground_frac=0.1, seed=2),
    "257": W.grid((257,), ground_frac=0.1, seed=3),
    "tile_of_2048": hub(700, 100, 600),
    "row_past_one_tile": hub(2600, 513, 2200),
    "row_past_two_tiles": hub(9001, 9000 - 256, 4300),
}


# Sums in another order than the oracle's (the dots over rows) differ by about n * 2^-53 <=
# 1e-12 of their size; three steps on these conditioned systems keep 1e-10.
@pytest.mark.parametrize("name", list(CASES))
def test_iterates_match_oracle(srw, name):  # noqa: F811
    A = CASES[name]
    M = srw.Matrix.from_host(A, DEV)
    F, ref = srw.build_factor(M, 8, 0.0, 5), O.build_factor(A, 8, 0.0, 5)
    b = np.random.default_rng(1).standard_normal(A.n)
    bt = torch.as_tensor(b, device=DEV)
    for k in (1, min(3, A.n - 1)):
        _, x, _, rel = srw.pcg_solve(M, F, bt, 0.0, k)
        _, rx, _, rrel = O.pcg(A, ref, b, 0.0, k)
        assert np.abs(np_(x) - rx).max() <= 1e-10 * np.abs(rx).max()
    # (the third BiCGSTAB iterate of a hub's matrix is no measure: one ulp of b changes the
    # oracle's by 5e-9)
    _, x, _, _ = srw.bicgstab_solve(M, None, bt, 0.0, 1)
    _, rx, _, _ = O.bicgstab(A, None, b, 0.0, 1)
    assert np.abs(np_(x) - rx).max() <= 1e-10 * np.abs(rx).max()


# mean row lengths past 32 and past 128 entries: 64 and 16 rows to a workgroup
DENSE = {
    "64_rows_at_once": W.random_graph(1003, 24000, seed=5, ground_frac=0.2),
    "16_rows_at_once": W.random_graph(515, 40000, seed=6, ground_frac=0.2),
    "partial_last_group": W.random_graph(130, 8300, seed=7, ground_frac=0.2),
}


@pytest.mark.parametrize("name", list(DENSE))
def test_iterates_of_dense_rows_match_oracle(srw, name):  # noqa: F811
    """The bound of the test above."""
    A = DENSE[name]
    M = srw.Matrix.from_host(A, DEV)
    F, ref = srw.build_factor(M, 8, 0.0, 5), O.build_factor(A, 8, 0.0, 5)
    b = np.random.default_rng(1).standard_normal(A.n)
    bt = torch.as_tensor(b, device=DEV)
    for k in (1, 3):
        _, x, _, rel = srw.pcg_solve(M, F, bt, 0.0, k)
        _, rx, _, rrel = O.pcg(A, ref, b, 0.0, k)
        assert np.abs(np_(x) - rx).max() <= 1e-10 * np.abs(rx).max()
        assert abs(rel - rrel) <= 1e-10 * rrel
        _, x, _, _ = srw.bicgstab_solve(M, None, bt, 0.0, k)
        _, rx, _, _ = O.bicgstab(A, None, b, 0.0, k)
        assert np.abs(np_(x) - rx).max() <= 1e-10 * np.abs(rx).max()


@pytest.mark.parametrize("name", ["255", "256", "257"])
def test_third_bicgstab_iterate_matches_oracle(srw, name):  # noqa: F811
    """Where one ulp of b changes the oracle's own third iterate by less than 1e-12."""
    A = CASES[name]
    b = np.random.default_rng(1).standard_normal(A.n)
    _, x, _, _ = srw.bicgstab_solve(srw.Matrix.from_host(A, DEV), None, torch.as_tensor(b, device=DEV), 0.0, 3)
    _, rx, _, _ = O.bicgstab(A, None, b, 0.0, 3)
    assert np.abs(np_(x) - rx).max() <= 1e-10 * np.abs(rx).max()
