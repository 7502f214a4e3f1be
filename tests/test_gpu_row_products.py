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
