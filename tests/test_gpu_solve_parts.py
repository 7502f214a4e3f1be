"""The triangular solves past the dense head in two launches (a wave per row over the chain,
16, 32 or 64 lanes per row over the rest, by the factor's mean row length), against the oracle,
and at the smallest size that takes two launches."""
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
