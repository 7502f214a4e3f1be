"""Batched solves where a matrix has more reduction tiles than lanes add them at once, rows of
one, two, three and many rounds of eight entries, and systems that stop long before others."""
import numpy as np
import pytest

import oracle as O
from paper_math_0609672_amd import workloads as W
from test_gpu_parity import DEV, np_, srw, torch  # noqa: F401
from test_gpu_row_products import hub

pytestmark = pytest.mark.gpu

MATS = [
    W.from_dense(np.array([[2.0, -1.0], [-1.0, 1.5]])),       # stops after two steps
    W.grid((17 * 1024 + 3,), ground_frac=0.05, seed=2),       # eighteen tiles
    hub(1500, 700, 300),                                      # a row of 300 entries
    W.grid((23, 31, 11), ground_frac=0.02, seed=4),           # rows of two to six rounds
]


@pytest.mark.parametrize("nrhs", [1, 3, 8])
@pytest.mark.parametrize("use_graph", [False, True])
def test_batched_solve_matches_oracle(srw, nrhs, use_graph):  # noqa: F811
    """Solutions to 1e-8 of the right-hand side (the tolerance asked for) and, at the
    device's own iteration count, the oracle's iterate to 1e-10, as in the tests of
    other batches."""
    seeds = [11, 12, 13, 14]
    Ms = [srw.Matrix.from_host(A, DEV) for A in MATS]
    F = srw.build_factor_batched(Ms, 64, 1e-3, seeds)
    _, off = srw.batch_info(F)
    Bh = np.random.default_rng(nrhs).standard_normal((off[-1], nrhs))
    if nrhs > 1:
        Bh[off[3]:off[4], 1] = 0.0
    st, X, it, rel = srw.pcg_solve_batched(F, torch.as_tensor(Bh, device=DEV), 1e-8, 500, use_graph=use_graph)
    assert st == srw.OK
    Xh = np_(X)
    for i, A in enumerate(MATS):
        ref = O.build_factor(A, 64, 1e-3, seeds[i])
        for j in range(nrhs):
            b, x = Bh[off[i]:off[i + 1], j], Xh[off[i]:off[i + 1], j]
            if not np.any(b):
                assert it[i, j] == 0 and not np.any(x)
                continue
            assert np.linalg.norm(b - A.to_scipy() @ x) <= 1e-8 * np.linalg.norm(b)
            _, rx, _, _ = O.pcg(A, ref, b, 0.0, max_iter=int(it[i, j]))
            assert np.linalg.norm(x - rx) <= 1e-10 * np.linalg.norm(rx), (i, j)
    F.free()
