"""Row features from entry tiles in LDS (256 rows, 1,024 entries at a time): sizes around a
workgroup's rows, rows over several tiles, and an output that is not 16-byte aligned."""
import ctypes

import numpy as np
import pytest

import oracle as O
from oracle import budget as B
from paper_math_0609672_amd import workloads as W
from test_gpu_parity import DEV, np_, srw, torch  # noqa: F401
from test_gpu_row_products import CASES, DENSE

pytestmark = pytest.mark.gpu


# float32 of features computed in float64 by the same operations: one unit in the last place
@pytest.mark.parametrize("name", list(CASES))
def test_features_match_oracle(srw, name):  # noqa: F811
    A = CASES[name]
    M = srw.Matrix.from_host(A, DEV)
    rank = srw.ordering(A.n, 11, DEV)
    ref = B.features(A, O.rank(A.n, 11)).astype(np.float32)
    whole = torch.full((8 * A.n + 1,), float("nan"), dtype=torch.float32, device=DEV)
    odd = whole[1:]  # 4 bytes past an aligned address
    csr = M.c()
    st = srw._lib.srw_row_features(ctypes.byref(csr), rank.data_ptr(), odd.data_ptr(), None)
    torch.cuda.synchronize()
    assert st == 0
    for f in (np_(srw.row_features(M, rank)), np_(odd).reshape(A.n, 8)):
        assert np.all(np.abs(f - ref) <= np.spacing(np.abs(ref)))


# mean row lengths past 12, 48 and 128 entries: 64 and 16 rows to a workgroup, a thread per row
@pytest.mark.parametrize("name", ["middle_rows"] + list(DENSE))
def test_features_of_dense_rows_match_oracle(srw, name):  # noqa: F811
    A = DENSE[name] if name in DENSE else W.random_graph(1003, 10000, seed=5, ground_frac=0.2)
    M = srw.Matrix.from_host(A, DEV)
    f = np_(srw.row_features(M, srw.ordering(A.n, 11, DEV)))
    ref = B.features(A, O.rank(A.n, 11)).astype(np.float32)
    assert np.all(np.abs(f - ref) <= np.spacing(np.abs(ref)))
