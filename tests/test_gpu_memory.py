"""Device memory kept between calls: results do not depend on what earlier calls left in it,
several threads share it, and it stays bounded."""
import os
import subprocess
import sys
import threading

import numpy as np
import pytest

from paper_math_0609672_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def srw():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_math_0609672_amd import srw as s
    return s


DEV = "cuda:0"


def solve(srw, A, seed, b, stream=None):
    M = srw.Matrix.from_host(A, DEV)
    F = srw.build_factor(M, 24, 1e-3, seed, stream=stream)
    st, x, it, _ = srw.pcg_solve(M, F, b, 1e-8, stream=stream)
    F.free()
    assert st == srw.OK
    return x.cpu().numpy()


def test_sizes_in_turn_give_the_same_results(srw):
    """Growing and shrinking sizes reuse one another's blocks; every repeat is bitwise equal."""
    mats = [W.grid((k, k + 3), seed=k) for k in (5, 64, 17, 90, 33)]
    bs = [torch.from_numpy(W.rhs(A.n, seed=i)).to(DEV) for i, A in enumerate(mats)]
    first = [solve(srw, A, i, b) for i, (A, b) in enumerate(zip(mats, bs))]
    for _ in range(3):
        for i in (3, 0, 4, 2, 1):
            assert np.array_equal(solve(srw, mats[i], i, bs[i]), first[i])


def test_threads_and_streams_share_the_blocks(srw):
    mats = [W.grid((20 + 9 * k, 31), seed=k) for k in range(4)]
    bs = [torch.from_numpy(W.rhs(A.n, seed=i)).to(DEV) for i, A in enumerate(mats)]
    want = [solve(srw, A, i, b) for i, (A, b) in enumerate(zip(mats, bs))]
    torch.cuda.synchronize()
    bad = []

    def work(i):
        try:
            s = torch.cuda.Stream(device=DEV)
            with torch.cuda.stream(s):
                for _ in range(6):
                    if not np.array_equal(solve(srw, mats[i], i, bs[i], stream=s), want[i]):
                        bad.append(i)
        except Exception as e:  # noqa: BLE001
            bad.append(e)

    ts = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad


def test_repeated_builds_do_not_grow(srw):
    A = W.grid((60, 60), seed=2)
    b = torch.from_numpy(W.rhs(A.n, seed=2)).to(DEV)
    for i in range(3):
        solve(srw, A, i, b)
    torch.cuda.synchronize()
    free0, _ = torch.cuda.mem_get_info()
    for i in range(40):  # seeds give factors of slightly different sizes
        solve(srw, A, i, b)
    torch.cuda.synchronize()
    free1, _ = torch.cuda.mem_get_info()
    assert free0 - free1 < 256 << 20


FEATURES_DURING_CAPTURE = """
import os, threading, torch
from paper_math_0609672_amd import srw, workloads as W
A = W.grid((90, 70), seed=1)
M = srw.Matrix.from_host(A, "cuda:0")
rank = torch.randperm(A.n, device="cuda:0").int()
one, out, got = torch.ones(1000, device="cuda:0"), torch.zeros(1000, device="cuda:0"), []
torch.cuda.synchronize()
g = torch.cuda.CUDAGraph()
with torch.cuda.graph(g, capture_error_mode="global"):
    out.copy_(one * 2)
    t = threading.Thread(target=lambda: got.append(srw.row_features(M, rank)))
    t.start()
    t.join()
    out.add_(1)
for k in range(3):
    out.zero_()
    g.replay()
    torch.cuda.synchronize()
    assert bool((out == 3).all())
    assert torch.equal(got[0], srw.row_features(M, rank))
print("done", flush=True)
os._exit(0)
"""


def test_a_call_while_another_thread_captures(srw):
    """The first call of a process, whose workspace is new memory, in one thread while another
    captures a graph in torch's default mode: both succeed.  (A process of its own has no kept
    blocks.  The call makes no cooperative launch: the runtime refused one in a child of a
    process that had made some.)"""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", FEATURES_DURING_CAPTURE], capture_output=True, text=True, cwd=root,
                       timeout=100)
    assert r.returncode == 0 and r.stdout.split()[-1:] == ["done"], r.stderr[-2000:]


def test_repeated_large_builds_do_not_grow(srw):
    """24 builds of tens of megabytes each, of slightly different sizes: one factor more than
    after the first four at most (a block of another size class here and there)."""
    A = W.grid((400, 400), seed=2)
    M = srw.Matrix.from_host(A, DEV)

    def build(seed):
        F = srw.build_factor(M, 24, 0.0, seed)
        size = 24 * F.stats()["nnz_y"] + 32 * A.n  # entries of Y by rows and by columns, row data
        F.free()
        return size

    size = max(build(i) for i in range(4))
    assert size > 20 << 20
    torch.cuda.synchronize()
    free0, _ = torch.cuda.mem_get_info()
    for i in range(4, 28):
        build(i)
    torch.cuda.synchronize()
    free1, _ = torch.cuda.mem_get_info()
    assert free0 - free1 <= size
