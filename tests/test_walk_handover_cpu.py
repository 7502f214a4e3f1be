"""The hand-over queue of the walk kernel, compiled for the host: every wave ends and every
walk is run once, whatever part of the workgroups the chip holds at once, in whatever order
they start, and also where waves leave at their wait limit."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("handover") / "handover")
    subprocess.run(["g++", "-O2", "-std=c++17", "-pthread", "-D__device__=", "-D__forceinline__=inline",
                    "-I", os.path.join(ROOT, "paper_math_0609672_amd", "csrc"),
                    os.path.join(ROOT, "tests", "native", "handover.cpp"), "-o", exe], check=True)

    def run(bulk, single, held, walks, slots, limit=0, order=0, seed=0, unasked=0, tail=False):
        args = [bulk, single, held, walks, slots, limit, order, seed, unasked]
        r = subprocess.run([exe] + [str(a) for a in args], capture_output=True, text=True,
                           check=True, timeout=60)
        return int(r.stderr) if tail else r.stdout.split()

    return run


@pytest.mark.parametrize("order", [0, 1])
@pytest.mark.parametrize("bulk,single,held", [(1, 0, 1), (6, 4, 10), (6, 4, 3), (12, 8, 4), (9, 3, 1)])
@pytest.mark.parametrize("walks,slots", [(3, 3), (400, 400), (400, 40)])
def test_every_wave_ends_and_every_walk_runs_once(model, order, bulk, single, held, walks, slots):
    for seed in range(10):
        assert model(bulk, single, held, walks, slots, order=order, seed=seed) == ["0", "0"], seed


@pytest.mark.parametrize("limit", [1, 20_000])  # ns: waves leave at once, or now and then
@pytest.mark.parametrize("bulk,single,held", [(6, 4, 10), (12, 8, 4)])
def test_waves_that_leave_lose_no_walk(model, limit, bulk, single, held):
    for seed in range(10):
        assert model(bulk, single, held, 2000, 2000, limit=limit, seed=seed) == ["0", "0"], seed


def test_a_wait_for_waves_not_started_would_stall(model):
    """What the rule is for: bulk waves that wait without asking hold the chip."""
    assert model(12, 8, 4, 400, 400, unasked=1)[-1] == "stalled"


@pytest.mark.parametrize("slots", [0, 1, 40])
def test_the_tail_stays_near_the_last_slot(model, slots):
    """However many walks find no slot: each wave asks once more at most."""
    assert model(6, 4, 10, 20_000, slots, tail=True) <= 6
