"""The weighted average of a solve over several rounds of samples: reading the
sample tensor (all of it where enough samples weigh something, else only what
does) against drawing the samples again, which always skips, bit for bit; and
with all samples alive against the FP64 oracle.  Sample counts around the
rounds of 1024 threads, binary32 sums and (from 65536 samples) binary64 ones,
weights from sharp to flat."""
import sys

import numpy as np
import pytest

from paper_2509_14726_amd import mppi as M
from paper_2509_14726_amd import synth
from tests.parity import build_pair, solve_and_compare

pytestmark = pytest.mark.gpu

OBJECTIVES = ["gate", "contour", "track"]


def say(*a):
    print("[gpu-case] average rounds", *a, flush=True)
    sys.stdout.flush()


@pytest.mark.parametrize("K", [8193, 12325, 20480, 65536, 69701, 73728])
@pytest.mark.parametrize("objective", OBJECTIVES)
@pytest.mark.parametrize("lam", [0.5, 10.0, 100.0, 1e5])
def test_stored_equals_drawn_again(lam, objective, K, monkeypatch):
    monkeypatch.setenv("MPPI_ROLLOUT_WAVES", "4")
    say("stored and drawn again", objective, "K", K, "lambda", lam)
    w = synth.single_solve_workload(K=K, N=3, objective=objective, seed=41, track_seed=3, **{"lambda": lam})
    out = []
    for flags in (0, M.FLAG_REGEN_AVERAGE):
        sv = M.Solver(w["quad"], dict(w["params"], flags=flags), gates=w["gates"], path=w.get("path"),
                      path_len=w.get("path_len", 0.0), xref=w.get("xref"), ref_dt=w.get("ref_dt", 0.0))
        x, got = np.array(w["x0"]), []
        for step in range(2):
            u0, U, info = sv.solve(x, step * 0.02)
            assert info["regen_average"] == (1 if flags else 0)
            wd = sv.get_warm()
            got.append((u0, U, info["J_min"], info["S"], info["ess"], np.array(wd.U), np.array(wd.V)))
            x = M.plant_step(w["quad"], x, u0, 0.02, 2)
        sv.close()
        out.append(got)
    for a, b in zip(*out):
        for xa, xb in zip(a, b):
            np.testing.assert_array_equal(xa, xb)


@pytest.mark.parametrize("flags", [0, M.FLAG_REGEN_AVERAGE])
@pytest.mark.parametrize("objective", OBJECTIVES)
@pytest.mark.parametrize("K", [9001, 66001])
def test_all_samples_alive_against_the_oracle(K, objective, flags, monkeypatch):
    monkeypatch.setenv("MPPI_ROLLOUT_WAVES", "4")
    say("oracle", objective, "K", K, "flags", flags)
    w = synth.single_solve_workload(K=K, N=4, objective=objective, seed=42, track_seed=3, **{"lambda": 1e4})
    w["params"] = dict(w["params"], flags=flags)
    dev, orc = build_pair(w, M.FP32)
    for t in (0.0, 0.02):
        solve_and_compare(dev, orc, w["x0"], t, M.FP32)
    st, info = dev.read_info()
    assert info["ess"] > 0.5 * K and info["regen_average"] == (1 if flags else 0)
    dev.close()
