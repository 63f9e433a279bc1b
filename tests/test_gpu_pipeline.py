"""The pipelined rollout at the sizes where its LDS rings can go wrong, against
the FP64 oracle through the C ABI: horizons around multiples of the ring sizes
(4 and 8 steps; the drawing waves take every third or fourth step), a ragged
last tile, three objectives, both precisions, with and without drag, a cold
and a warm solve each; and rings of 4 steps (more tiles than CUs) against
rings of 8 (one tile per CU)."""
import sys

import numpy as np
import pytest

from paper_2509_14726_amd import mppi as M
from paper_2509_14726_amd import synth
from tests.parity import build_pair, solve_and_compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [M.FP64, M.FP32], ids=["fp64", "fp32"])
@pytest.mark.parametrize("objective", ["gate", "contour", "track"])
@pytest.mark.parametrize("N", [1, 2, 3, 4, 5, 7, 8, 9, 12, 15, 16, 17])
def test_horizons_around_the_rings(N, objective, precision):
    _check(130, N, objective, precision, drag=N % 2 == 1)


@pytest.mark.parametrize("objective", ["gate", "contour", "track"])
@pytest.mark.parametrize("N", [1, 4, 5, 9, 31])
def test_ring_sizes_give_the_same_bits(N, objective):
    """A cold solve's cost of sample m does not depend on the sample count:
    with more tiles than CUs (rings of 4 steps, two workgroups per CU) the
    first samples cost the same, bit for bit, as in a small solve (rings of 8
    steps, which the test above holds against the oracle)."""
    import torch
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    print("[gpu-case] ring sizes", objective, "N", N, flush=True)
    sys.stdout.flush()
    J = []
    for K in (130, 64 * n_cu + 70):
        w = synth.single_solve_workload(K=K, N=N, objective=objective, seed=77 + N, track_seed=3)
        sv = M.Solver(w["quad"], w["params"], gates=w["gates"], path=w.get("path"), path_len=w.get("path_len", 0.0),
                      xref=w.get("xref"), ref_dt=w.get("ref_dt", 0.0))
        sv.solve(w["x0"])
        J.append(sv.read_samples()[0])
        sv.close()
    assert np.array_equal(J[0], J[1][:130])


@pytest.mark.parametrize("precision", [M.FP32, M.FP64], ids=["fp32", "fp64"])
@pytest.mark.parametrize("objective", ["gate", "contour", "track"])
@pytest.mark.parametrize("N", [1, 2, 3, 4, 7, 8, 9, 16, 17, 40])
def test_rate_input_pipeline_equals_one_wave(N, objective, precision, monkeypatch):
    """The rate input's pipelined rollout against its one-wave rollout (which
    other tests hold against the oracle): costs, clipped samples, solution and
    handed-on speed bit for bit over three warm solves, horizons around the
    ring sizes, a ragged last tile, with and without drag."""
    print("[gpu-case] rate pipeline", objective, "N", N, "fp64" if precision == M.FP64 else "fp32", flush=True)
    sys.stdout.flush()
    w = synth.single_solve_workload(K=200, N=N, objective=objective, seed=31 + N, track_seed=4, sigma=(8.0,) * 4,
                                    sigma_v=5.0, input_model=M.INPUT_RATE, rate_lim=(-10.0, 10.0),
                                    dv_lim=(-20.0, 20.0), **{"lambda": 20.0})
    if N % 2:
        w["quad"] = dict(w["quad"], drag=(0.3, 0.3, 0.15))
    x0 = np.concatenate([w["x0"], np.full(4, synth.hover_thrust())])
    out = []
    for waves in (None, "1"):
        if waves:
            monkeypatch.setenv("MPPI_ROLLOUT_WAVES", waves)
        else:
            monkeypatch.delenv("MPPI_ROLLOUT_WAVES", raising=False)
        sv = M.Solver(w["quad"], w["params"], gates=w["gates"], path=w.get("path"), path_len=w.get("path_len", 0.0),
                      xref=w.get("xref"), ref_dt=w.get("ref_dt", 0.0), precision=precision)
        x, got = x0.copy(), []
        for step in range(3):
            u0, U, info = sv.solve(x, step * 0.02)
            J, Us = sv.read_samples(want_U=True)
            wd = sv.get_warm()
            got.append((u0, U, J, Us, info["J_min"], info["S"], info["J_nom"], info["rollout_waves"], np.array(wd.V),
                        np.array(wd.allow), wd.vtheta, wd.theta0))
            x = M.plant_step_rate(w["quad"], x, u0, 0.02, 2)
        out.append(got)
        sv.close()
    for a, b in zip(*out):
        for xa, xb in zip(a, b):
            np.testing.assert_array_equal(xa, xb)


def _check(K, N, objective, precision, drag):
    print("[gpu-case] pipeline", objective, "K", K, "N", N, "fp64" if precision == M.FP64 else "fp32", flush=True)
    sys.stdout.flush()
    w = synth.single_solve_workload(K=K, N=N, objective=objective, seed=77 + N, track_seed=3, **{"lambda": 20.0})
    if drag:
        w["quad"] = dict(w["quad"], drag=(0.3, 0.3, 0.15))
    dev, orc = build_pair(w, precision)
    for t in (0.0, 0.02):
        st = solve_and_compare(dev, orc, w["x0"], t, precision)
        assert st["info"]["rollout_waves"] == 4
    dev.close()
