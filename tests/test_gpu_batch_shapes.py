"""Batched steps at the sizes where their launch shapes change, against the
same contexts solved alone (which other tests hold against the oracle): bit
for bit, since every layout keeps its arithmetic and its order of additions.

* horizons around the chunks of the weighted average (four steps for gate and
  tracking, three for contouring), sample counts of one, two, three and many
  rounds of its threads, sharp weights (most samples are skipped) and spread;
* a step with more tiles than two pipelines per CU, whose pipelined contexts
  run one-wave rollouts in the pipeline's arithmetic;
* a last tile that holds the nominal alone (K a multiple of 64);
* rate-input contexts, which draw their samples in the rollout.
"""
import sys

import numpy as np
import pytest

from paper_2509_14726_amd import mppi as M
from paper_2509_14726_amd import synth

pytestmark = pytest.mark.gpu

SHAPES = [(64, 1), (200, 2), (2048, 3), (2050, 4), (4096, 5), (4100, 6), (6200, 7), (1000, 8), (8192, 9), (64, 50)]


def solver_for(w, precision):
    return M.Solver(w["quad"], w["params"], gates=w["gates"], path=w.get("path"), path_len=w.get("path_len", 0.0),
                    xref=w.get("xref"), ref_dt=w.get("ref_dt", 0.0), precision=precision)


def workload(i, K, N, objective, rate, lam, **over):
    if rate:
        over.update(sigma=(8.0,) * 4, sigma_v=5.0, input_model=M.INPUT_RATE, rate_lim=(-10.0, 10.0), dv_lim=(-20.0, 20.0))
    w = synth.single_solve_workload(K=K, N=N, objective=objective, seed=300 + i, track_seed=300 + i, **{"lambda": lam}, **over)
    if i % 2:
        w["quad"] = dict(w["quad"], drag=(0.3, 0.3, 0.15))
    if rate:
        w["x0"] = np.concatenate([w["x0"], np.full(4, synth.hover_thrust())])
    return w


def outcome(sv, want_U=True):
    status, info = sv.read_info()
    J, Us = sv.read_samples(want_U=want_U)
    wd = sv.get_warm()
    return [status, info["J_min"], info["S"], info["J_nom"], info["ess"], J, Us if want_U else 0, np.array(wd.U),
            np.array(wd.V), np.array(wd.allow), wd.theta0, wd.vtheta]


def check_batch(ws, precision, waves, use_graph, what, want_U=True, **cfg):
    import torch
    solo = [solver_for(w, precision) for w in ws]
    bat = [solver_for(w, precision) for w in ws]
    B = M.Batch(bat, rollout_waves=waves, use_graph=use_graph, **cfg)
    reqs = torch.zeros((len(ws), M.REQ_DOUBLES), dtype=torch.float64, device="cuda")
    u0s = torch.zeros((len(ws), 4), dtype=torch.float64, device="cuda")
    xs = [np.array(w["x0"]) for w in ws]
    for step in range(3):
        for i, x in enumerate(xs):
            reqs[i, :13] = torch.from_numpy(x[:13])
            reqs[i, 13] = step * 0.02
            if len(x) > 13:
                reqs[i, M.REQ_THRUST:M.REQ_THRUST + 4] = torch.from_numpy(x[13:])
        torch.cuda.synchronize()
        B.solve_device(reqs.data_ptr(), u0s.data_ptr())
        torch.cuda.synchronize()
        got = u0s.cpu().numpy()
        for i, w in enumerate(ws):
            print("[gpu-case]", what, "step", step, "K", w["params"]["K"], "N", w["params"]["N"], flush=True)
            sys.stdout.flush()
            u0, _, _ = solo[i].solve(xs[i], step * 0.02)
            np.testing.assert_array_equal(got[i], u0)
            for a, b in zip(outcome(bat[i], want_U), outcome(solo[i], want_U)):
                np.testing.assert_array_equal(a, b)
            plant = M.plant_step_rate if len(xs[i]) > 13 else M.plant_step
            xs[i] = plant(w["quad"], xs[i], u0, 0.02, 2)
    B.close()
    for s in solo + bat:
        s.close()


@pytest.mark.parametrize("precision", [M.FP32, M.FP64], ids=["fp32", "fp64"])
@pytest.mark.parametrize("objective", ["gate", "contour", "track"])
@pytest.mark.parametrize("lam,waves", [(0.5, 4), (1e4, 1)])
def test_average_chunks(lam, waves, objective, precision, monkeypatch):
    monkeypatch.setenv("MPPI_ROLLOUT_WAVES", str(waves))
    ws = [workload(i, K, N, objective, False, lam, ctrl_cost=0.3 if i % 3 == 0 else 0.0) for i, (K, N) in enumerate(SHAPES)]
    check_batch(ws, precision, waves, waves == 4, "average %s lambda %g" % (objective, lam))


@pytest.mark.parametrize("use_graph,regen,n_iter", [(True, False, 1), (False, True, 2)])
def test_wide_steps(use_graph, regen, n_iter, monkeypatch):
    import torch
    monkeypatch.setenv("MPPI_ROLLOUT_WAVES", "4")
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    ws = []
    for j, objective in enumerate(("gate", "contour", "track")):
        for i, (K, N) in enumerate([(128 * n_cu + 70, 5), (8192, 9), (64, 1), (2500, 6)]):
            ws.append(workload(10 * j + i, K, N, objective, False, 20.0, n_iter=n_iter,
                               ctrl_cost=0.2 if i == 1 and not regen else 0.0))
    check_batch(ws, M.FP32, 4, use_graph, "wide graph %d regen %d" % (use_graph, regen), want_U=not regen,
                **(dict(regen_average=True) if regen else {}))


@pytest.mark.parametrize("precision", [M.FP32, M.FP64], ids=["fp32", "fp64"])
@pytest.mark.parametrize("mixed", [False, True], ids=["rate", "rate+thrust"])
def test_rate_contexts(mixed, precision, monkeypatch):
    monkeypatch.setenv("MPPI_ROLLOUT_WAVES", "1")
    ws = [workload(i, K, N, ("gate", "contour", "track")[i % 3], not (mixed and i % 2), 20.0,
                   ctrl_cost=0.1 if i == 2 else 0.0) for i, (K, N) in enumerate(SHAPES)]
    check_batch(ws, precision, 1, not mixed, "rate mixed %d" % mixed)


@pytest.mark.parametrize("objective", ["gate", "contour", "track"])
@pytest.mark.parametrize("K,N", [(64, 1), (128, 7), (1024, 50)])
def test_nominal_alone_in_its_tile(K, N, objective, monkeypatch):
    """One-wave rollouts that draw against those that read the sample kernel's
    samples."""
    monkeypatch.setenv("MPPI_ROLLOUT_WAVES", "1")
    print("[gpu-case] nominal tile", objective, "K", K, "N", N, flush=True)
    sys.stdout.flush()
    out = []
    for draw in ("1", "0"):
        monkeypatch.setenv("MPPI_ROLLOUT_DRAW", draw)
        w = workload(N, K, N, objective, False, 20.0)
        sv = solver_for(w, M.FP32)
        x, got = np.array(w["x0"]), []
        for step in range(3):
            u0, _, _ = sv.solve(x, step * 0.02)
            got.append(outcome(sv))
            x = M.plant_step(w["quad"], x, u0, 0.02, 2)
        sv.close()
        out.append(got)
    for a, b in zip(*out):
        for xa, xb in zip(a, b):
            np.testing.assert_array_equal(xa, xb)
