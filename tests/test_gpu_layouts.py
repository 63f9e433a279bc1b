"""Which rollout a solve ran, at the sizes where the tests of the pair, of the
rate input's pipeline and of wide batch steps compare two layouts bit for bit:
the layout under test in one arm, its counterpart in the other."""
import sys

import numpy as np
import pytest

from paper_2509_14726_amd import mppi as M
from paper_2509_14726_amd import synth


def say(*a):
    print("[gpu-case] layouts", *a, flush=True)
    sys.stdout.flush()


def n_cu():
    import torch
    return torch.cuda.get_device_properties(0).multi_processor_count


def solver(K, N, objective, precision=M.FP32, rate=False, flags=0):
    over = dict(flags=flags)
    if rate:
        over.update(sigma=(8.0,) * 4, sigma_v=5.0, input_model=M.INPUT_RATE, rate_lim=(-10.0, 10.0), dv_lim=(-20.0, 20.0))
    w = synth.single_solve_workload(K=K, N=N, objective=objective, seed=5, track_seed=3, **{"lambda": 20.0})
    w["params"] = dict(w["params"], **over)
    if rate:
        w["x0"] = np.concatenate([w["x0"], np.full(4, synth.hover_thrust())])
    sv = M.Solver(w["quad"], w["params"], gates=w["gates"], path=w.get("path"), path_len=w.get("path_len", 0.0),
                  xref=w.get("xref"), ref_dt=w.get("ref_dt", 0.0), precision=precision)
    return sv, w


def ran(*args, **kw):
    """(layout bits, report) of one solve."""
    sv, w = solver(*args, **kw)
    assert sv.layout_ran() == 0
    _, _, info = sv.solve(w["x0"])
    bits = sv.layout_ran()
    sv.close()
    return bits, info


@pytest.fixture(autouse=True)
def automatic(monkeypatch):
    for k in ("MPPI_ROLLOUT_WAVES", "MPPI_ROLLOUT_DRAW"):
        monkeypatch.delenv(k, raising=False)


def test_nothing_solved():
    assert M.lib.mppi_layout_ran(None) == 0 and M.lib.mppi_batch_layout_ran(None) == 0


@pytest.mark.gpu
@pytest.mark.parametrize("objective,limit", [("gate", 12), ("contour", 8), ("track", 12)])
def test_pair(objective, limit, monkeypatch):
    tile_row = 64 * n_cu()
    for extra in (0, 70, 37):
        say("pair", objective, "K", 2 * tile_row + extra)
        bits, info = ran(2 * tile_row + extra, 2, objective)
        assert bits == M.RAN_PAIR and info["rollout_waves"] == 1 and info["rollout_draw"] == 0
    # the last tile count of the pipeline, and both sides of the pair's limit
    assert ran(2 * tile_row - 1, 2, objective)[0] == 0
    assert ran(limit * tile_row - 1, 1, objective)[0] == M.RAN_PAIR
    assert ran(limit * tile_row, 1, objective)[0] == 0
    monkeypatch.setenv("MPPI_ROLLOUT_WAVES", "1")
    assert ran(2 * tile_row, 2, objective)[0] == 0


@pytest.mark.gpu
@pytest.mark.parametrize("objective", ["gate", "contour", "track"])
def test_pair_in_place_of_the_drawing_wave(objective, monkeypatch):
    tile_row = 64 * n_cu()
    K, N = 4 * tile_row + 1000, 256
    say("pair, large tensor", objective, "K", K, "N", N)
    assert 16 * K * N > 256 * 2 ** 20
    for flags in (0, M.FLAG_REGEN_AVERAGE):
        bits, info = ran(K, N, objective, flags=flags)
        assert bits == M.RAN_PAIR and info["rollout_draw"] == 1 and info["regen_average"] == (1 if flags else 0)
    monkeypatch.setenv("MPPI_ROLLOUT_WAVES", "1")
    bits, info = ran(K, N, objective)
    assert bits == 0 and info["rollout_draw"] == 1


@pytest.mark.gpu
@pytest.mark.parametrize("precision", [M.FP32, M.FP64], ids=["fp32", "fp64"])
@pytest.mark.parametrize("objective", ["gate", "contour", "track"])
def test_rate_input_pipeline(objective, precision, monkeypatch):
    say("rate pipeline", objective, precision)
    fits = precision == M.FP32 or objective != "contour"
    bits, info = ran(200, 5, objective, precision=precision, rate=True)
    assert bits == (M.RAN_RATE_PIPE if fits else 0) and info["rollout_waves"] == 1
    assert ran(64 * n_cu(), 2, objective, precision=precision, rate=True)[0] == 0   # more tiles than CUs
    monkeypatch.setenv("MPPI_ROLLOUT_WAVES", "1")
    assert ran(200, 5, objective, precision=precision, rate=True)[0] == 0


@pytest.mark.gpu
@pytest.mark.parametrize("use_graph", [True, False])
@pytest.mark.parametrize("K,per_cu", [(4000, 3), (20000, 6)], ids=["rings of 8", "rings of 4"])
@pytest.mark.parametrize("objective", ["gate", "contour", "track"])
def test_wide_steps(objective, K, per_cu, use_graph, monkeypatch):
    """A step with more tiles than the wide limit, then one with fewer, against
    the contexts alone."""
    import torch
    monkeypatch.setenv("MPPI_ROLLOUT_WAVES", "4")
    tiles = (K + 64) // 64
    n = per_cu * n_cu() // tiles + 1
    assert (n - 1) * tiles <= per_cu * n_cu() < n * tiles and (tiles > n_cu()) == (per_cu == 6)
    Ns = [(5, 9, 1, 6)[i % 4] for i in range(n)]
    sw = [solver(K, N, objective) for N in Ns]
    alone = [solver(K, N, objective)[0] for N in Ns]
    B = M.Batch([s for s, _ in sw], rollout_waves=4, use_graph=use_graph)
    assert B.layout_ran() == 0
    reqs = torch.zeros((n, M.REQ_DOUBLES), dtype=torch.float64, device="cuda")
    u0s = torch.zeros((n, 4), dtype=torch.float64, device="cuda")
    for i, (_, w) in enumerate(sw):
        reqs[i, :13] = torch.from_numpy(w["x0"][:13])
    for step, wide in enumerate([True, False, True]):
        reqs[:, 13] = 0.02 * step
        torch.cuda.synchronize()
        say("wide", objective, "K", K, "graph", use_graph, "step", step)
        ids = list(range(n if wide else n - 1))
        B.solve_device(reqs.data_ptr(), u0s.data_ptr(), active=ids)
        assert bool(B.layout_ran() & M.RAN_WIDE) == wide
        torch.cuda.synchronize()
        got = u0s.cpu().numpy()
        for i in ids:
            u0, _, _ = alone[i].solve(sw[i][1]["x0"], 0.02 * step)
            np.testing.assert_array_equal(got[i], u0)
            np.testing.assert_array_equal(sw[i][0].read_samples()[0], alone[i].read_samples()[0])
            np.testing.assert_array_equal(np.array(sw[i][0].get_warm().U), np.array(alone[i].get_warm().U))
    B.close()
    for s in [s for s, _ in sw] + alone:
        s.close()


@pytest.mark.gpu
@pytest.mark.parametrize("rates", [(False, True), (True, True), (False, False)])
def test_both_input_models_share_a_launch(rates, monkeypatch):
    import torch
    sw = [solver(700, 6, "gate", rate=r) for r in rates]
    B = M.Batch([s for s, _ in sw], rollout_waves=1)
    reqs = torch.zeros((2, M.REQ_DOUBLES), dtype=torch.float64, device="cuda")
    u0s = torch.zeros((2, 4), dtype=torch.float64, device="cuda")
    for i, (_, w) in enumerate(sw):
        reqs[i, :13] = torch.from_numpy(w["x0"][:13])
        reqs[i, M.REQ_THRUST:M.REQ_THRUST + 4] = synth.hover_thrust()
    torch.cuda.synchronize()
    say("input models", rates)
    B.solve_device(reqs.data_ptr(), u0s.data_ptr())
    torch.cuda.synchronize()
    assert bool(B.layout_ran() & M.RAN_MIXED) == (rates == (False, True))
    B.close()
    for s, _ in sw:
        s.close()


@pytest.mark.gpu
def test_a_number_of_rollout_workgroups_holds_the_pipeline(monkeypatch):
    """A batch with more tiles than pipelines: wide with the automatic number of
    rollout workgroups, also when that number is set again, pipelines with
    another one; the same results either way."""
    import torch
    monkeypatch.setenv("MPPI_ROLLOUT_WAVES", "4")
    sizes = [(384 * n_cu() + 70, 5), (3000, 9)]
    reqs = torch.zeros((2, M.REQ_DOUBLES), dtype=torch.float64, device="cuda")
    out = []
    for how in ("automatic", "as reported", "others"):
        sw = [solver(K, N, "gate") for K, N in sizes]
        u0s = torch.zeros((2, 4), dtype=torch.float64, device="cuda")
        for i, (_, w) in enumerate(sw):
            reqs[i, :13] = torch.from_numpy(w["x0"][:13])
        torch.cuda.synchronize()
        B = M.Batch([s for s, _ in sw], rollout_waves=4, rollout_groups=100 if how == "others" else 0)
        if how == "as reported":
            cfg = B.get_cfg()
            B.set_cfg(**dict(cfg, use_graph=True, regen_average=False))
            assert B.get_cfg() == cfg
        say("rollout workgroups", how)
        B.solve_device(reqs.data_ptr(), u0s.data_ptr())
        torch.cuda.synchronize()
        assert B.get_cfg()["rollout_groups"] == 100 if how == "others" else B.get_cfg()["rollout_groups"] > 100
        assert bool(B.layout_ran() & M.RAN_WIDE) == (how != "others")
        out.append((u0s.cpu().numpy(), [s.read_samples()[0] for s, _ in sw]))
        B.close()
        for s, _ in sw:
            s.close()
    for u0, J in out[1:]:
        np.testing.assert_array_equal(u0, out[0][0])
        for a, b in zip(J, out[0][1]):
            np.testing.assert_array_equal(a, b)
