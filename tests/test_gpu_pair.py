"""A pair of waves per tile (more than two tiles per CU) against one wave per
tile, which other tests hold against the oracle: every output bit for bit over
warm solves.  Horizons around the pair's LDS rings of four steps, a last tile
that holds the nominal alone, ragged last tiles, drag, control cost, several
iterations, and the average that draws the samples again."""
import sys

import numpy as np
import pytest

from paper_2509_14726_amd import mppi as M
from paper_2509_14726_amd import synth

pytestmark = pytest.mark.gpu


def outputs(K, N, objective, seed, want_U, flags=0, drag=False, **over):
    w = synth.single_solve_workload(K=K, N=N, objective=objective, seed=seed, track_seed=3, **{"lambda": 20.0}, **over)
    if flags:
        w["params"] = dict(w["params"], flags=w["params"].get("flags", 0) | flags)
    if drag:
        w["quad"] = dict(w["quad"], drag=(0.3, 0.3, 0.15))
    sv = M.Solver(w["quad"], w["params"], gates=w["gates"], path=w.get("path"), path_len=w.get("path_len", 0.0),
                  xref=w.get("xref"), ref_dt=w.get("ref_dt", 0.0))
    x, out = np.array(w["x0"]), []
    for step in range(3):
        u0, U, info = sv.solve(x, step * 0.02)
        J, Us = sv.read_samples(want_U=want_U)
        wd = sv.get_warm()
        out.append((u0, U, J, Us if want_U else 0, info["J_min"], info["S"], info["J_nom"], info["rollout_waves"],
                    info["status"] if "status" in info else 0, np.array(wd.U), np.array(wd.V), np.array(wd.allow),
                    wd.theta0))
        x = M.plant_step(w["quad"], x, u0, 0.02, 2)
    sv.close()
    return out


def compare(monkeypatch, env, *args, **kw):
    for k in ("MPPI_ROLLOUT_WAVES", "MPPI_ROLLOUT_DRAW"):
        monkeypatch.delenv(k, raising=False)
    pair = outputs(*args, **kw)
    for k, v in env.items():
        monkeypatch.setenv(k, v)
    one = outputs(*args, **kw)
    for a, b in zip(pair, one):
        for xa, xb in zip(a, b):
            np.testing.assert_array_equal(xa, xb)


def tiles_per_cu():
    import torch
    return 64 * torch.cuda.get_device_properties(0).multi_processor_count


@pytest.mark.parametrize("objective", ["gate", "contour", "track"])
@pytest.mark.parametrize("N", [1, 2, 3, 4, 5, 6, 7, 8, 9, 23])
def test_pair_equals_one_wave(N, objective, monkeypatch):
    K = 2 * tiles_per_cu() + (0, 70, 37)[N % 3]
    print("[gpu-case] pair", objective, "K", K, "N", N, flush=True)
    sys.stdout.flush()
    compare(monkeypatch, {"MPPI_ROLLOUT_WAVES": "1"}, K, N, objective, 50 + N, True, drag=N % 2 == 1,
            ctrl_cost=0.3 if N % 3 == 1 else 0.0, n_iter=2 if N % 4 == 1 else 1)


@pytest.mark.parametrize("objective", ["gate", "contour", "track"])
@pytest.mark.parametrize("regen", [False, True])
def test_pair_in_place_of_the_drawing_wave(regen, objective, monkeypatch):
    """A sample tensor beyond the last-level cache, stored or drawn again."""
    K, N = 4 * tiles_per_cu() + 1000, 256
    print("[gpu-case] pair, large tensor", objective, "K", K, "N", N, "regen", regen, flush=True)
    sys.stdout.flush()
    compare(monkeypatch, {"MPPI_ROLLOUT_WAVES": "1"}, K, N, objective, 9, False,
            flags=M.FLAG_REGEN_AVERAGE if regen else 0)
