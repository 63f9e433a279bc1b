"""The batched average with one horizon step per block (where the steps do not
outnumber the CUs) and with several (beyond), against the same contexts solved
alone, which other tests hold against the oracle: bit for bit.  One batch
changes between the two as its active contexts change, with captured launch
sequences and without."""
import sys

import numpy as np
import pytest

from paper_2509_14726_amd import mppi as M
from paper_2509_14726_amd import synth

pytestmark = pytest.mark.gpu

# horizons around the chunks of 3 and 4 steps; one, two, three and many rounds of samples
SHAPES = [(64, 1), (200, 2), (2048, 3), (2050, 4), (4096, 5), (4100, 6), (6200, 7), (1000, 8), (8192, 9), (17000, 11)]


def n_cu():
    import torch
    return torch.cuda.get_device_properties(0).multi_processor_count


def solver(i, K, N, objective, lam, rate=False):
    over = {"lambda": lam}
    if rate:
        over.update(sigma=(8.0,) * 4, sigma_v=5.0, input_model=M.INPUT_RATE, rate_lim=(-10.0, 10.0), dv_lim=(-20.0, 20.0))
    w = synth.single_solve_workload(K=K, N=N, objective=objective, seed=70 + i, track_seed=3, **over)
    if rate:
        w["x0"] = np.concatenate([w["x0"], np.full(4, synth.hover_thrust())])
    return M.Solver(w["quad"], w["params"], gates=w["gates"], path=w.get("path"), path_len=w.get("path_len", 0.0),
                    xref=w.get("xref"), ref_dt=w.get("ref_dt", 0.0)), w


def outcome(sv):
    status, info = sv.read_info()
    wd = sv.get_warm()
    return [status, info["J_min"], info["S"], info["J_nom"], info["ess"], np.array(wd.U), np.array(wd.V),
            np.array(wd.allow), wd.theta0, wd.vtheta]


@pytest.mark.parametrize("regen,use_graph", [(False, True), (False, False), (True, True)])
@pytest.mark.parametrize("objective", ["gate", "contour", "track"])
@pytest.mark.parametrize("lam", [0.5, 1e4])
def test_one_and_several_steps_a_block(lam, objective, regen, use_graph, monkeypatch):
    import torch
    monkeypatch.setenv("MPPI_ROLLOUT_WAVES", "4" if regen else "1")
    rate = not regen and objective == "contour"
    # the long horizons at the end carry the sum past the CUs
    shapes = SHAPES + [(64, 128)] * (n_cu() // 128 + 1)
    few = list(range(len(SHAPES)))
    assert sum(N for _, N in SHAPES) <= n_cu() < sum(N for _, N in shapes)
    sw = [solver(i, K, N, objective, lam, rate and i % 2 == 0) for i, (K, N) in enumerate(shapes)]
    solo = [solver(i, K, N, objective, lam, rate and i % 2 == 0)[0] for i, (K, N) in enumerate(shapes)]
    B = M.Batch([s for s, _ in sw], rollout_waves=4 if regen else 1, use_graph=use_graph, regen_average=regen)
    reqs = torch.zeros((len(sw), M.REQ_DOUBLES), dtype=torch.float64, device="cuda")
    u0s = torch.zeros((len(sw), 4), dtype=torch.float64, device="cuda")
    for step, active in enumerate([None, few, few, None]):
        ids = few if active is not None else list(range(len(sw)))
        for slot, i in enumerate(ids):
            x = sw[i][1]["x0"]
            reqs[slot, :13] = torch.from_numpy(x[:13])
            reqs[slot, 13] = step * 0.02
            if len(x) > 13:
                reqs[slot, M.REQ_THRUST:M.REQ_THRUST + 4] = torch.from_numpy(x[13:])
        torch.cuda.synchronize()
        print("[gpu-case] batch average", objective, "lambda", lam, "regen", regen, "step", step, flush=True)
        sys.stdout.flush()
        B.solve_device(reqs.data_ptr(), u0s.data_ptr(), active=active)
        torch.cuda.synchronize()
        assert bool(B.layout_ran() & M.RAN_SINGLE) == (active is not None)
        got = u0s.cpu().numpy()
        for slot, i in enumerate(ids):
            u0, _, _ = solo[i].solve(sw[i][1]["x0"], step * 0.02)
            np.testing.assert_array_equal(got[slot], u0)
            for a, b in zip(outcome(sw[i][0]), outcome(solo[i])):
                np.testing.assert_array_equal(a, b)
    B.close()
    for s in [s for s, _ in sw] + solo:
        s.close()
