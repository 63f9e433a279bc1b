"""Autotuner cache: an entry is taken over only by what it was timed for.  The
stored average reads no sample whose weight is exactly zero, so the choice
between it and the regenerating one depends on how sharp the weights are."""
import json
import sys

import pytest

from paper_2509_14726_amd import mppi as M
from paper_2509_14726_amd import synth

pytestmark = pytest.mark.gpu


def say(*a):
    print("[gpu-case] tune cache", *a, flush=True)
    sys.stdout.flush()


def solver(**over):
    w = synth.single_solve_workload(K=2000, N=20, seed=3, **over)
    return M.Solver(w["quad"], w["params"], gates=w["gates"]), w


def request(ws):
    import torch
    r = torch.zeros((len(ws), M.REQ_DOUBLES), dtype=torch.float64, device="cuda")
    for i, w in enumerate(ws):
        r[i, :13] = torch.from_numpy(w["x0"])
    torch.cuda.synchronize()
    return r


BASE = {"lambda": 1.0, "sigma": (1.0,) * 4}
OTHERS = [{"lambda": 1e4}, {"lambda": 0.01}, {"sigma": (0.1,) * 4}, {"n_iter": 2}]


@pytest.mark.parametrize("kind", ["context", "batch"])
def test_choices_are_not_shared(kind, tmp_path):
    import torch
    cache = str(tmp_path / "tune.json")

    def tuned(over):
        say(kind, over)
        sv, w = solver(**{**BASE, **over})
        req = request([w])
        if kind == "context":
            hit = bool(sv.autotune(req.data_ptr(), reps=1, cache_path=cache)["from_cache"])
        else:
            u0 = torch.zeros((1, 4), dtype=torch.float64, device="cuda")
            B = M.Batch([sv])
            hit = B.autotune(req.data_ptr(), u0.data_ptr(), reps=1, cache_path=cache)[2]
            B.close()
        sv.close()
        return hit

    assert not tuned({})
    assert tuned({})
    for i, over in enumerate(OTHERS):
        assert not tuned(over), over
        assert len(json.load(open(cache))) == 2 + i
        assert tuned(over)


def test_layouts_and_other_kernels_have_entries_of_their_own(tmp_path, monkeypatch):
    cache = str(tmp_path / "tune.json")

    def tuned(waves, draw=None):
        say("waves", waves, "draw", draw)
        monkeypatch.setenv("MPPI_ROLLOUT_WAVES", waves)
        if draw:
            monkeypatch.setenv("MPPI_ROLLOUT_DRAW", draw)
        sv, w = solver(**BASE)
        r = sv.autotune(request([w]).data_ptr(), reps=1, cache_path=cache)
        sv.close()
        return bool(r["from_cache"])

    assert not tuned("4") and tuned("4")
    assert not tuned("3") and not tuned("1", "1") and tuned("1", "1")
    assert len(json.load(open(cache))) == 3
    # an entry that another version of the kernels left is not taken over
    data = json.load(open(cache))
    with open(cache, "w") as f:
        f.write("{\n" + ",\n".join('"%s": %s' % (k[:k.rindex("|")], json.dumps(v)) for k, v in data.items()) + "\n}\n")
    assert not tuned("1", "1")
