"""Completion candidates of chains with a device a type, at the edges of the kernel's rows: 1 to 4 types a device, 1, 4, 5 and 8 devices (devices
with different numbers of types and with none), several chains, the largest jitter and number of micro-batches, a cap that leaves no schedule."""
import numpy as np
import pytest

from paper_2311_15269_amd import workloads as W
from tests.test_gpu_dag import gpu  # noqa: F401

pytestmark = pytest.mark.gpu


def _chains(devs, D, nr, cap, seed):
    """a chain for every list of devices: forward on the first half of it, backward on the rest, times from 1 to 3"""
    flat = [d for ds in devs for d in ds]
    m = [(1 if k < len(ds) // 2 else -1 if k >= len(ds) - len(ds) // 2 else 0) for ds in devs for k in range(len(ds))]
    deps, at = [], 0
    for ds in devs:
        deps += [(at + k, at + k + 1) for k in range(len(ds) - 1)]
        at += len(ds)
    return {"name": "chains", "D": D, "K": len(flat), "NR": nr, "M": cap, "t": [1 + (i * 7 + seed) % 3 for i in range(len(flat))], "m": m,
            "dev_mask": [1 << d for d in flat], "deps": deps, "space": "sampled_repair", "seed": seed, "lead_step_q16": 30000, "fixed_leads": None}


CASES = {
    "1dev-1type": (_chains([[0]], 1, 2, 4, 1), 5, 3),
    "1dev-4types": (_chains([[0, 0, 0, 0]], 1, 3, 4, 2), 17, 5),
    "4dev-2types": (W.pipeline_problem(W.linear_placement(4), [1, 2, 1, 2], [2, 3, 1, 2], 4, 4, 4, "sampled_repair", seed=9, lead_step_q16=20000), 30, 4),
    "4dev-uneven": (_chains([[0, 1, 3, 3, 1, 0], [1, 3, 1], [0]], 4, 3, 4, 3), 23, 7),
    "5dev-2types": (_chains([[0, 1, 2, 3, 4, 4, 3, 2, 1, 0]], 5, 4, 4, 4), 29, 2),
    "5dev-3types": (_chains([[0, 2, 4, 4, 2, 0], [1, 2, 1], [3]], 5, 4, 4, 5), 31, 9),
    "8dev-8chains": (_chains([[k, (k + 3) % 8, (k + 3) % 8, k] for k in range(8)], 8, 2, 5, 6), 19, 63),
    "some-without-schedule": (_chains([[1, 4, 0, 0, 4, 1], [3, 3, 3, 3], [0, 2, 1, 1, 2, 0]], 5, 3, 3, 271), 25, 6),
    "no-schedule": (_chains([[1, 0, 1, 1, 0, 1]], 2, 3, 2, 178), 25, 6),
    "8dev-few-types": (_chains([[6], [1, 1]], 8, 3, 4, 7), 21, 5),
    "8dev-idle-between": (_chains([[7, 2, 2, 7], [2, 5, 2]], 8, 4, 4, 8), 26, 11),
    "4dev-idle-first": (_chains([[3, 1, 1, 3]], 4, 2, 3, 9), 18, 2),
    "longest": (W.xshape_problem(4, 1, 2, 2, 4), 1023, 6),
}


@pytest.mark.parametrize("replay", ["0", "1"])
@pytest.mark.parametrize("name", CASES)
def test_completions_of_chains(gpu, monkeypatch, name, replay):  # noqa: F811
    from oracle import Oracle
    prob, N, J = CASES[name]
    monkeypatch.setenv("TESSEL_REPLAY_BLOCKS", replay)
    g, o = gpu.Problem(prob), Oracle(prob)
    g.eval_candidates(0, 3000)
    assert g.best()["feasible"], name
    status, leads, orders = o.decode(g.best()["index"])
    for first, n in ((0, 1), (0, 130), ((1 << 33) + 7, 63)):
        n = min(n, 40) if N > 500 else n
        want, best, ordinal = o.completion_scores(leads, orders, N, first, n, J)
        assert np.array_equal(g.score_completions(N, J, first, n).cpu().numpy(), want), (name, first)
    g.search_completions(N, J, first, n)
    if best is None:
        with pytest.raises(gpu.TesselError) as e:
            g.best_completion(N)
        assert e.value.code == -10
    else:
        got = g.best_completion(N)
        assert (got["makespan"], got["ordinal"]) == (best, ordinal), name


@pytest.mark.parametrize("n", [64, 65, 64 * 1024 - 1, 64 * 1024, 64 * 1024 + 1, 64 * 1025 + 3])
def test_the_best_of_many_workgroups(gpu, n):  # noqa: F811
    """the search's best = the first least makespan of the same range, around the number of records that are read at a time"""
    prob, N, J = CASES["5dev-2types"]
    g = gpu.Problem(prob)
    g.eval_candidates(0, 3000)
    first = 12345
    scores = g.score_completions(N, J, first, n).cpu().numpy()
    g.search_completions(N, J, first, n)
    got = g.best_completion(N)
    assert (got["makespan"], got["ordinal"]) == (int(scores.min()), first + int(scores.argmin()))


STUCK = {"all": (_chains([[2, 1, 1, 2, 0, 0, 2, 1, 1, 2]], 3, 8, 2, 612), 25, 6),
         "most-waves": (_chains([[1, 0, 0, 1, 1, 0, 0, 1]], 2, 4, 2, 846), 25, 6)}


@pytest.mark.parametrize("n", [1, 64, 65, 4100])
@pytest.mark.parametrize("name", STUCK)
def test_waves_that_get_stuck(gpu, name, n):  # noqa: F811
    """whole waves without a schedule stop early; waves with one candidate that has one, and a last wave with lanes to spare, do not"""
    from oracle import Oracle
    prob, N, J = STUCK[name]
    g, o = gpu.Problem(prob), Oracle(prob)
    g.eval_candidates(0, 3000)
    status, leads, orders = o.decode(g.best()["index"])
    want, best, ordinal = o.completion_scores(leads, orders, N, 0, n, J)
    assert (best is None) == (name == "all" or n < 100)
    assert np.array_equal(g.score_completions(N, J, 0, n).cpu().numpy(), want)
    g.search_completions(N, J, 0, n)
    if best is not None:
        got = g.best_completion(N)
        assert (got["makespan"], got["ordinal"]) == (best, ordinal)
