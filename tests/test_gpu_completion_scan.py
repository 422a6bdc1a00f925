"""The completion search of what is not a few chains on single devices: blocks on several devices, graphs with up to four producers and consumers,
more than eight chains, 32 types, more than 64 KB of rows, types looked at in fours and a rest, no and large jitters, tight caps; windows as a matrix and block by block.
Every candidate's makespan, the best one and where nothing fits, against the oracle."""
import numpy as np
import pytest

from paper_2311_15269_amd import workloads as W
from tests.test_gpu_dag import gpu  # noqa: F401
from tests.test_gpu_graph_kernel import fan
from tests.test_gpu_stage import on_some
from tests.test_gpu_wide import shared_block

pytestmark = pytest.mark.gpu


def chains(number, length, D, nr, cap):
    """`number` chains of `length` types, the k-th type of all on device k mod D; the first type holds what the last gives back where both share it"""
    K = number * length
    dev = [(c + k) % D for c in range(number) for k in range(length)]
    m = [0] * K
    for c in range(number):
        if dev[c * length] == dev[c * length + length - 1] and length > 1:
            m[c * length], m[c * length + length - 1] = 1, -1
    return {"name": "chains", "D": D, "K": K, "NR": nr, "M": cap, "t": [1 + (7 * i) % 5 for i in range(K)], "m": m, "dev_mask": [1 << d for d in dev],
            "deps": [(c * length + k, c * length + k + 1) for c in range(number) for k in range(length - 1)], "space": "sampled_repair",
            "seed": 0xF0FFEE, "lead_step_q16": 15000, "fixed_leads": None}


def forked():
    """a chain of 25 types on 8 devices whose last but one feeds another: 24 consumed types with rings of 16 micro-batches each (leads from 0 to 3 and
    more at windows of five), for which the kernel asks for 67,856 bytes of LDS"""
    K, D = 26, 8
    m = [0] * K
    for i in (0, 1, 5):
        m[i], m[i + 8] = 1, -1
    return {"name": "forked", "D": D, "K": K, "NR": 5, "M": 100, "t": [1 + (5 * i) % 4 for i in range(K)], "m": m, "dev_mask": [1 << i % D for i in range(K)],
            "deps": [(i, i + 1) for i in range(24)] + [(23, 25)], "space": "sampled_repair", "seed": 21, "lead_step_q16": 12000, "fixed_leads": None}


CASES = {"forked": (forked(), 33, 4), "shared-2": (shared_block(2, 3, 7), 14, 3), "shared-8": (shared_block(8, 4, 100), 23, 6), "shared-5-tight": (shared_block(5, 2, 5), 17, 0),
         "some-4": (on_some(4, 3, 100), 40, 63), "chains-9": (chains(9, 3, 8, 1, 100), 17, 2),
         "chains-16": (chains(16, 2, 8, 1, 100), 24, 5), "fan-4": (fan(4, 3, 0), 13, 4), "fan-3": (fan(3, 5, 0), 30, 1), "kshape-8": (W.kshape_problem(8, 9), 40, 9),
         "diamond-5": (W.diamond_problem(5, 5), 33, 2), "one-type": (chains(1, 2, 1, 1, 3), 6, 1)}


@pytest.mark.parametrize("replay", ["0", "1"])
@pytest.mark.parametrize("name", CASES)
def test_makespans(gpu, monkeypatch, name, replay):  # noqa: F811
    from oracle import Oracle
    monkeypatch.setenv("TESSEL_REPLAY_BLOCKS", replay)
    prob, N, J = CASES[name]
    g, o = gpu.Problem(prob), Oracle(prob)
    g.eval_candidates(0, 6000)
    status, leads, orders = o.decode(g.best()["index"])
    assert name != "forked" or max(leads) - min(leads) >= 3
    n = 321
    want, best, ordinal = o.completion_scores(leads, orders, N, 0, n, J)
    assert np.array_equal(g.score_completions(N, J, 0, n).cpu().numpy(), want), name
    g.search_completions(N, J, 0, n)
    if best is not None:
        got = g.best_completion(N)
        assert (got["makespan"], got["ordinal"]) == (best, ordinal)
