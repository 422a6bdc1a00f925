"""CANONICAL ranges by tables of the orders that go together (TESSEL_PAIRS=1: wherever they fit, 0: nowhere), against the oracle:
one to several words of 32 orders of the first device, ranges that begin and end inside a word, of one candidate and of several lead
vectors, units shared out without equal distances (scattered), indices from 2^32 on, devices of one, two and four types or none, dependencies that come back to a device, fixed leads."""
import pytest

from paper_2311_15269_amd import workloads as W
from tests.test_gpu_ranked import LEADS, forward, linear, rounds

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU: the HIP path has no CPU fallback")
    from paper_2311_15269_amd import binding
    binding.load_library()
    return binding


def placed(where, D, nr, cap):
    return W.pipeline_problem(where, [1 + i % 3 for i in range(len(where))], [2 + i % 2 for i in range(len(where))], D, nr, cap, "canonical")


def seventeen(nr):
    """two devices, chains of one, one and two types: 17 boundary values at five micro-batches"""
    return {"name": "seventeen", "D": 2, "K": 4, "NR": nr, "M": 0, "t": [2, 3, 1, 4], "m": [0] * 4, "dev_mask": [1, 2, 1, 2], "deps": [(2, 3)],
            "space": "canonical", "seed": 0, "lead_step_q16": 0, "fixed_leads": None}


# name, problem, first index (None: the last `count` candidates), count
CASES = [("6-orders-whole", linear(2, 2, 2), 0, 288), ("6-orders-three-devices", linear(3, 2, 2), 17, 1001),
         ("20-orders", linear(4, 3, 3), 1000003, 40000), ("20-orders-end", linear(4, 3, 3), None, 5003),
         ("70-orders-one", linear(4, 4, 4), 1063399420, 1), ("70-orders-in-a-word", linear(4, 4, 4), 1063399423, 7),
         ("70-orders-across-words", linear(4, 4, 4), 1063399400, 130), ("70-orders", linear(4, 4, 4), 1063390001, 40001),
         ("70-orders-leads", linear(2, 4, 5), 5000, 60001), ("252-orders", linear(3, 5, 5), 900000001, 30007),
         ("252-orders-scattered", linear(3, 5, 5), 900000001, 63501),
         ("6-orders-8-devices", linear(8, 2, 2), 9000001, 30001), ("above-2^32", linear(5, 4, 6), 284464890000, 9001),
         ("across-2^32", dict(forward(4, 2, 6), fixed_leads=LEADS), (1 << 32) - 2000, 4001),
         ("four-types", placed([0, 1, 1, 0], 2, 2, 3), 777, 20011), ("back-and-forth", placed([0, 1, 0, 2], 3, 2, 3), 30000, 20011),
         ("no-blocks-on-1", placed([0, 2, 3], 4, 3, 2), 4001, 30001), ("nothing-on-the-first", placed([1, 2], 3, 3, 3), 5, 2001),
         ("one-type-on-the-first", forward(3, 1, 3), 0, 10), ("three-types", rounds(2, 3, 2), 100, 8001),
         ("17-values", seventeen(5), 30011, 20011)]


@pytest.mark.parametrize("name,prob,first,count", CASES, ids=[c[0] for c in CASES])
def test_orders_that_go_together(gpu, monkeypatch, name, prob, first, count):
    from oracle import Oracle
    handle = gpu.Problem(prob)
    space = handle.candidate_count()
    count = min(count, space)
    first = space - count if first is None else min(first, space - count)
    want = Oracle(prob).sweep(first, count)
    for pairs in ("1", "0"):
        monkeypatch.setenv("TESSEL_PAIRS", pairs)
        handle.reset()
        handle.eval_candidates(first, count)
        got = handle.best()
        assert (got["n_evaluated"], got["n_feasible"], got["n_reject"][1:]) == (count, want["n_feasible"], want["n_reject"][1:]), pairs
        if want["n_feasible"]:
            assert (got["period"], got["index"], got["peak"]) == (want["period"], want["index"], want["peak"]), pairs
