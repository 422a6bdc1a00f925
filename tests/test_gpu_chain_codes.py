"""Chains that the graph kernel builds on masks by code: every layout of its records (order and entries left in one word or not, one to three
bits a symbol), 32 codes and one device more, 64 codes, and problems just inside and just outside what a record's fields hold (memory, end times
in 16 bits, a dependency listed twice)."""
import pytest

from paper_2311_15269_amd import workloads as W
from tests.test_gpu_dag import _compare, gpu  # noqa: F401
from tests.test_gpu_detail_lanes import folded, three_on_one
from tests.test_gpu_wide import crowded, inference, vshape

pytestmark = pytest.mark.gpu


def heavy(prob, factor):
    """memory deltas and cap `factor` times as large"""
    return dict(prob, m=[factor * x for x in prob["m"]], M=factor * prob["M"], name="%s-m%d" % (prob["name"], factor))


def slow(prob, factor):
    return dict(prob, t=[factor * x for x in prob["t"]], name="%s-t%d" % (prob["name"], factor))


def twice(prob):
    return dict(prob, deps=prob["deps"] + prob["deps"][2:4], name=prob["name"] + "-twice")


SHAPES = [
    (vshape(16, 8, 12), 900), (vshape(16, 9, 14), 700), (vshape(17, 8, 12), 700), (vshape(32, 3, 5), 1200),      # 32 and 64 codes, one word and two
    (vshape(9, 7, 100), 900), (vshape(3, 15, 17), 900), (vshape(12, 1, 1), 1500), (inference(10, 7), 900), (inference(32, 9), 500),
    (folded(9, 3, 9), 900), (folded(16, 8, 12), 300), (three_on_one(9, 10), 900), (three_on_one(16, 2, "sampled_strict"), 3000),
    (crowded(4, 4, 4, 9), 900), (crowded(4, 3, 5, 30, step=4000), 900), (crowded(8, 4, 2, 9, step=3000), 700), (crowded(5, 3, 3, 8), 900),
    (crowded(2, 4, 1, 3, space="sampled_strict"), 3000), (vshape(11, 2, 4, space="sampled_strict", step=9000), 3000),
    (heavy(vshape(10, 4, 5), 571), 900), (heavy(vshape(10, 4, 5), 572), 900),                  # 14 signed bits of memory: spans to 8,000 and above
    (heavy(folded(9, 2, 5), 2500), 600), (heavy(crowded(4, 3, 4, 9), 2), 900), (heavy(crowded(4, 3, 4, 9), 3), 900),   # 16 and 8 bits (to 120)
    (slow(vshape(10, 4, 5), 22), 900), (slow(vshape(10, 4, 5), 23), 900),                     # the end of the last sweep below and above 65,536
    (twice(vshape(10, 4, 5)), 900), (dict(vshape(12, 9, 30), fixed_leads=[0] * 24), 600),
    (dict(crowded(4, 3, 3, 30), fixed_leads=[2] * 8 + [1] * 8 + [0] * 8), 900),
]


@pytest.mark.parametrize("prob,n", SHAPES, ids=["%s-nr%d-cap%d-%s" % (p["name"], p["NR"], p["M"], p["space"]) for p, _ in SHAPES])
def test_scores(gpu, prob, n):  # noqa: F811
    _compare(gpu, prob, 1 << 33 if prob["space"] == "sampled_repair" else 0, n)


@pytest.mark.parametrize("prob", [vshape(16, 8, 12), crowded(4, 3, 4, 9), folded(9, 4, 8)], ids=lambda p: p["name"])
def test_many_rounds(gpu, prob):  # noqa: F811
    """several rounds a wave: slots are reused, first sweeps run on full waves, stragglers collect; split or whole, the same best"""
    n = 1100003
    whole, parts = gpu.Problem(prob), gpu.Problem(prob)
    whole.eval_candidates(5, n)
    for at in range(0, n, 70001):
        parts.eval_candidates(5 + at, min(70001, n - at))
    a, b = whole.best(), parts.best()
    assert a["n_evaluated"] == n
    for k in ("period", "index", "peak", "n_evaluated", "n_feasible", "n_reject"):
        assert a[k] == b[k], k
    code, peak = whole.score_candidates(5, n)
    ok = code > 0
    assert int(ok.sum()) == a["n_feasible"] and int(code[ok].min()) == a["period"] and int((code == a["period"]).nonzero()[0][0]) + 5 == a["index"]


@pytest.mark.parametrize("k", [0, 1, 3, 5, 9, 11, 13, 16, 17, 19, 24, 28])
def test_against_words_by_type(gpu, monkeypatch, k):  # noqa: F811
    """the same scores and peaks by masks by code and by a word a type, of full waves and a last one that is not"""
    prob, n = SHAPES[k][0], 20011
    codes = gpu.Problem(prob).score_candidates(1 << 20, n)
    monkeypatch.setenv("TESSEL_GRAPH_WORDS", "1")
    words = gpu.Problem(prob).score_candidates(1 << 20, n)
    assert (codes[0] == words[0]).all() and (codes[1] == words[1]).all()
