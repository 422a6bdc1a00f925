"""The graph kernel on masks by code for graphs with up to two producers and two consumers a type, at the edges of what it takes: windows
of 1 to 8 micro-batches, 16 devices and 16 types, memory prefixes, consumers on the producer's device, both consumers on one device,
fixed leads, long times; random graphs inside these limits and one step outside; against the oracle, and against words by type."""
import random

import pytest

from paper_2311_15269_amd import workloads as W
from tests.test_gpu_dag import _compare

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU: the HIP path has no CPU fallback")
    from paper_2311_15269_amd import binding
    binding.load_library()
    return binding


def graph(dev, deps, nr, cap, space="sampled_repair", t=None, m=None, fixed=None, step=20000, name="graph"):
    K, D = len(dev), max(dev) + 1
    return {"name": name, "D": D, "K": K, "NR": nr, "M": cap, "t": t or [1 + (5 * i) % 7 for i in range(K)], "m": m or [0] * K,
            "dev_mask": [1 << d for d in dev], "deps": deps, "space": space, "seed": 0xE0FFEE, "lead_step_q16": step, "fixed_leads": fixed}


def ladder(rungs, nr, **kw):
    """two chains side by side with rungs between them: two producers and two consumers a type"""
    deps = [(2 * i + a, 2 * i + 2 + b) for i in range(rungs - 1) for a in (0, 1) for b in (0, 1)]
    return graph(list(range(2 * rungs)), deps, nr, 0, name="ladder", **kw)


def random_graph(rng, wide):
    D, nr = rng.randint(2, 8), rng.randint(1, 6)
    K = rng.randint(max(3, D), min(2 * D, 16))
    dev = [i % D for i in range(K)]
    rng.shuffle(dev)
    ins, outs, deps = [0] * K, [0] * K, []
    for b in range(1, K):
        for a in rng.sample(range(b), min(b, rng.randint(1, 3))):
            if ins[b] < 2 + wide and outs[a] < 2:
                deps.append((a, b))
                ins[b] += 1
                outs[a] += 1
    if any(i == 0 and o == 0 for i, o in zip(ins, outs)):
        return random_graph(rng, wide)
    m = [0] * K
    for d in range(D):
        on = [i for i in range(K) if dev[i] == d]
        if len(on) == 2:
            m[on[0]] = rng.randint(0, 3)
            m[on[1]] = -m[on[0]]
    return graph(dev, deps, nr, rng.randint(1, 12), rng.choice(["sampled_repair", "sampled_strict"]), [rng.randint(1, 9) for _ in range(K)], m,
                 step=rng.choice([0, 9000, 30000, 65536]), name="random")


SHAPES = [W.kshape_problem(nr, max(2, nr - 1), space=s) for nr in (1, 2, 5, 8) for s in ("sampled_repair", "sampled_strict")]
SHAPES += [W.diamond_problem(nr, nr + 1) for nr in (1, 3, 8)]
SHAPES += [ladder(8, 2), ladder(8, 8, step=5000), ladder(2, 5, space="sampled_strict"), ladder(3, 4, fixed=[3, 2, 2, 1, 1, 0])]
SHAPES += [graph([0, 0, 1, 1, 2, 2], [(0, 1), (0, 2), (1, 3), (2, 3), (3, 4), (2, 4), (4, 5)], 4, 6, m=[3, -3, 2, -2, 0, 0]),
           graph([0, 1, 1, 2], [(0, 1), (0, 2), (1, 3), (2, 3)], 6, 0),
           graph([0, 1, 2, 3], [(0, 1), (0, 2), (1, 3), (2, 3)], 4, 0, t=[1, 200, 3, 150]),
           graph([0, 1, 0, 1, 2], [(0, 1), (0, 3), (1, 2), (3, 4), (2, 4)], 8, 50000, m=[700, 900, -700, -900, 0])]


@pytest.mark.parametrize("words", [False, True])
@pytest.mark.parametrize("prob", SHAPES, ids=["%s-%ddev-nr%d-%s-%d" % (p["name"], p["D"], p["NR"], p["space"], k) for k, p in enumerate(SHAPES)])
def test_shapes(gpu, monkeypatch, prob, words):
    if words:
        monkeypatch.setenv("TESSEL_GRAPH_WORDS", "1")
    _compare(gpu, prob, 12345, 3000)


@pytest.mark.parametrize("seed", range(24))
def test_random_graphs(gpu, seed):
    _compare(gpu, random_graph(random.Random(1000 + seed), seed % 6 == 5), seed * 7919, 2000)


@pytest.mark.parametrize("prob", [W.kshape_problem(4, 4), W.diamond_problem(3, 3), W.diamond_problem(4, 5)], ids=["kshape", "diamond-3", "diamond-4"])
def test_many_rounds(gpu, monkeypatch, prob):
    """several rounds a wave: slots are used again, stragglers wait for the longer search; periods of cycles through two windows"""
    n = 700001
    got = []
    for words in (None, "1"):
        if words:
            monkeypatch.setenv("TESSEL_GRAPH_WORDS", words)
        g = gpu.Problem(prob)
        g.eval_candidates(99, n)
        r = g.best()
        got.append([r[k] for k in ("period", "index", "peak", "n_evaluated", "n_feasible", "n_reject")])
        code, peak = g.score_candidates(99, n)
        got[-1] += [code, peak]
    assert got[0][:6] == got[1][:6] and bool((got[0][6] == got[1][6]).all()) and bool((got[0][7] == got[1][7]).all())
