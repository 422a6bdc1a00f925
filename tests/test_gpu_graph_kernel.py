"""The graph kernel at the edges of what its tables hold, element by element against the oracle: most producers a type's
word has fields for and one more (which the general kernel takes), most consumers and one more and many more, windows with an odd
number of blocks, an exhaustive space whole, blocks on several devices of a branching graph, a type without dependencies, forward-only pipelines
(whose boundary values never grow alike), ranges around one wave, and every period left to the general kernel."""
import numpy as np
import pytest

from paper_2311_15269_amd import workloads as W
from tests.test_gpu_dag import _compare, random_graph_problem
from tests.test_gpu_wide import inference, random_crowded_graph, random_wide_graph, shared_block, vshape

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU: the HIP path has no CPU fallback")
    from paper_2311_15269_amd import binding
    binding.load_library()
    return binding


def fan(width, nr, cap, space="sampled_repair", lonely=False):
    """one stage feeds `width` stages on devices of their own, which feed one last stage; forward only where the cap is 0"""
    D = width + 2 + lonely
    deps = [(0, 1 + i) for i in range(width)] + [(1 + i, width + 1) for i in range(width)]
    return {"name": "fan-%d" % width, "D": D, "K": D, "NR": nr, "M": cap, "t": [1 + (3 * i) % 5 for i in range(D)], "m": [0] * D,
            "dev_mask": [1 << i for i in range(D)], "deps": deps, "space": space, "seed": 0xFA11 + width, "lead_step_q16": 25000,
            "fixed_leads": None}


def branch(nr, cap, space):
    """five stages on three devices, two of them a device but on the last: one feeds two, which feed one, which feeds the last"""
    return {"name": "branch", "D": 3, "K": 5, "NR": nr, "M": cap, "t": [2, 3, 1, 4, 2], "m": [1, 1, 0, -1, -1], "dev_mask": [1, 2, 4, 1, 2],
            "deps": [(0, 1), (0, 2), (1, 3), (2, 3), (3, 4)], "space": space, "seed": 0, "lead_step_q16": 0, "fixed_leads": None}


SHAPES = [
    ("three-producers-nr16", fan(3, 16, 0), 5, 700),             # all fields of a word with five-bit counts
    ("four-producers-nr16", fan(4, 16, 0), 5, 400),              # one too many: the general kernel
    ("four-producers-nr8", fan(4, 8, 0), 9, 700),
    ("four-producers-nr4-strict", fan(4, 4, 0, "sampled_strict"), 0, 3000),
    ("five-producers-nr4", fan(5, 4, 0), 9, 700),                # more consumers than the tables hold: the general kernel
    ("type-without-dependencies", fan(2, 3, 0, lonely=True), 3, 1000),
    ("odd-blocks", inference(9, 3), 11, 1500),
    ("odd-blocks-canonical", branch(3, 1, "canonical"), 0, 1 << 20),          # (the whole space)
    ("odd-blocks-canonical-roomy", branch(3, 3, "canonical"), 0, 1 << 20),
    ("nine-producers", fan(9, 3, 0), 6, 1500),                   # the best is decoded with all counts compared
    ("sixteen-producers-strict", fan(16, 1, 0, "sampled_strict"), 6, 1500),
    ("forward-only-two-passes", {"name": "two-passes", "D": 9, "K": 18, "NR": 3, "M": 0, "t": [1 + (5 * i) % 7 for i in range(18)],
                                 "m": [0] * 18, "dev_mask": [1 << (i % 9) for i in range(18)],
                                 "deps": [(i, i + 1) for i in range(17)], "space": "sampled_repair", "seed": 77,
                                 "lead_step_q16": 30000, "fixed_leads": None}, 1 << 33, 1500),
    ("shared-ten-fixed-leads", dict(shared_block(10, 2, 7), fixed_leads=[0] * 22), 3, 1500),
    ("kshape-one-micro-batch", W.kshape_problem(1, 3), 0, 500),
]


@pytest.mark.parametrize("name,prob,first,n", SHAPES, ids=[s[0] for s in SHAPES])
def test_edges_of_the_tables(gpu, name, prob, first, n):
    _compare(gpu, prob, first, n)


@pytest.mark.parametrize("n", [1, 63, 64, 65, 129, 191, 193])
def test_ranges_around_a_wave(gpu, n):
    _compare(gpu, vshape(9, 3, 4), 1 << 20, n)


def on_several_devices(rng):
    """a random graph of the other tests with some of its stages spread over several devices"""
    while True:
        prob = [random_graph_problem, random_wide_graph, random_crowded_graph][int(rng.integers(0, 3))](rng)
        masks, K = list(prob["dev_mask"]), prob["K"]
        for i in range(K // 2):
            if rng.random() < 0.3:
                masks[i] |= sum(1 << d for d in range(prob["D"]) if rng.random() < 0.4)
                masks[K - 1 - i] = masks[i]
        most = max(sum(m >> d & 1 for m in masks) for d in range(prob["D"]))
        if most <= 8 and most * prob["NR"] <= 32:
            return dict(prob, dev_mask=masks, M=prob["M"] + 2)


@pytest.mark.parametrize("seed", [61, 62, 63])
def test_random_graphs_with_blocks_on_several_devices(gpu, seed):
    rng = np.random.default_rng(seed)
    for case in range(8):
        _compare(gpu, on_several_devices(rng), int(rng.integers(0, 1 << 40)), int(rng.integers(500, 1500)))


def test_periods_left_to_the_general_kernel(gpu, monkeypatch):
    monkeypatch.setenv("TESSEL_DAG_TRIES", "0")
    for prob in (W.kshape_problem(3, 5), vshape(12, 2, 2), inference(32, 2)):
        _compare(gpu, prob, 4242, 1500)


def on_two(prob):
    """the first type on the first two devices, and a last type that gives its memory back there"""
    K = prob["K"]
    return dict(prob, K=K + 2, t=prob["t"] + [2, 3], m=prob["m"] + [1, -1], dev_mask=prob["dev_mask"] + [3, 3],
                deps=prob["deps"] + [(K, 0), (K - 1, K + 1)], name=prob["name"] + "-two")


EXHAUSTIVE = [(W.kshape_problem(nr, 2), space, at) for nr in (1, 2, 3) for space in ("canonical", "factorial") for at in (0.0, 0.5)]
EXHAUSTIVE += [(W.diamond_problem(2, 2), space, at) for space in ("canonical", "factorial") for at in (0.0, 0.6)]
EXHAUSTIVE += [(on_two(W.kshape_problem(nr, 4)), space, 0.3) for nr in (1, 2) for space in ("canonical", "factorial")]
EXHAUSTIVE += [(inference(9, 3), "factorial", 0.4), (inference(9, 2), "canonical", 0.0)]


@pytest.mark.parametrize("prob,space,at", EXHAUSTIVE, ids=["%s-nr%d-%s-%g" % (p["name"], p["NR"], s, a) for p, s, a in EXHAUSTIVE])
def test_exhaustive_spaces_on_both_sides_of_the_line(gpu, prob, space, at):
    """the graph kernel takes some of them and leaves the others to the general kernel; waves without a candidate left"""
    prob = dict(prob, space=space)
    count = gpu.Problem(prob).candidate_count()
    _compare(gpu, prob, int(count * at), 4000)


@pytest.mark.parametrize("tries", ["1", "8"])
@pytest.mark.parametrize("nr", [1, 2, 3])
@pytest.mark.parametrize("prob", [lambda nr: fan(2, nr, 0), lambda nr: fan(3, nr, 0), lambda nr: fan(4, nr, 0), lambda nr: W.kshape_problem(nr, nr + 1),
                                  lambda nr: W.diamond_problem(nr, nr + 1), lambda nr: vshape(9, nr, nr + 1), lambda nr: shared_block(9, nr, nr + 4)],
                         ids=["fan2", "fan3", "fan4", "kshape", "diamond", "chain", "shared"])
def test_values_of_a_window_boundary(gpu, monkeypatch, prob, nr, tries):
    """one, an odd and an even number of rings, a device or two more than the reads go by, windows of one to three micro-batches;
    with one sweep at first most periods are settled in the longer search"""
    monkeypatch.setenv("TESSEL_DAG_TRIES", tries)
    for space in ("sampled_repair", "sampled_strict"):
        _compare(gpu, dict(prob(nr), space=space), 77, 1100)
