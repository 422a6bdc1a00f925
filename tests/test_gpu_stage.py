"""The fast kernel's first build phase on problems with blocks on several devices, whose length goes by the rounds of
candidates a wave has, and which long launches find from their own first candidates: the same best candidate and counts as with every length forced, and as the oracle on the
start of the range; blocks on all devices and on some of them."""
import pytest

from paper_2311_15269_amd import workloads as W
from tests.test_gpu_dag import _compare
from tests.test_gpu_wide import shared_block

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU: the HIP path has no CPU fallback")
    from paper_2311_15269_amd import binding
    binding.load_library()
    return binding


def on_some(D, nr, cap):
    """the block around the pipeline on the first two devices only"""
    prob = shared_block(D, nr, cap)
    return dict(prob, dev_mask=[3] + prob["dev_mask"][1:-1] + [3], name="some-%d" % D)


# tight and wide caps; strict: deadlocks instead of the cap
SHAPES = [shared_block(2, 2, 4), shared_block(2, 4, 11), shared_block(4, 4, 6), shared_block(4, 2, 100), shared_block(7, 4, 9),
          shared_block(8, 2, 4), shared_block(3, 2, 9, space="sampled_strict"), on_some(4, 3, 8), on_some(8, 2, 100)]


@pytest.mark.parametrize("prob", SHAPES, ids=["%s-nr%d-cap%d-%s" % (p["name"], p["NR"], p["M"], p["space"]) for p in SHAPES])
def test_lengths_of_the_first_phase(gpu, monkeypatch, prob):
    _compare(gpu, prob, 1 << 30, 1500)
    n, words = 7000000, (prob["K"] * prob["NR"] + 5) // 6      # enough rounds for the waves to choose (24 of 16 waves a CU)

    def best():
        g = gpu.Problem(prob)
        g.eval_candidates(7, n)
        r = g.best()
        return {k: r[k] for k in ("period", "index", "peak", "n_evaluated", "n_feasible", "n_reject")}
    want = best()
    assert want["n_evaluated"] == n
    for length in sorted({1, 2, words // 2, words} - {0}):
        monkeypatch.setenv("TESSEL_STAGE_WORDS", str(length))
        assert best() == want


@pytest.mark.parametrize("prob", [shared_block(8, 4, 6), on_some(8, 4, 9), shared_block(4, 3, 6), shared_block(8, 4, 6, space="sampled_strict")],
                         ids=lambda p: "%s-nr%d-cap%d-%s" % (p["name"], p["NR"], p["M"], p["space"]))
def test_lengths_by_rounds(gpu, monkeypatch, prob):
    """launches of half a round to eleven rounds: the same as in one phase"""
    for n in (100001, 200003, 300007, 420001, 2100001):
        got = []
        for whole in (False, True):
            if whole:
                monkeypatch.setenv("TESSEL_STAGE_WORDS", str((prob["K"] * prob["NR"] + 5) // 6))
            else:
                monkeypatch.delenv("TESSEL_STAGE_WORDS", raising=False)
            g = gpu.Problem(prob)
            g.eval_candidates(1 << 31, n)
            r = g.best()
            got.append([r[k] for k in ("period", "index", "peak", "n_evaluated", "n_feasible", "n_reject")])
        assert got[0] == got[1] and got[0][3] == n


@pytest.mark.parametrize("D", [4, 5, 8])
def test_scores_by_rounds(gpu, monkeypatch, D):
    """scores and peaks of launches that end with a nearly empty and with a nearly full round: the same as in one phase"""
    prob = W.pipeline_problem(W.folded_placement(D), [1 + (3 * i) % 4 for i in range(2 * D)], [2 + (5 * i) % 7 for i in range(2 * D)],
                              D, 4, 6, "sampled_repair", seed=9, lead_step_q16=8000)
    g = gpu.Problem(prob)
    for n in (200003, 262144, 300007, 470009):
        monkeypatch.delenv("TESSEL_STAGE_WORDS", raising=False)
        code, peak = g.score_candidates(12345, n)
        for words in (4, (prob["K"] * 4 + 5) // 6):
            monkeypatch.setenv("TESSEL_STAGE_WORDS", str(words))
            c, p = g.score_candidates(12345, n)
            assert bool((c == code).all()) and bool((p == peak).all())
