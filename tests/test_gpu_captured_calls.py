"""Scoring calls captured once in a HIP graph and replayed: the running best changes in the workspace without a host call
of the library, and every question about it has to see that.  Two ranges, each captured as a search of its own (reset and
score) and one as a continuation, replayed in turns with eager calls between; each answer against the one of eager calls."""
import pytest

from paper_2311_15269_amd import workloads as W

pytestmark = pytest.mark.gpu
KEYS = ("period", "index", "peak", "peak_max", "n_evaluated", "n_feasible", "n_reject", "feasible")
# a problem of each scoring kernel and two ranges of its space with a best candidate each
CASES = [("fast", W.config5(), ((0, 20000), (1 << 21, 30000))),
         ("canonical", W.config2(), ((0, 20000), (1063390000, 30000))),
         ("graph", W.kshape_problem(4, 4), ((0, 20000), (1 << 21, 30000)))]


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU: the HIP path has no CPU fallback")
    from paper_2311_15269_amd import binding
    binding.load_library()
    return binding


def _answers(g):
    best = g.best()
    out = {k: best[k] for k in KEYS}
    if best["feasible"]:
        c = g.best_candidate()
        out["candidate"] = (c["leads"], c["orders"], c["starts"].tolist())
    return out


@pytest.mark.parametrize("noalloc", [False, True], ids=["workspace", "noalloc"])
@pytest.mark.parametrize("name,prob,ranges", CASES, ids=[c[0] for c in CASES])
def test_replayed_searches_are_seen(gpu, name, prob, ranges, noalloc):
    import torch

    def score(g, first, n):
        (g.eval_candidates_noalloc if noalloc else g.eval_candidates)(first, n)

    want = []
    for first, n in ranges:
        g = gpu.Problem(prob)
        score(g, first, n)
        want.append(_answers(g))
    assert want[0]["index"] != want[1]["index"]
    g = gpu.Problem(prob)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        score(g, 5, 100)                                   # (binds the workspace: uploads stay out of the graphs)
        g.best()
        graphs = []
        for first, n in ranges:
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=stream):
                g.reset()
                score(g, first, n)
            graphs.append(graph)
        more = torch.cuda.CUDAGraph()
        with torch.cuda.graph(more, stream=stream):
            score(g, *ranges[1])
        for turn in (0, 1, 1, 0, 1, 0):
            graphs[turn].replay()
            assert _answers(g) == want[turn], turn
        for turn in range(3):                              # the search goes on: counters add up, the better of the two stays
            more.replay()
            got = _answers(g)
            assert got["n_evaluated"] == ranges[0][1] + (turn + 1) * ranges[1][1]
            assert (got["period"], got["index"]) == min((w["period"], w["index"]) for w in want)
        g.reset()                                          # eager work between replays
        score(g, *ranges[1])
        assert _answers(g) == want[1]
        graphs[0].replay()
        assert _answers(g) == want[0]
    stream.synchronize()
