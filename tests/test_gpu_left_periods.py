"""Problems whose periods the graph kernel's sweeps do not settle, so that all or many of their candidates are left to the
general kernel: chains of two blocks round a ring of devices.  Element by element against the oracle; more of them in one
launch than its list holds, in both workspaces and replayed from a graph after a reset, against launches that fit."""
import pytest

from tests.test_gpu_dag import _compare
from tests.test_gpu_period_check import ring

pytestmark = pytest.mark.gpu
KEYS = ("period", "index", "peak", "peak_max", "n_evaluated", "n_feasible", "n_reject", "feasible")
LISTED = 1 << 20                                           # candidates a launch's list holds


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU: the HIP path has no CPU fallback")
    from paper_2311_15269_amd import binding
    binding.load_library()
    return binding


@pytest.mark.parametrize("prob", [ring(32, 1, 2), ring(16, 2, 9), ring(9, 4, 3), ring(10, 5, 40)], ids=lambda p: "%s-nr%d" % (p["name"], p["NR"]))
def test_rings(gpu, prob):
    _compare(gpu, prob, 1 << 35, 1500)


def test_more_than_the_list_holds(gpu):
    import torch
    prob, first, n = ring(32, 1, 2), 99, LISTED + 70
    g = gpu.Problem(prob)
    for k in range(2):
        g.eval_candidates(first + k * (n // 2), n // 2)
    want = {k: v for k, v in g.best().items() if k in KEYS}
    assert want["n_evaluated"] == n and want["n_feasible"] == n

    def best(h):
        return {k: v for k, v in h.best().items() if k in KEYS}
    h = gpu.Problem(prob)
    h.eval_candidates(first, n)
    assert best(h) == want
    h.reset()
    h.eval_candidates_noalloc(first, n)
    assert best(h) == want
    h = gpu.Problem(prob)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        h.eval_candidates(0, 64)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            h.eval_candidates(first, n)
        for _ in range(3):
            h.reset()
            graph.replay()
            assert best(h) == want
    stream.synchronize()
