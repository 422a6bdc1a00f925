"""Periods of the fast kernel's longer search that are found although some values of the window boundary keep growing more slowly than
others: pipelines with a slow last device, forward-only ones, several chains, a block on several devices; scores against the oracle, with the usual first search
and with one of a single sweep, which leaves nearly all candidates to the longer one."""
import pytest

from paper_2311_15269_amd import workloads as W
from tests.test_gpu_dag import _compare
from tests.test_gpu_ranked import forward
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


def slow_end(D, nr, cap, space="sampled_repair"):
    return W.pipeline_problem(W.linear_placement(D), [1 + i for i in range(D)], [2 + 2 * i for i in range(D)], D, nr, cap, space, seed=5, lead_step_q16=20000)


def sampled(prob, step):
    return dict(prob, space="sampled_repair", seed=11, lead_step_q16=step)


SHAPES = [slow_end(2, 2, 3), slow_end(4, 4, 5), slow_end(5, 7, 7), slow_end(8, 8, 9), slow_end(3, 3, 4, "sampled_strict"), sampled(forward(8, 1, 8), 20000),
          sampled(forward(4, 2, 4), 9000), sampled(forward(2, 4, 3), 30000), W.xshape_problem(3, 2, 5, 2, 4), shared_block(4, 3, 100)]


@pytest.mark.parametrize("tries", [None, "1"])
@pytest.mark.parametrize("prob", SHAPES, ids=["%s-%ddev-nr%d-%d" % (p["name"], p["D"], p["NR"], k) for k, p in enumerate(SHAPES)])
def test_periods(gpu, monkeypatch, prob, tries):
    if tries:
        monkeypatch.setenv("TESSEL_EIGEN_TRIES", tries)
    _compare(gpu, prob, 4321, 3000)
