"""The fast kernel's variants by devices and boundary values: two, four and eight devices with the most values of one variant and the
fewest of the next (4 and 5, 8 and 9, 16 and 17), with and without repair and in the exhaustive spaces; scores against the oracle."""
import pytest

from paper_2311_15269_amd import workloads as W
from tests.test_gpu_dag import _compare, gpu  # noqa: F401
from tests.test_gpu_ranked import forward

pytestmark = pytest.mark.gpu
# devices, chains, micro-batches: boundary values = devices + chains * micro-batches
SIZES = [(2, 1, 2), (2, 1, 3), (2, 2, 7), (2, 3, 5), (4, 1, 4), (4, 1, 5), (3, 1, 6), (4, 2, 6), (4, 2, 7), (8, 1, 8), (7, 2, 5), (5, 2, 6)]


@pytest.mark.parametrize("space", ["sampled_repair", "sampled_strict", "canonical"])
@pytest.mark.parametrize("D,chains,nr", SIZES)
def test_variants(gpu, D, chains, nr, space):  # noqa: F811
    prob = dict(forward(D, chains, nr), space=space, seed=3, lead_step_q16=20000)
    prob["t"] = [1 + (7 * i * i + 3 * i) % 11 for i in range(prob["K"])]
    if space == "canonical":
        prob["fixed_leads"] = [1 if i % D == 0 else 0 for i in range(prob["K"])]
    _compare(gpu, prob, 12345 if space != "canonical" else 0, 2500)


@pytest.mark.parametrize("p,nr", [(2, 1), (2, 2), (3, 3), (4, 2), (4, 3), (4, 4)])
def test_two_ways(gpu, p, nr):  # noqa: F811
    _compare(gpu, W.xshape_problem(p, 2, 5, nr, nr + 2), 777, 4000)
