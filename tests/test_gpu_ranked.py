"""The CANONICAL space on the fast kernel, element by element against the oracle, on both sides of the lines at which its
decode changes: indices below and from 2^32 on (digits by 32-bit reciprocals or by 64-bit divisions), and spaces whose
orders or lead vectors are too many for the tables by rank (unranked symbol by symbol)."""
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


def linear(D, nr, cap):
    return W.pipeline_problem(W.linear_placement(D), [1 + i % 2 for i in range(D)], [2 + i % 3 for i in range(D)], D, nr, cap, "canonical")


def forward(D, chains, nr):
    """forward-only chains, each with a stage on every device, the second in the other direction and so on"""
    K = D * chains
    return {"name": "forward", "D": D, "K": K, "NR": nr, "M": 0, "t": [1 + (3 * i) % 5 for i in range(K)], "m": [0] * K,
            "dev_mask": [1 << (i if c % 2 == 0 else D - 1 - i) for c in range(chains) for i in range(D)],
            "deps": [(c * D + i, c * D + i + 1) for c in range(chains) for i in range(D - 1)], "space": "canonical",
            "seed": 0, "lead_step_q16": 0, "fixed_leads": None}


def rounds(D, per, nr):
    """one forward-only chain that passes every device `per` times"""
    K = D * per
    return {"name": "rounds", "D": D, "K": K, "NR": nr, "M": 0, "t": [1 + (3 * i) % 5 for i in range(K)], "m": [0] * K,
            "dev_mask": [1 << (i % D) for i in range(K)], "deps": [(i, i + 1) for i in range(K - 1)], "space": "canonical",
            "seed": 0, "lead_step_q16": 0, "fixed_leads": None}


LEADS = [5, 3, 1, 0, 5, 2, 1, 1]                             # most orders around index 2^32 can execute
CASES = [("below-2^32", dict(forward(4, 2, 6), fixed_leads=LEADS), (1 << 32) - 4000),
         ("across-2^32", dict(forward(4, 2, 6), fixed_leads=LEADS), (1 << 32) - 2000),
         ("above-2^32", dict(forward(4, 2, 6), fixed_leads=LEADS), 1 << 32),
         ("five-devices-below-2^32", linear(5, 4, 6), (1 << 32) - 9000), ("five-devices-above-2^32", linear(5, 4, 6), 284464890000),
         ("12870-orders", linear(2, 8, 9), 3528919000), ("12870-orders-above-2^32", linear(2, 8, 8), 19000000000),
         ("34650-orders", rounds(2, 3, 4), 1232711000), ("34650-orders-above-2^32", rounds(2, 3, 4), 60000000000),
         ("369600-orders", rounds(2, 4, 3), 2635465720000), ("3675-leads", forward(4, 2, 5), 9262186229000),
         ("10976-leads", forward(4, 2, 6), 40), ("10976-leads-above-2^32", forward(4, 2, 6), 7786107047306000)]


@pytest.mark.parametrize("name,prob,first", CASES, ids=[c[0] for c in CASES])
def test_canonical_decode(gpu, name, prob, first):
    _compare(gpu, prob, first, 4000)
