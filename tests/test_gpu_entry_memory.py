"""Memory at the window entry (every type's lead times its memory delta) in the fast kernel: one to four types a device, deltas of both
signs up to what its 8-bit prefix holds, leads above zero, in the exhaustive spaces (sums of products) and the sampled ones (dot products)."""
import pytest

from tests.test_gpu_dag import _compare, gpu  # noqa: F401

pytestmark = pytest.mark.gpu


def _problem(mem, nr, cap, space):
    """`mem`: the deltas of every device's types; one chain through all types, device by device in turns"""
    order = [(d, y) for y in range(max(len(m) for m in mem)) for d in range(len(mem)) if y < len(mem[d])]
    K = len(order)
    return {"name": "entry", "D": len(mem), "K": K, "NR": nr, "M": cap, "t": [1 + (3 * i) % 4 for i in range(K)], "m": [mem[d][y] for d, y in order],
            "dev_mask": [1 << d for d, _ in order], "deps": [(i, i + 1) for i in range(K - 1)], "space": space, "seed": 5, "lead_step_q16": 30000,
            "fixed_leads": None}


MEM = [([[0], [7, -7]], 3, 9), ([[13, -7, 5, -11], [9, -9], [-20, 20]], 2, 14), ([[-3, 3], [1, 2, -3], [0], [4, -4]], 2, 7),
       ([[20, -20], [-19, 1, 18], [10, -10]], 2, 21), ([[1, -1]] * 8, 2, 2), ([[6, -6, 6, -6], [-5, 5, -5, 5]], 2, 9)]


@pytest.mark.parametrize("space", ["factorial", "canonical", "sampled_strict", "sampled_repair"])
@pytest.mark.parametrize("k", range(len(MEM)))
def test_entry_memory(gpu, k, space):  # noqa: F811
    from oracle import Oracle
    mem, nr, cap = MEM[k]
    prob = _problem(mem, nr, cap, space)
    count = Oracle(prob).count
    for first in sorted({0, 0 if count < 6000 else min(count, 1 << 40) // 7 * 3}):
        _compare(gpu, prob, first, 3000)
