"""The best candidate as the host decodes it from its index, against the oracle candidate by candidate: one to eight types a device, the most and
nearly the most devices, micro-batches and producers, blocks on several devices, every space, fixed leads."""
import numpy as np
import pytest

from paper_2311_15269_amd import workloads as W
from tests.test_gpu_dag import gpu  # noqa: F401
from tests.test_gpu_graph_kernel import fan, on_two
from tests.test_gpu_wide import crowded, inference, shared_block, vshape

pytestmark = pytest.mark.gpu


def folded(D, nr, cap):
    return W.pipeline_problem(W.folded_placement(D), [1 + i % 3 for i in range(2 * D)], [2 + i % 4 for i in range(2 * D)], D, nr, cap,
                              "sampled_repair", seed=78, lead_step_q16=6000, name="folded-%d" % D)


def three_on_one(D, nr, space="sampled_repair"):
    """a forward-only pipeline whose last two stages sit on device 0 as well"""
    prob = inference(D, nr, space)
    K = D + 2
    return dict(prob, name="three-on-one-%d" % D, K=K, t=prob["t"] + [2, 3], m=[0] * K, dev_mask=prob["dev_mask"] + [1, 1],
                deps=[(i, i + 1) for i in range(K - 1)])


SHAPES = [inference(1, 4), inference(32, 16), vshape(16, 8, 12), vshape(17, 3, 6), vshape(32, 16, 40), folded(8, 8, 10), folded(9, 2, 9),
          folded(16, 8, 30), crowded(4, 4, 4, 20, step=3000), crowded(8, 4, 4, 30, step=1000), crowded(8, 3, 2, 30, step=1000), three_on_one(16, 9),
          three_on_one(17, 9), three_on_one(17, 2, "sampled_strict"), fan(4, 16, 0), fan(5, 4, 0), shared_block(8, 4, 14), shared_block(16, 4, 100),
          shared_block(17, 2, 100), on_two(crowded(3, 3, 3, 30, step=1000)), W.kshape_problem(4, 6), W.diamond_problem(3, 8),
          vshape(3, 3, 6, "canonical"), vshape(2, 8, 9, "canonical"), vshape(9, 1, 3, "canonical"), vshape(9, 1, 3, "factorial"),
          dict(vshape(12, 9, 30), fixed_leads=[0] * 24)]


@pytest.mark.parametrize("prob", SHAPES, ids=["%s-nr%d-%s" % (p["name"], p["NR"], p["space"]) for p in SHAPES])
def test_decoded_candidates(gpu, prob):  # noqa: F811
    from oracle import Oracle
    orc, g = Oracle(prob), gpu.Problem(prob)
    rng = np.random.default_rng(9)
    space = min(orc.count, 1 << 40)
    chosen = [0, space - 1] + [int(x) for x in rng.integers(0, space, 12)]
    if space < 1 << 20:                       # exhaustive: most are rejected
        chosen = [i for i in range(space) if orc.eval_index(i)["status"] == 0][:: max(1, space // 4000)]
    seen = 0
    for i in chosen:
        want = orc.eval_index(i, want_starts=True)
        g.reset()
        g.eval_candidates(i, 1)
        got = g.best()
        assert got["feasible"] == (want["status"] == 0), i
        if not got["feasible"]:
            continue
        seen += 1
        assert (got["period"], got["peak"]) == (want["period"], list(want["peak"])[:prob["D"]]), i
        _, leads, orders = orc.decode(i)
        c = g.best_candidate()
        assert c["leads"] == list(leads) and c["orders"] == orders and (c["starts"] == want["starts"]).all(), i
    if prob["space"] == "sampled_repair":
        assert seen > 0, prob["name"]
