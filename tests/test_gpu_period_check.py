"""tessel_best reports a period only if it is the least one of the decoded candidate's orders, worked out on the host without the
kernels' sweeps: a record whose period is one more or one less is refused, before and after the best has been read, for
every scoring kernel, for periods that a cycle takes exactly and for ratios rounded up; start times keep every constraint."""
import pytest

from oracle import Oracle
from paper_2311_15269_amd import workloads as W
from tests import schedule_checks as SC
from tests.test_gpu_wide import crowded, shared_block, vshape

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU: the HIP path has no CPU fallback")
    from paper_2311_15269_amd import binding
    binding.load_library()
    return binding


def ring(D, nr, t):
    """D chains of two blocks, the second of each on the device of the next chain's first: the cycle round all devices
    crosses a number of window boundaries that does not divide its time"""
    return {"name": "ring-%d" % D, "D": D, "K": 2 * D, "NR": nr, "M": 0, "t": [t + (7 * i) % 5 for i in range(2 * D)], "m": [0] * (2 * D),
            "dev_mask": [1 << ((c + k) % D) for c in range(D) for k in range(2)], "deps": [(2 * c, 2 * c + 1) for c in range(D)],
            "space": "sampled_repair", "seed": 0xD1CE + D, "lead_step_q16": 25000, "fixed_leads": None}


CASES = [W.config1(), W.config3(), W.config5(), dict(W.config4(), M=12), W.kshape_problem(4, 4), vshape(12, 2, 2), shared_block(10, 2, 7),
         crowded(3, 3, 3, 5), ring(3, 1, 3), ring(9, 2, 4), ring(32, 1, 2)]


@pytest.mark.parametrize("prob", CASES, ids=[p["name"] for p in CASES])
def test_a_wrong_period_is_refused(gpu, prob):
    import torch
    g = gpu.Problem(prob)
    n = 576 if prob["space"] == "factorial" else 4000

    def record():
        at = -g._ws.data_ptr() % 256
        return g._ws[at:at + 4].view(torch.int32)          # DevResult::period

    for by in (1, -1):
        g.reset()
        g.eval_candidates(0, n)
        right = int(record().item())
        record().fill_(right + by)
        with pytest.raises(gpu.TesselError) as err:
            g.best()
        assert err.value.code == -6                        # TESSEL_E_HIP
        record().fill_(right)
        got = g.best()
        assert got["feasible"] and got["period"] == right
        record().fill_(right + by)
        with pytest.raises(gpu.TesselError):
            g.best()
        record().fill_(right)
        assert g.best() == got
    cand = g.best_candidate()
    ref = Oracle(prob).eval_index(got["index"], want_starts=True)
    assert ref["period"] == right and (cand["starts"] == ref["starts"]).all()
    assert SC.check_periodic(prob, cand["leads"], cand["orders"], cand["starts"].tolist(), right)
