"""Which problems the graph kernel builds on masks by code, on the host: a problem that it would leave to the general kernel if it had no words by
type (TESSEL_GRAPH_WORDS=0) needs another workspace then.  The shapes of the GPU test, and one beyond every limit of the rule."""
import pytest

from paper_2311_15269_amd import binding, workloads as W
from tests.test_gpu_chain_codes import SHAPES
from tests.test_gpu_wide import crowded, shared_block, vshape

BY_TYPE = {"vshape-10-m572", "crowded-4x3-m3", "vshape-10-t23", "vshape-10-twice"}       # memory, end times, a doubled dependency
CASES = [(p, p["name"] not in BY_TYPE) for p, _ in SHAPES]
CASES += [(crowded(8, 4, 2, 9), True), (crowded(9, 3, 2, 9), False),                       # 64 and 72 codes
          (vshape(9, 2, 4, space="canonical"), False), (shared_block(9, 2, 9), False), (W.kshape_problem(4, 4), False)]


@pytest.mark.parametrize("prob,codes", CASES, ids=["%s-nr%d-%s" % (p["name"], p["NR"], p["space"]) for p, _ in CASES])
def test_rule(monkeypatch, prob, codes):
    def workspace(words):
        if words is None:
            monkeypatch.delenv("TESSEL_GRAPH_WORDS", raising=False)
        else:
            monkeypatch.setenv("TESSEL_GRAPH_WORDS", words)
        return binding.Problem(prob).workspace_bytes()
    monkeypatch.setenv("TESSEL_FORCE_GENERAL", "1")
    general = workspace(None)
    monkeypatch.delenv("TESSEL_FORCE_GENERAL")
    assert workspace(None) != general                            # the graph kernel takes it, one way or the other
    assert (workspace(None) == workspace("0")) == codes
    assert codes or workspace(None) == workspace("1")


def test_the_cases_stand_at_the_limits():
    assert BY_TYPE <= {p["name"] for p, _ in SHAPES}
