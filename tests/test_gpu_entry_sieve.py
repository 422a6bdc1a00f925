"""The fast kernel's look at the leads before anything else, on problems with blocks on several devices: candidates whose entry memory
alone exceeds the cap leave there, the others queue for the build.  Several rounds a wave (one workgroup a compute unit), ragged
ranges, caps that nearly all, some, few and none of the lead vectors exceed; against the oracle."""
import pytest

from tests.test_gpu_stage import on_some
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


SHAPES = [shared_block(4, 4, cap) for cap in (2, 4, 6, 8, 9, 100)] + [shared_block(2, 3, 5), shared_block(8, 4, 6), shared_block(7, 2, 4), on_some(4, 3, 4),
          on_some(8, 2, 4), dict(shared_block(4, 3, 4), fixed_leads=[2] * 5 + [0] * 5)]


@pytest.mark.parametrize("prob", SHAPES, ids=["%s-nr%d-cap%d%s" % (p["name"], p["NR"], p["M"], "-fixed" if p.get("fixed_leads") else "") for p in SHAPES])
def test_candidates_that_leave_by_their_leads(gpu, monkeypatch, prob):
    import torch
    from oracle import Oracle
    monkeypatch.setenv("TESSEL_BLOCKS_PER_CU", "1")
    lanes = 64 * torch.cuda.get_device_properties(0).multi_processor_count
    handle, oracle = gpu.Problem(prob), Oracle(prob)
    for first, count in ((12345, lanes + 1), (1 << 33, 3 * lanes + 77)):
        handle.reset()
        handle.eval_candidates(first, count)
        got, want = handle.best(), oracle.sweep(first, count)
        assert (got["n_evaluated"], got["n_feasible"], got["n_reject"][1:]) == (count, want["n_feasible"], want["n_reject"][1:])
        if want["n_feasible"]:
            assert (got["period"], got["index"], got["peak"]) == (want["period"], want["index"], want["peak"])
