"""The grid of a scoring launch is one that the chip holds at once, on the host: a compute unit gives LDS out in pieces of 1,280 bytes, so that of workgroups
with 12,288 bytes it holds 12.  The workspace has room for the queues of every workgroup of the grid, which tells how many there are."""
from paper_2311_15269_amd import binding

# 30 blocks, ten of them on two of three devices: 2,048 + 1,536 bytes of tables, 4,096 of records, 4,608 of times and counters a workgroup
PROBLEM = {"name": "two-on-two", "D": 3, "K": 6, "NR": 5, "M": 12, "t": [1, 2, 1, 8, 5, 3], "m": [1, 1, 1, -1, -1, -1], "dev_mask": [5, 1, 4, 4, 1, 5],
           "deps": [(i, i + 1) for i in range(5)], "space": "sampled_repair", "seed": 723441678, "lead_step_q16": 38757, "fixed_leads": None}


def test_workgroups_of_twelve_kilobytes(monkeypatch):
    def workspace(most):
        if most is None:
            monkeypatch.delenv("TESSEL_BLOCKS_PER_CU", raising=False)
        else:
            monkeypatch.setenv("TESSEL_BLOCKS_PER_CU", str(most))
        return binding.Problem(PROBLEM).workspace_bytes()
    assert workspace(11) < workspace(12) == workspace(None)
