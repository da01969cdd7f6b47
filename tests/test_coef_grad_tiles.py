"""What a plan says of its coefficient gradient: coef_grad_split 1 wherever one
tensor is in LDS at a time, on the plan's tiles or on the gradient's own, and
the ownership check replays the gradient's own tiles too.  Host-only plans."""
import pytest
import torch

import workloads

ss = pytest.importorskip("paper_1705_06661_amd")
F64, F32 = torch.float64, torch.float32

CASES = [
    # shape, d, dtype, inplace, coef_grad_split
    ((600, 24, 24, 24), 3, F64, False, 1),  # whole cubes too large for both: own tiles
    ((600, 22, 22, 22), 3, F64, False, 1),  # ragged ones
    ((600, 26, 26, 26), 3, F64, False, 1),
    ((600, 100, 100), 2, F64, False, 1),
    ((600, 32, 32, 32), 3, F64, True, 1),   # the plan's tiles
    ((600, 16, 16, 16), 3, F64, False, 0),  # whole cubes, both tensors
    ((600, 25, 25, 25), 3, F64, False, 0),  # no rows of whole 16-byte chunks
    ((600, 32, 32, 32), 3, F32, False, 0),  # tiles of several chunks a thread
]


@pytest.mark.parametrize("shape,d,dtype,inplace,split", CASES)
def test_coef_grad_tiles(shape, d, dtype, inplace, split):
    p = ss.spinsum_plan(shape, 1, d, [workloads.antisymmetrizer(d)], dtype=dtype, inplace=inplace,
                        flags=ss.SPINSUM_FLAG_HOST_ONLY)
    assert p.info()["coef_grad_split"] == split
    assert ss.spinsum_plan_check_ownership(p) == (True, "")
