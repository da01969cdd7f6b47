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
    ((600, 128, 128), 2, F32, False, 0),    # own tiles of both tensors
    ((600, 148, 148), 2, F32, True, 0),
    ((600, 160, 160), 2, F32, False, 0),
]


@pytest.mark.parametrize("shape,d,dtype,inplace,split", CASES)
def test_coef_grad_tiles(shape, d, dtype, inplace, split):
    p = ss.spinsum_plan(shape, 1, d, [workloads.antisymmetrizer(d)], dtype=dtype, inplace=inplace,
                        flags=ss.SPINSUM_FLAG_HOST_ONLY)
    assert p.info()["coef_grad_split"] == split
    assert ss.spinsum_plan_check_ownership(p) == (True, "")


@pytest.mark.gpu
@pytest.mark.parametrize("n,inplace", [(128, False), (132, True), (148, False), (160, True)])
def test_both_gradients_on_own_tiles_of_both_tensors(n, inplace):
    """2D FP32 cubes too large for both tensors: the adjoint's bits, and
    coefficients within 1e-12 of sum |g| |x|, the bound of each."""
    import numpy as np
    import oracle
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    shape = (5, n, n)
    terms = [[((0, 1), 2.0), ((1, 0), -0.75)]]
    p = ss.spinsum_plan(shape, 1, 2, terms, dtype=F32, inplace=inplace)
    dev = torch.device("cuda:0")
    x = workloads.uniform(shape, 9800, device=dev, dtype=F32)
    g = workloads.uniform(shape, 9801, device=dev, dtype=F32)
    want = g.clone() if inplace else torch.empty_like(g)
    ss.spinsum_adjoint(p, want if inplace else g, want)
    got = g.clone() if inplace else torch.empty_like(g)
    c = ss.spinsum_adjoint_coef_grad(p, x, got if inplace else g, got)
    alone = ss.spinsum_coef_grad(p, x, g)
    torch.cuda.synchronize()
    assert torch.equal(got, want)
    xh, gh = x.cpu().to(F64).numpy(), g.cpu().to(F64).numpy()
    ref = oracle.coef_grad(xh, gh, 1, 2)
    for have in (c, alone):
        assert np.max(np.abs(have.cpu().numpy() - ref)) <= 1e-12 * np.sum(np.abs(xh)) * np.max(np.abs(gh))
