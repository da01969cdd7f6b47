"""spinsum_adjoint_coef_grad (both gradients of a backward pass from one read
of the upstream gradient) on an MI355X: the tensor's gradient bit for bit that
of spinsum_adjoint, the coefficients' within the order of summation of
spinsum_coef_grad's and against the oracle.  The plans take each kernel: whole
cubes at both workgroup sizes, the plan's tiles with one and with two tensors
in LDS, tiles of the gradient's own, and the forms that run two launches.

Bars: coefficient gradients 1e-12 relative to the largest (1e-12 as well in
FP32: the sums are formed in double on the same FP32 values)."""
import itertools

import numpy as np
import pytest
import torch

import oracle
import workloads

pytestmark = pytest.mark.gpu

ss = pytest.importorskip("paper_1705_06661_amd")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

DEV = torch.device("cuda:0")
F64, F32 = torch.float64, torch.float32

CASES = [
    # shape, d, dtype, inplace, flags
    ((5, 8, 8, 8), 3, F64, False, 0),          # whole cubes
    ((3, 16, 16, 16), 3, F64, True, 0),
    ((3, 20, 20, 20), 3, F64, False, 0),       # one pair per CU
    ((2, 24, 24, 24), 3, F32, False, 0),
    ((2, 32, 32, 32), 3, F64, True, 0),        # tiles, one tensor in LDS
    ((2, 36, 36, 36), 3, F64, False, 0),       # ragged tiles
    ((2, 24, 24, 24), 3, F64, False, 0),       # the gradient's own tiles
    ((2, 22, 22, 22), 3, F64, False, 0),       # ragged ones
    ((2, 32, 32, 32), 3, F32, False, 0),       # two tensors in LDS, packed orbits
    ((2, 16, 16, 16, 8), 3, F64, False, 0),    # inner runs
    ((3, 33, 33), 2, F64, False, 0),
    ((2, 140, 140), 2, F64, True, 0),
    ((2, 6, 6, 6, 6), 4, F64, False, 0),       # two launches: 4D, stages, a subgroup
    ((3, 12, 12, 12), 3, F64, False, "chain"),
    ((3, 12, 12, 12), 3, F64, True, "multi"),
    ((3, 12, 12, 12), 3, F64, False, "sub"),
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_adjoint_coef_grad(case):
    shape, d, dtype, inplace, form = CASES[case]
    stages = [[(p, 0.5 + 0.25 * i) for i, p in enumerate(itertools.permutations(range(d)))]]
    flags = 0
    if form == "chain":
        stages, flags = workloads.FACTORED_PIJ_PJK, ss.SPINSUM_FLAG_CHAIN_STAGES
    elif form == "multi":
        stages, flags = workloads.FACTORED_PIJ_PJK, ss.SPINSUM_FLAG_MULTI_PASS
    elif form == "sub":
        stages = [[((0, 1, 2), 2.0), ((1, 0, 2), -1.0)]]
    ident = tuple(range(d))
    for bad in (False, True) if form == 0 else (False,):
        if bad:  # zero coefficients: non-finite gradients reach the terms' outputs alone
            stages, flags = [[(ident, 2.0), (ident[1:] + (0,), -0.5)]], ss.SPINSUM_FLAG_FULL_GROUP
        p = ss.spinsum_plan(shape, 1, d, stages, dtype=dtype, inplace=inplace, flags=flags)
        x = workloads.uniform(shape, 9700 + case, device=DEV, dtype=dtype)
        g = workloads.uniform(shape, 9800 + case, device=DEV, dtype=dtype)
        if bad:
            g.view(-1)[7] = float("inf")
            g.view(-1)[g.numel() - 3] = float("nan")
        want = g.clone() if inplace else torch.empty_like(g)
        ss.spinsum_adjoint(p, want if inplace else g, want)
        c0 = ss.spinsum_coef_grad(p, x, g)
        got = g.clone() if inplace else torch.full_like(g, 3.0)
        c1 = ss.spinsum_adjoint_coef_grad(p, x, got if inplace else g, got)
        torch.cuda.synchronize()
        assert torch.equal(got.isnan(), want.isnan())
        assert torch.equal(got.nan_to_num(nan=0.0, posinf=1e30, neginf=-1e30),
                           want.nan_to_num(nan=0.0, posinf=1e30, neginf=-1e30))
        if bad:
            continue
        ref = oracle.coef_grad(x.cpu().to(F64).numpy(), g.cpu().to(F64).numpy(), 1, d)
        for c in (c0, c1):
            assert np.max(np.abs(c.cpu().numpy() - ref)) <= 1e-12 * np.max(np.abs(ref))


def test_adjoint_coef_grad_refusals():
    shape = (3, 33, 33, 33)  # rows that are not whole 16-byte chunks
    p = ss.spinsum_plan(shape, 1, 3, [workloads.CONFIG_3D_ALPHA])
    x = torch.zeros(shape, dtype=F64, device=DEV)
    g, gx = torch.zeros_like(x), torch.zeros_like(x)
    with pytest.raises(ss.SpinSumError) as e:
        ss.spinsum_adjoint_coef_grad(p, x, g, gx)
    assert e.value.status == ss.SPINSUM_ERR_UNSUPPORTED
    shape = (3, 8, 8, 8)
    p = ss.spinsum_plan(shape, 1, 3, [workloads.CONFIG_3D_ALPHA])
    x = torch.zeros(shape, dtype=F64, device=DEV)
    g = torch.zeros_like(x)
    for a, b, c in ((x, g, g), (x, g, x)):  # gx over g, gx over x
        with pytest.raises(ss.SpinSumError) as e:
            ss.spinsum_adjoint_coef_grad(p, a, b, c)
        assert e.value.status == ss.SPINSUM_ERR_ALIASING
