"""The planner's store mode, on an MI355X, at row strides on and off 64-byte
sectors, against the other mode of the same plan (bitwise: the mode changes
only how a finished value is stored) and against the oracle: the sum, its
adjoint, the fused backward pass, and unpacking, out of place and in place.

Bars against the oracle: FP64 normwise 1e-14, FP32 2e-6 (on the FP32-rounded
input)."""
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
TOL = {F64: 1e-14, F32: 2e-6}

CASES = [
    # shape, group_first, d, dtype, store mode out of place
    ((3, 28, 28, 28), 1, 3, F64, 0),
    ((2, 34, 34, 34), 1, 3, F64, 0),
    ((2, 40, 40, 40), 1, 3, F64, 1),
    ((1, 60, 60, 60), 1, 3, F64, 0),
    ((2, 24, 24, 24, 5), 1, 3, F64, 0),
    ((3, 32, 32, 32), 1, 3, F32, 0),
    ((2, 134, 134), 1, 2, F64, 0),
    ((2, 160, 160), 1, 2, F64, 1),
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_store_modes(case):
    shape, gf, d, dtype, mode = CASES[case]
    terms = [(p, 0.5 + 0.25 * i) for i, p in enumerate(itertools.permutations(range(d)))]
    x = workloads.uniform(shape, 8800 + case, device=DEV, dtype=dtype)
    g = workloads.uniform(shape, 8900 + case, device=DEV, dtype=dtype)
    xh = x.cpu().to(F64).numpy()
    outs = []
    for flags in (0, ss.SPINSUM_FLAG_NO_NT_STORES if mode else ss.SPINSUM_FLAG_NT_STORES):
        for inplace in (False, True):
            p = ss.spinsum_plan(shape, gf, d, [terms], dtype=dtype, inplace=inplace, flags=flags)
            if not inplace:
                assert ss.spinsum_plan_get_info(p)["nt_stores"] == (1 - mode if flags else mode)
            y = x.clone() if inplace else torch.full_like(x, float("nan"))
            ss.spinsum_exec(p, y if inplace else x, y)
            a = g.clone() if inplace else torch.full_like(x, float("nan"))
            ss.spinsum_adjoint(p, a if inplace else g, a)
            b = g.clone() if inplace else torch.full_like(x, float("nan"))
            c = ss.spinsum_adjoint_coef_grad(p, x, b if inplace else g, b)
            u = torch.full_like(x, float("nan"))
            ss.spinsum_unpack(p, workloads.uniform(ss.packed_shape(p), 8700 + case, device=DEV,
                                                   dtype=dtype), u)
            outs.append((y, a, b, c, u))
    for other in outs[1:]:
        for have, want in zip(other, outs[0]):
            assert torch.equal(have, want)
    want = oracle.spinsum(xh, terms, gf, d, nthreads=8)
    have = outs[0][0].cpu().to(F64).numpy()
    assert np.linalg.norm(have - want) <= TOL[dtype] * np.linalg.norm(want)


@pytest.mark.parametrize("n,dtype", [(30, F64), (38, F64), (46, F64), (36, F32), (44, F32)])
def test_wide_tiles(n, dtype):
    """The wider tiles of the sum, bitwise against explicit 8^3 ones, forward
    and adjoint, out of place and in place."""
    shape = (3, n, n, n)
    terms = [(p, 0.5 + 0.25 * i) for i, p in enumerate(itertools.permutations(range(3)))]
    x = workloads.uniform(shape, 9100 + n, device=DEV, dtype=dtype)
    for inplace in (False, True):
        p = ss.spinsum_plan(shape, 1, 3, [terms], dtype=dtype, inplace=inplace)
        q = ss.spinsum_plan(shape, 1, 3, [terms], dtype=dtype, inplace=inplace)
        ss.spinsum_plan_set_tile(q, 8, variant=ss.SPINSUM_VARIANT_DIRECT_LDS)
        assert ss.spinsum_plan_get_info(p)["sum_bl"] > 8
        assert ss.spinsum_plan_get_info(q)["sum_bl"] == 0
        for run in (ss.spinsum_exec, ss.spinsum_adjoint):
            outs = []
            for plan in (p, q):
                y = x.clone() if inplace else torch.full_like(x, float("nan"))
                run(plan, y if inplace else x, y)
                outs.append(y)
            assert torch.equal(*outs)
