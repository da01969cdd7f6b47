"""The persistent whole-cube kernel (cubes of which one fits a CU, at least two
per CU) on an MI355X: bit for bit against the one-item-per-workgroup kernels
(SPINSUM_FLAG_NO_XCD_REMAP; both form every output as the same chain of fused
multiply-adds) and against the oracle on sampled cubes.  The extents leave
cubes that start on any element, ends of 0 to 3 elements, both numbers of
chunks per thread and uneven shares of cubes.

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
    # shape, d, dtype, inplace
    ((517, 24, 24, 24), 3, F64, True),
    ((517, 24, 24, 24), 3, F64, False),
    ((512, 26, 26, 26), 3, F64, True),      # more than 8 chunks a thread
    ((771, 25, 25, 25), 3, F64, False),     # cubes at odd elements
    ((513, 29, 29, 29), 3, F32, True),      # ends of one element
    ((514, 30, 30, 30), 3, F32, False),
    ((515, 31, 31, 31), 3, F32, True),      # ends of three
    ((520, 111, 111), 2, F64, True),
    ((512, 151, 151), 2, F32, False),
    ((519, 13, 13, 13, 5), 3, F64, False),  # inner runs
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_cube_kernel(case):
    shape, d, dtype, inplace = CASES[case]
    ident = tuple(range(d))
    forms = [
        ([[(p, 0.5 + 0.25 * i) for i, p in enumerate(itertools.permutations(range(d)))]], 0, False),
        # a permutation left out: non-finite inputs take the term-by-term path
        ([[(ident, 2.0), (ident[1:] + (0,), -0.5)]], ss.SPINSUM_FLAG_FULL_GROUP, True),
    ]
    if d == 3:
        forms.append((workloads.FACTORED_PIJ_PJK, ss.SPINSUM_FLAG_CHAIN_STAGES, False))
    sample = [0, 1, 255, 256, shape[0] - 1]
    for stages, flags, bad in forms:
        p = ss.spinsum_plan(shape, 1, d, stages, dtype=dtype, inplace=inplace, flags=flags)
        q = ss.spinsum_plan(shape, 1, d, stages, dtype=dtype, inplace=inplace,
                            flags=flags | ss.SPINSUM_FLAG_NO_XCD_REMAP)
        x = workloads.uniform(shape, 9500 + case, device=DEV, dtype=dtype)
        if bad:
            x.view(-1)[3] = float("inf")
            x.view(-1)[x.numel() - 1] = float("nan")
        for run, ref in ((ss.spinsum_exec, oracle.spinsum_chain),
                         (ss.spinsum_adjoint, oracle.spinsum_chain_adjoint)):
            outs = []
            for plan in (p, q):
                y = x.clone() if inplace else torch.empty_like(x)
                run(plan, y if inplace else x, y)
                outs.append(y)
            torch.cuda.synchronize()
            assert torch.equal(outs[0].isnan(), outs[1].isnan())
            assert torch.equal(outs[0].nan_to_num(nan=0.0, posinf=1e30, neginf=-1e30),
                               outs[1].nan_to_num(nan=0.0, posinf=1e30, neginf=-1e30))
            if not bad:
                want = ref(x[sample].cpu().to(F64).numpy(), stages, 1, d)
                got = outs[0][sample].cpu().to(F64).numpy()
                assert np.max(np.abs(got - want)) <= TOL[dtype] * np.max(np.abs(want))
