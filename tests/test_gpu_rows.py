"""Parity, on an MI355X, of the kernel for tile rows that start on any element
(extents whose rows are not whole 16-byte chunks, spinsum_plan_info_t.sum_bl):
bitwise against the register kernel on an explicit tile (both form every
output as the same chain of fused multiply-adds) and against the oracle.  The
extents leave every possible end of a row, a last block of one element, and
blocks that divide the extent.

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
    # shape, group_first, d, dtype, an explicit register tile
    ((3, 33, 33, 33), 1, 3, F64, 7),      # last block of one element
    ((2, 35, 35, 35), 1, 3, F64, 7),
    ((2, 33, 33, 33), 1, 3, F32, 9),      # ends of 1, 2 and 3 elements
    ((2, 34, 34, 34), 1, 3, F32, 8),
    ((2, 39, 39, 39), 1, 3, F32, 9),
    ((2, 27, 27, 27, 3), 1, 3, F64, 5),   # inner runs
    ((2, 3, 11, 11, 11, 11), 2, 4, F64, 3),
    ((1, 13, 13, 13, 13), 1, 4, F64, 3),
    ((2, 13, 13, 13, 13), 1, 4, F32, 3),  # 16-byte rows
    ((1, 14, 14, 14, 14), 1, 4, F32, 2),
    ((3, 151, 151), 1, 2, F64, 31),
    ((2, 301, 301), 1, 2, F32, 41),
]


def stages_of(d, sparse):
    if sparse:  # a permutation left out, so non-finite inputs take the term-by-term path
        ident = tuple(range(d))
        return [[(ident, 2.0), ((1, 0) + ident[2:], -0.75), (ident[1:] + (0,), 0.5)]]
    return [[(p, 0.5 + 0.25 * i) for i, p in enumerate(itertools.permutations(range(d)))]]


@pytest.mark.parametrize("case", range(len(CASES)))
@pytest.mark.parametrize("flags", [0, ss.SPINSUM_FLAG_NT_STORES | ss.SPINSUM_FLAG_REVERSE_ORDER])
def test_rows_kernel_against_register_kernel_and_oracle(case, flags):
    shape, gf, d, dtype, bl = CASES[case]
    inplace = case % 2 == 0
    flags |= ss.SPINSUM_FLAG_FULL_GROUP
    for sparse in (False, True):
        stages = stages_of(d, sparse)
        p = ss.spinsum_plan(shape, gf, d, stages, dtype=dtype, inplace=inplace, flags=flags)
        assert ss.spinsum_plan_get_info(p)["sum_bl"] > 0
        q = ss.spinsum_plan(shape, gf, d, stages, dtype=dtype, inplace=inplace, flags=flags)
        ss.spinsum_plan_set_tile(q, bl, variant=ss.SPINSUM_VARIANT_REG_ONESHOT)
        assert ss.spinsum_plan_get_info(q)["sum_bl"] == 0
        x = workloads.uniform(shape, 8100 + case, device=DEV, dtype=dtype)
        if sparse:
            x.view(-1)[5] = float("inf")
            x.view(-1)[x.numel() - 2] = float("nan")
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
            if not sparse:
                want = ref(x.cpu().to(F64).numpy(), stages, gf, d)
                got = outs[0].cpu().to(F64).numpy()
                assert np.max(np.abs(got - want)) <= TOL[dtype] * np.max(np.abs(want))


def test_rows_kernel_chained_stages():
    """Chained stages and one launch per stage on the same tiles."""
    shape = (2, 33, 33, 33)
    x = workloads.uniform(shape, 8200, device=DEV)
    want = oracle.spinsum_chain(x.cpu().numpy(), workloads.FACTORED_PIJ_PJK, 1, 3)
    for flags in (ss.SPINSUM_FLAG_CHAIN_STAGES, ss.SPINSUM_FLAG_MULTI_PASS):
        p = ss.spinsum_plan(shape, 1, 3, workloads.FACTORED_PIJ_PJK, flags=flags)
        assert ss.spinsum_plan_get_info(p)["sum_bl"] > 0
        y = torch.empty_like(x)
        ss.spinsum_exec(p, x, y)
        torch.cuda.synchronize()
        got = y.cpu().numpy()
        assert np.max(np.abs(got - want)) <= 1e-14 * np.max(np.abs(want))
