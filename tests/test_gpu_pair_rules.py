"""Index-pair plans at the tile edges and workgroup sizes the planner picks by
size (64 to 512 threads, whole group cubes, tiles that divide the extent,
ragged tiles), on an MI355X against the oracle, in and out of place.

Bars: FP64 normwise 1e-14, FP32 2e-6 (on the FP32-rounded input)."""
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
    # V, N, d, dtype, inplace, bl, threads
    (9, 4, 3, F64, True, 4, 64),
    (8, 5, 3, F32, False, 5, 64),
    (11, 7, 3, F64, True, 7, 128),
    (11, 8, 3, F32, False, 8, 128),
    (11, 9, 3, F64, True, 9, 256),
    (11, 10, 3, F64, False, 10, 256),
    (4, 12, 3, F64, True, 6, 256),
    (11, 12, 3, F32, True, 12, 256),
    (3, 20, 3, F64, True, 10, 512),
    (3, 20, 3, F64, False, 8, 512),    # ragged
    (3, 20, 3, F32, True, 8, 256),
    (3, 24, 3, F32, False, 12, 512),
    (3, 6, 4, F64, True, 4, 256),
    (4, 4, 4, F64, False, 4, 256),
    (12, 8, 2, F64, True, 8, 64),
    (23, 21, 2, F64, False, 21, 128),
    (5, 48, 2, F64, True, 48, 512),
    (3, 100, 2, F64, True, 40, 512),
    # fewer items than CUs
    (6, 7, 3, F64, True, 7, 512),
    (4, 10, 3, F64, False, 8, 512),
    (7, 10, 3, F32, True, 10, 512),
    (4, 12, 3, F32, True, 8, 256),
    (9, 21, 2, F64, False, 21, 512),
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_pair_rules(case):
    V, N, d, dtype, inplace, bl, threads = CASES[case]
    shape = (V,) * d + (N,) * d
    terms = [(p, 0.5 + 0.25 * i) for i, p in enumerate(itertools.permutations(range(d)))]
    p = ss.spinsum_plan(shape, d, d, [terms], dtype=dtype, inplace=inplace,
                        flags=ss.SPINSUM_FLAG_INDEX_PAIRS)
    info = ss.spinsum_plan_get_info(p)
    assert (info["bl"], info["threads"]) == (bl, threads)
    x = workloads.uniform(shape, 9900 + case, device=DEV, dtype=dtype)
    xh = x.cpu().to(F64).numpy()
    for run, want in ((ss.spinsum_exec, oracle.spinsum(xh, terms, d, d, nthreads=8, pairs=True)),
                      (ss.spinsum_adjoint,
                       oracle.spinsum_chain_adjoint(xh, [terms], d, d, nthreads=8, pairs=True))):
        y = x.clone() if inplace else torch.empty_like(x)
        run(p, y if inplace else x, y)
        torch.cuda.synchronize()
        got = y.cpu().to(F64).numpy()
        assert np.max(np.abs(got - want)) <= TOL[dtype] * np.max(np.abs(want))
