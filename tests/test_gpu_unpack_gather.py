"""Unpacking by gather (spinsum_plan_info_t.unpack_gather) on an MI355X: bit
for bit against the kernel on tiles (SPINSUM_FLAG_NO_XCD_REMAP; every output
is the same one product either way) and against the oracle on sampled cubes
(first, last, and cubes that a workgroup takes second).  The sizes are one
packed value per cube (the 16-byte loads at the tensor's end), several cubes
per item with a partial last item, rows whose threads do not divide the
workgroup, parts of a cube, and large 4D cubes whose rows are described in
batches.

Bars against the oracle: FP64 normwise 1e-14, FP32 2e-6 (on the FP32-rounded
input)."""
import itertools
import math

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
    # shape, d, dtype, unpack_gather
    ((600, 32, 32, 32), 3, F64, 2),
    ((1100, 32, 32, 32), 3, F32, 2),
    ((20003, 8, 8, 8), 3, F64, 2),          # several cubes per item, a partial last one
    ((70001, 4, 4, 4, 4), 4, F32, 2),        # one packed value per cube
    ((40001, 4, 4, 4, 4), 4, F64, 2),
    ((280001, 4, 4, 4), 3, F32, 2),
    ((2300, 20, 20, 20), 3, F32, 2),         # 5 chunks a row
    ((520, 12, 12, 12, 12), 4, F64, 2),
    ((700, 160, 160), 2, F64, 1),
    ((700, 100, 100), 2, F64, 2),
    ((9000, 44, 44), 2, F32, 2),
    ((10001, 6, 6, 6, 4), 3, F64, 2),        # inner runs
    ((17003, 5, 5, 5, 8), 3, F32, 2),
    ((100, 32, 32, 32), 3, F64, 1),         # parts of a cube
    ((270, 48, 48, 48), 3, F64, 1),
    ((260, 20, 20, 20, 20), 4, F32, 1),     # batches of rows
    ((30, 24, 24, 24, 24), 4, F64, 1),
    ((300, 20, 20, 20), 3, F64, 1),
]


def stages_of(d, kind):
    if kind == "anti":
        return [workloads.antisymmetrizer(d)]
    if kind == "all":  # every coefficient its own
        return [[(p, 1.5 + 0.25 * i) for i, p in enumerate(itertools.permutations(range(d)))]]
    ident = tuple(range(d))  # zero coefficients
    return [[(ident, 2.0), (ident[1:] + (0,), -0.5)]]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_unpack_gather(case):
    shape, d, dtype, mode = CASES[case]
    n, ncube = shape[1], shape[0]
    pshape = (ncube, math.comb(n, d)) + tuple(shape[1 + d:])
    pk = workloads.uniform(pshape, 9100 + case, device=DEV, dtype=dtype)
    a = torch.empty(shape, dtype=dtype, device=DEV)
    b = torch.empty(shape, dtype=dtype, device=DEV)
    sample = sorted(c for c in {0, 1, 33, 257, 300, 513, ncube // 2, ncube - 2, ncube - 1} if 0 <= c < ncube)
    if n ** d > 100000:
        sample = [0, ncube - 1]
    for kind in ("anti", "all", "zeros"):
        print(shape, dtype, kind, flush=True)
        stages = stages_of(d, kind)
        p = ss.spinsum_plan(shape, 1, d, stages, dtype=dtype, flags=ss.SPINSUM_FLAG_FULL_GROUP)
        q = ss.spinsum_plan(shape, 1, d, stages, dtype=dtype,
                            flags=ss.SPINSUM_FLAG_FULL_GROUP | ss.SPINSUM_FLAG_NO_XCD_REMAP)
        assert ss.spinsum_plan_get_info(p)["unpack_gather"] == mode
        assert ss.spinsum_plan_get_info(q)["unpack_gather"] == 0
        if kind == "zeros":  # non-finite values reach the terms' outputs alone
            pk.view(-1)[0] = float("inf")
            pk.view(-1)[-1] = float("nan")
        a.fill_(float("nan"))
        b.fill_(float("nan"))
        ss.spinsum_unpack(p, pk, a)
        ss.spinsum_unpack(q, pk, b)
        torch.cuda.synchronize()
        assert torch.equal(a.isnan(), b.isnan())
        assert torch.equal(a.nan_to_num(nan=0.0), b.nan_to_num(nan=0.0))
        if kind != "zeros":
            ref = oracle.unpack(pk[sample].cpu().to(F64).numpy(), (len(sample),) + shape[1:], stages, 1, d)
            got = a[sample].cpu().to(F64).numpy()
            assert np.max(np.abs(got - ref)) <= TOL[dtype] * np.max(np.abs(ref))


def test_unpack_gather_unaligned_packed_and_stream():
    """Packed values at any element alignment, on a side stream."""
    shape = (4200, 16, 16, 16)
    for dtype in (F64, F32):
        p = ss.spinsum_plan(shape, 1, 3, [workloads.antisymmetrizer(3)], dtype=dtype)
        assert ss.spinsum_plan_get_info(p)["unpack_gather"] == 2
        pk = workloads.uniform(ss.packed_shape(p), 9300, device=DEV, dtype=dtype)
        ref = torch.empty(shape, dtype=dtype, device=DEV)
        ss.spinsum_unpack(p, pk, ref)
        torch.cuda.synchronize()
        s = torch.cuda.Stream()
        for off in (1, 2, 3):
            room = torch.empty(pk.numel() + 8, dtype=dtype, device=DEV)
            view = room[off:off + pk.numel()].view(pk.shape)
            view.copy_(pk)
            out = torch.empty(shape, dtype=dtype, device=DEV)
            torch.cuda.synchronize()
            ss.spinsum_unpack(p, view, out, stream=s)
            s.synchronize()
            assert torch.equal(out, ref)
