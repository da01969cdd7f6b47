"""SPINSUM_FLAG_NO_NT_STORES reaches unpacking: plans that would unpack by
gather, which stores non-temporally, unpack on tiles with cached stores
instead.  Host-only plans; on a GPU both forms bit for bit."""
import pytest
import torch

import workloads

ss = pytest.importorskip("paper_1705_06661_amd")

SHAPES = [
    # shape, d, dtype, unpack_gather of the default plan
    ((700, 32, 32, 32), 3, torch.float64, 2),
    ((200, 48, 48, 48), 3, torch.float64, 1),
    ((600, 12, 12, 12, 12), 4, torch.float64, 2),
    ((1100, 32, 32, 32), 3, torch.float32, 2),
    ((600, 120, 120), 2, torch.float64, 2),
]


@pytest.mark.parametrize("shape,d,dtype,mode", SHAPES)
def test_flag_reaches_unpacking(shape, d, dtype, mode):
    terms = [workloads.antisymmetrizer(d)]
    H = ss.SPINSUM_FLAG_HOST_ONLY
    info = ss.spinsum_plan(shape, 1, d, terms, dtype=dtype, flags=H).info()
    assert info["unpack_gather"] == mode
    info = ss.spinsum_plan(shape, 1, d, terms, dtype=dtype, flags=H | ss.SPINSUM_FLAG_NO_NT_STORES).info()
    assert (info["unpack_gather"], info["unpack_nt_stores"]) == (0, 0)


@pytest.mark.gpu
@pytest.mark.parametrize("shape,d,dtype,mode", SHAPES)
def test_unpacking_with_the_flag(shape, d, dtype, mode):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    terms = [workloads.antisymmetrizer(d)]
    outs = []
    for flags in (0, ss.SPINSUM_FLAG_NO_NT_STORES):
        p = ss.spinsum_plan(shape, 1, d, terms, dtype=dtype, flags=flags)
        pk = workloads.uniform(ss.packed_shape(p), 9650, device=torch.device("cuda:0"), dtype=dtype)
        outs.append(ss.spinsum_unpack(p, pk, torch.empty(shape, dtype=dtype, device=pk.device)))
    torch.cuda.synchronize()
    assert torch.equal(*outs)


@pytest.mark.parametrize("shape,d,dtype,nt", [
    ((400, 300, 300), 2, torch.float64, 1), ((400, 250, 250), 2, torch.float64, 1),
    ((100, 500, 500), 2, torch.float64, 1), ((100, 300, 300, 3), 2, torch.float32, 1),
    ((600, 54, 54, 54), 3, torch.float64, 0),  # the plan's own 8^3 tiles
])
def test_store_mode_of_unpackings_own_tiles(shape, d, dtype, nt):
    """Unpacking on large tiles of its own stores non-temporally also where
    rows are off 64-byte sectors; on the plan's tiles as the plan does."""
    info = ss.spinsum_plan(shape, 1, d, [workloads.antisymmetrizer(d)], dtype=dtype,
                           flags=ss.SPINSUM_FLAG_HOST_ONLY).info()
    assert (info["unpack_gather"], info["unpack_nt_stores"]) == (0, nt)
