"""The tile that an index-pair plan reports can be set on it, the workgroup
sizes of small whole group cubes among them; elsewhere these stay refused."""
import itertools

import pytest
import torch

import workloads

ss = pytest.importorskip("paper_1705_06661_amd")

# shape, d, dtype, threads the planner takes
SHAPES = [
    ((20, 20, 20, 4, 4, 4), 3, torch.float64, 64),
    ((20, 20, 20, 7, 7, 7), 3, torch.float64, 128),
    ((16, 16, 16, 8, 8, 8), 3, torch.float32, 128),
    ((40, 40, 9, 9), 2, torch.float64, 64),
    ((16, 16, 16, 8, 8, 8), 3, torch.float64, 256),
    ((6, 6, 6, 24, 24, 24), 3, torch.float64, 512),
    ((4, 4, 4, 4, 8, 8, 8, 8), 4, torch.float64, 256),
]


def _plan(shape, d, dtype, flags=0):
    terms = [[(p, 0.5 + 0.25 * i) for i, p in enumerate(itertools.permutations(range(d)))]]
    return ss.spinsum_plan(shape, d, d, terms, dtype=dtype, inplace=True,
                           flags=flags | ss.SPINSUM_FLAG_INDEX_PAIRS)


@pytest.mark.parametrize("shape,d,dtype,threads", SHAPES)
def test_reported_tile_can_be_set(shape, d, dtype, threads):
    p = _plan(shape, d, dtype, ss.SPINSUM_FLAG_HOST_ONLY)
    info = p.info()
    assert info["threads"] == threads
    ss.spinsum_plan_set_tile(p, info["bl"], info["cubes_per_wg"], info["lds_pad"], info["threads"],
                             info["variant"])
    assert p.info() == info
    if threads in (64, 128):
        return
    whole = info["bl"] == shape[-1] and d <= 3
    for small in (32, 64, 128):
        if whole and small != 32:
            continue
        with pytest.raises(ss.SpinSumError) as e:
            ss.spinsum_plan_set_tile(p, info["bl"], threads=small)
        assert e.value.status == ss.SPINSUM_ERR_UNSUPPORTED
        assert p.info() == info


@pytest.mark.gpu
@pytest.mark.parametrize("shape,d,dtype,threads", SHAPES[:4])
def test_small_workgroups(shape, d, dtype, threads):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    x = workloads.uniform(shape, 9700, device=torch.device("cuda:0"), dtype=dtype)
    outs = []
    for th in (0, 64, 128, 256):
        p = _plan(shape, d, dtype)
        if th:
            ss.spinsum_plan_set_tile(p, shape[-1], threads=th)
        y = x.clone()
        outs.append(ss.spinsum_exec(p, y, y))
    torch.cuda.synchronize()
    assert all(torch.equal(o, outs[0]) for o in outs[1:])
