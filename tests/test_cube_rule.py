"""Which plans run whole cubes persistently (one workgroup of 1024 threads per
CU, reported as persistent_per_cu 1): those whose tile the planner chose.  A
requested whole-cube tile runs one item per workgroup with the workgroup size
it names.  Host-only plans; on a GPU the requested forms against the chosen
one bit for bit."""
import itertools

import pytest
import torch

import workloads

ss = pytest.importorskip("paper_1705_06661_amd")
F64, F32 = torch.float64, torch.float32

SHAPES = [
    ((517, 24, 24, 24), 3, F64, True),
    ((517, 24, 24, 24), 3, F64, False),
    ((512, 26, 26, 26), 3, F64, True),
    ((771, 25, 25, 25), 3, F64, False),
    ((513, 29, 29, 29), 3, F32, True),
    ((514, 30, 30, 30), 3, F32, False),
    ((515, 31, 31, 31), 3, F32, True),
    ((520, 111, 111), 2, F64, True),
    ((512, 151, 151), 2, F32, False),
    ((519, 13, 13, 13, 5), 3, F64, False),
]


def _plan(shape, d, dtype, inplace, flags=0):
    terms = [[(p, 0.5 + 0.25 * i) for i, p in enumerate(itertools.permutations(range(d)))]]
    return ss.spinsum_plan(shape, 1, d, terms, dtype=dtype, inplace=inplace, flags=flags)


@pytest.mark.parametrize("shape,d,dtype,inplace", SHAPES)
def test_cube_rule(shape, d, dtype, inplace):
    H = ss.SPINSUM_FLAG_HOST_ONLY
    n = shape[1]
    assert _plan(shape, d, dtype, inplace, H).info()["persistent_per_cu"] == 1
    q = _plan(shape, d, dtype, inplace, H | ss.SPINSUM_FLAG_NO_XCD_REMAP)
    assert q.info()["persistent_per_cu"] == 0
    few = (511,) + shape[1:]
    assert _plan(few, d, dtype, inplace, H).info()["persistent_per_cu"] == 0
    p = _plan(shape, d, dtype, inplace, H)
    for threads in (256, 512, 1024):
        ss.spinsum_plan_set_tile(p, n, threads=threads, variant=ss.SPINSUM_VARIANT_DIRECT_LDS)
        info = p.info()
        assert (info["bl"], info["threads"], info["persistent_per_cu"], info["sum_bl"]) == (n, threads, 0, 0)
    ss.spinsum_plan_set_tile(p, 0)  # the planner's choice again
    assert p.info()["persistent_per_cu"] == 1


@pytest.mark.gpu
@pytest.mark.parametrize("case", [0, 1, 3, 9])
def test_requested_cubes(case):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    shape, d, dtype, inplace = SHAPES[case]
    x = workloads.uniform(shape, 9600 + case, device=torch.device("cuda:0"), dtype=dtype)
    outs = []
    for threads in (0, 256, 512, 1024):
        p = _plan(shape, d, dtype, inplace)
        if threads:
            ss.spinsum_plan_set_tile(p, shape[1], threads=threads, variant=ss.SPINSUM_VARIANT_DIRECT_LDS)
        y = x.clone() if inplace else torch.empty_like(x)
        outs.append(ss.spinsum_exec(p, y if inplace else x, y))
    torch.cuda.synchronize()
    assert all(torch.equal(o, outs[0]) for o in outs[1:])
