"""The tiles exec runs on, read from the planner on the CPU
(tests/sanitize/sum_tiles_driver.cpp): what the plan's info does not show."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SAN = os.path.join(ROOT, "tests", "sanitize")
CSRC = os.path.join(ROOT, "paper_1705_06661_amd", "csrc")

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")


@pytest.fixture(scope="module")
def tiles(tmp_path_factory):
    """(d, N, inner, dtype, inplace, cubes) -> (own edge or 0, items, orbits
    of a cube, store mode, the plan's store mode)"""
    tmp = tmp_path_factory.mktemp("sum_tiles")
    base = ["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
            "-I" + os.path.join(ROOT, "include"), "-I" + CSRC]
    objs, procs = [], []
    for src in (os.path.join(CSRC, "spinsum_plan.cpp"), os.path.join(CSRC, "spinsum_tune.cpp"),
                os.path.join(SAN, "hip_host_stub.cpp"), os.path.join(SAN, "sum_tiles_driver.cpp")):
        objs.append(str(tmp / (os.path.basename(src) + ".o")))
        procs.append(subprocess.Popen(base + ["-c", src, "-o", objs[-1]], stdout=subprocess.PIPE,
                                      stderr=subprocess.STDOUT, text=True))
    for p in procs:
        out, _ = p.communicate(timeout=600)
        assert p.returncode == 0, out[-4000:]
    exe = str(tmp / "sum_tiles_driver")
    subprocess.run(["g++"] + objs + ["-o", exe], check=True, timeout=300)

    def ask(*case):
        r = subprocess.run([exe] + [str(int(c) if isinstance(c, bool) else c) for c in case],
                           check=True, capture_output=True, text=True, timeout=300)
        return tuple(int(v) for v in r.stdout.split())
    return ask


@pytest.mark.parametrize("n,inner,dtype,cubes,packed", [
    (13, 1, "f64", 1, False), (13, 1, "f64", 146, False), (13, 1, "f64", 147, True),
    (17, 1, "f64", 73, False), (17, 1, "f64", 74, True), (15, 2, "f32", 20, False),
    (15, 2, "f32", 200, True), (13, 1, "f32", 1, False), (13, 1, "f32", 500, False)])
def test_orbits_of_odd_rows_are_packed_where_there_are_many(tiles, n, inner, dtype, cubes, packed):
    """4D orbits of which three fit a CU: one an item below 20 a CU (256 CUs),
    several above; of which six fit (FP32): one an item."""
    bl, items, orbits, _, _ = tiles(4, n, inner, dtype, True, cubes)
    assert bl == 4
    assert items < orbits * cubes if packed else items == orbits * cubes



@pytest.mark.parametrize("d,n,inner,dtype,edge", [
    (4, 9, 3, "f64", 0), (4, 11, 3, "f64", 0), (4, 9, 5, "f64", 2), (4, 9, 3, "f32", 4),
    (3, 29, 3, "f32", 0), (3, 33, 3, "f32", 0), (3, 41, 3, "f32", 0), (3, 27, 3, "f32", 4),
    (3, 31, 3, "f32", 4), (3, 37, 3, "f32", 4), (3, 33, 5, "f32", 4), (3, 33, 3, "f64", 6),
    (3, 33, 1, "f32", 8), (3, 34, 1, "f32", 8), (3, 33, 1, "f64", 8)])
def test_short_rows_stay_on_the_register_path(tiles, d, n, inner, dtype, edge):
    """4D rows of part sectors at the register path's edge, and edges a third
    narrower that do not cover an eighth less: its tiles stay."""
    assert tiles(d, n, inner, dtype, True, 600)[0] == edge


@pytest.mark.parametrize("n,dtype,edge", [(30, "f64", 10), (46, "f64", 10), (70, "f64", 10),
                                          (78, "f64", 10), (90, "f64", 10), (36, "f32", 12),
                                          (108, "f32", 12)])
def test_wide_tiles_store_as_the_plans_tiles(tiles, n, dtype, edge):
    for inplace in (False, True):
        bl, _, _, nts, plan_nts = tiles(3, n, 1, dtype, inplace, 100)
        assert (bl, nts) == (edge, plan_nts)


@pytest.mark.parametrize("d,n,inner,dtype,cubes,edge", [
    (3, 24, 1, "f64", 1213, 24), (3, 24, 1, "f64", 1214, 0), (3, 24, 1, "f64", 2427, 0),
    (3, 24, 1, "f64", 2428, 24), (2, 120, 1, "f64", 1165, 120), (2, 120, 1, "f64", 2000, 0),
    (2, 120, 1, "f64", 2400, 120), (3, 24, 2, "f32", 600, 0), (3, 24, 2, "f32", 4854, 0),
    (3, 24, 2, "f32", 4855, 24), (3, 16, 5, "f32", 1638, 16), (3, 16, 5, "f32", 3000, 16)])
def test_tiles_where_the_infinity_cache_holds_the_tensor(tiles, d, n, inner, dtype, cubes, edge):
    """Whole cubes in place of tiles of whole sectors: not for 128 to 256 MB
    in FP64, up to 512 MB in FP32 (tiles of part sectors: at every size)."""
    assert tiles(d, n, inner, dtype, True, cubes)[0] == edge


@pytest.mark.gpu
@pytest.mark.parametrize("shape,dtype", [((150, 13, 13, 13, 13), "f64"), ((40, 13, 13, 13, 13), "f64"),
                                         ((200, 15, 15, 15, 15, 2), "f32")])
def test_packed_and_single_orbits(shape, dtype):
    """Both sides of the rule bit for bit against the register path."""
    import itertools
    import torch
    import paper_1705_06661_amd as ss
    import workloads
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    terms = [[(p, 0.5 + 0.25 * i) for i, p in enumerate(itertools.permutations(range(4)))]]
    p = ss.spinsum_plan(shape, 1, 4, terms, dtype=dtype)
    q = ss.spinsum_plan(shape, 1, 4, terms, dtype=dtype, flags=ss.SPINSUM_FLAG_NO_DIRECT_LDS)
    assert p.info()["sum_bl"] == 4 and q.info()["sum_bl"] == 0
    x = workloads.uniform(shape, 9750, device=torch.device("cuda:0"), dtype=p.dtype)
    y, z = ss.spinsum_exec(p, x, torch.empty_like(x)), ss.spinsum_exec(q, x, torch.empty_like(x))
    torch.cuda.synchronize()
    assert torch.equal(y, z)
