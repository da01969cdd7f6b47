"""Launches of 2^32 threads and more, which the runtime would cut short: small
cubes one to a workgroup (a requested tile), and index pairs with many tile
orbits, of one block and of several.  Every path against plain torch on the
same values, exactly: coefficients and inputs are small whole numbers."""
import itertools

import pytest
import torch

pytestmark = pytest.mark.gpu

ss = pytest.importorskip("paper_1705_06661_amd")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

DEV = torch.device("cuda:0")
F32 = torch.float32
CUBES = 4_300_000  # of 2^3, a workgroup of 1024 threads each: 4.4e9 threads


def _ints(shape, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return torch.randint(-8, 9, shape, dtype=torch.int32, device=DEV, generator=g).to(F32)


def _perms(d):
    return [(p, float(1 + i)) for i, p in enumerate(itertools.permutations(range(d)))]


def _sum(x, terms, first, pairs=False):
    """out[.., i_0.., i_{d-1}] = sum a in[.., i_{p[0]}, .., i_{p[d-1]}]"""
    out = torch.zeros_like(x)
    for p, a in terms:
        d = len(p)
        inv = [p.index(m) for m in range(d)]
        axes = list(range(x.dim()))
        for m in range(d):
            axes[first + m] = first + inv[m]
            if pairs:
                axes[first - d + m] = first - d + inv[m]
        out += a * x.permute(axes)
    return out


@pytest.mark.parametrize("variant,threads,cubes", [
    (ss.SPINSUM_VARIANT_DIRECT_LDS, 1024, CUBES),
    (ss.SPINSUM_VARIANT_REG_ONESHOT, 0, 4 * CUBES)])
def test_many_small_cubes(variant, threads, cubes):
    shape = (cubes, 2, 2, 2)
    p = ss.spinsum_plan(shape, 1, 3, [_perms(3)], dtype="f32")
    ss.spinsum_plan_set_tile(p, 2, cubes_per_wg=1, lds_pad=0, threads=threads, variant=variant)
    info = p.info()
    assert info["variant"] == variant and info["nitems"] * info["threads"] >= 1 << 32
    x = _ints(shape, 1)
    y = ss.spinsum_exec(p, x, torch.full_like(x, float("nan")))
    assert torch.equal(y, _sum(x, _perms(3), 1))


def test_many_small_cubes_gradients_and_packing():
    shape = (CUBES, 3, 3, 3)
    p = ss.spinsum_plan(shape, 1, 3, [_perms(3)], dtype="f32")
    ss.spinsum_plan_set_tile(p, 3, cubes_per_wg=1, lds_pad=0, threads=1024,
                             variant=ss.SPINSUM_VARIANT_DIRECT_LDS)
    x = _ints(shape, 2)
    # packing and unpacking (on tiles: one packed value a cube)
    packed = ss.spinsum_pack(p, x, torch.full(ss.packed_shape(p), float("nan"), dtype=F32, device=DEV))
    full = ss.spinsum_unpack(p, packed, torch.full_like(x, float("nan")))
    e = torch.zeros_like(x)
    e[:, 0, 1, 2] = packed[:, 0]
    assert torch.equal(full, _sum(e, _perms(3), 1))
    adj = [(tuple(q.index(m) for m in range(3)), a) for q, a in _perms(3)]
    assert torch.equal(packed[:, 0], _sum(x, adj, 1)[:, 0, 1, 2])
    del e, full
    # both gradients: four times the cubes, 256 threads each
    shape = (4 * CUBES, 2, 2, 2)
    p = ss.spinsum_plan(shape, 1, 3, [_perms(3)], dtype="f32")
    ss.spinsum_plan_set_tile(p, 2, cubes_per_wg=1, lds_pad=0, variant=ss.SPINSUM_VARIANT_DIRECT_LDS)
    assert p.info()["nitems"] * 256 >= 1 << 32
    x, g = _ints(shape, 3), _ints(shape, 4)
    gx = torch.full_like(g, float("nan"))
    c = ss.spinsum_adjoint_coef_grad(p, x, g, gx)
    assert torch.equal(gx, _sum(g, adj, 1))
    want = [torch.sum((g * _sum(x, [(q, 1.0)], 1)).to(torch.int64)).item() for q, _ in _perms(3)]
    assert c.tolist() == want


@pytest.mark.parametrize("shape", [(6000, 6000, 2, 2), (3, 4400, 4400, 2, 2)])
def test_many_pair_orbits(shape):
    first = len(shape) - 2
    p = ss.spinsum_plan(shape, first, 2, [_perms(2)], dtype="f32",
                        flags=ss.SPINSUM_FLAG_INDEX_PAIRS)
    ss.spinsum_plan_set_tile(p, 2, threads=256)
    info = p.info()
    assert info["nitems"] * info["threads"] >= 1 << 32
    x = _ints(shape, 5)
    y = ss.spinsum_exec(p, x, torch.full_like(x, float("nan")))
    assert torch.equal(y, _sum(x, _perms(2), first, pairs=True))
