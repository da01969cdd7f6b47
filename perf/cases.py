"""Cases that time the public entry points of the spin-summation library.

A case is a dict of plain values.  ``prepare`` makes what a program holds
before the call (tensors, and the plan it keeps), ``run`` is one pass through
the public entry points, ``exact`` the same result from plain torch in 64
bits, ``work`` the bytes and operations a pass cannot do without: every input
read once, every output written once, two operations per term and element.

Tensors are named as in ``workloads``: T[a,b,c,i,j,k] with v values of each
virtual index a, b, c and o values of each occupied index i, j, k, the
permuted group.  Values are uniform in [-1, 1), made on the GPU from the seed.

The operators are those of ``workloads`` divided by their largest eigenvalue
(12 for the 3D set, 60 for case 5 of Table II, the coefficient sum for the
24 random coefficients, 3 a factor for (2 - P_ij)(2 - P_jk)), so that a
program that applies them in place again and again keeps finite values.

Entry points (``kind``):
  exec     spinsum_exec, or spinsum_adjoint with ``adjoint``
  vjp      SpinSumFunction, forward and backward
  train    SpinSumCoefFunction, forward and backward to the tensor and to
           the coefficients (a new plan on every call, as that class makes)
  cgrad    spinsum_coef_grad
  unpack   spinsum_unpack of an antisymmetric tensor, pack its adjoint
  pairs    spinsum_exec of an index-pair plan, partners and group permuted
           together
  batched  one spinsum_graph_launch over many blocks
"""
from __future__ import annotations

import itertools
import math

import numpy as np
import torch

import workloads
import paper_1705_06661_amd as ss

_DTYPE = {"f64": torch.float64, "f32": torch.float32}


# ------------------------------------------------------------------ operators
def _scaled(stage, s):
    return [(tuple(p), a * s) for p, a in stage]


def operator(name: str, d: int):
    """Stages (innermost first) of a named operator over d indices."""
    if name == "anti":      # the projector on the antisymmetric part
        return [_scaled(workloads.antisymmetrizer(d), 1.0 / math.factorial(d))]
    if name == "subgroup":  # (1 + P_12)/2: moves the first two axes only
        ident = tuple(range(d))
        return [[(ident, 0.5), ((1, 0) + ident[2:], 0.5)]]
    if name == "dense":     # 24 random coefficients, every permutation present
        st = workloads.random_4d_alpha(3)
        return [_scaled(st, 1.0 / sum(a for _, a in st))]
    if name == "factored":  # (2 - P_ij)(2 - P_jk)
        return [_scaled(st, 1.0 / 3.0) for st in workloads.FACTORED_PIJ_PJK]
    if d == 2:              # 2 - P_12
        return [[((0, 1), 2.0 / 3.0), ((1, 0), -1.0 / 3.0)]]
    if d == 3:              # identity 4, transpositions -2, 3-cycles 1
        return [_scaled(workloads.CONFIG_3D_ALPHA, 1.0 / 12.0)]
    _, stages = workloads.table2_case(5)
    return [_scaled(stages[0], 1.0 / 60.0)] + stages[1:]


def _expanded(stages, d):
    """The operator as one sum, {permutation: coefficient}."""
    acc = {tuple(range(d)): 1.0}
    for st in stages:
        nxt = {}
        for q, b in acc.items():
            for p, a in st:
                # stage p reads position p of what the stages before it made
                r = tuple(p[q[m]] for m in range(d))
                nxt[r] = nxt.get(r, 0.0) + a * b
        acc = nxt
    return {p: a for p, a in acc.items() if a != 0.0}


def _axes(p, first, ndim, pairs=False):
    """Axes for torch.permute of the term with permutation p: the output
    index m of the group reads the input's axis where p holds m."""
    d = len(p)
    inv = [0] * d
    for m in range(d):
        inv[p[m]] = m
    axes = list(range(ndim))
    for m in range(d):
        axes[first + m] = first + inv[m]
        if pairs:
            axes[first - d + m] = first - d + inv[m]
    return axes


def _apply(x, stages, first, d, adjoint=False, pairs=False):
    """The operator by plain torch in 64 bits, a stage after the other."""
    for st in (reversed(stages) if adjoint else stages):
        acc = None
        for p, a in st:
            axes = _axes(p, first, x.dim(), pairs)
            if adjoint:
                inv = [0] * len(axes)
                for m, ax in enumerate(axes):
                    inv[ax] = m
                axes = inv
            t = x.permute(axes)
            acc = t * a if acc is None else acc.add_(t, alpha=a)
        x = acc
    return x.contiguous()


# --------------------------------------------------------------------- shapes
def _shape(case):
    """(shape, first dim of the group) of a case's tensor."""
    o, d = case["o"], case["d"]
    if case["kind"] == "pairs":
        return (case["v"],) * d + (o,) * d, d
    outer = tuple(int(e) for e in case["outer"].split("x")) if case["outer"] else ()
    inner = (case["inner"],) if case.get("inner", 1) > 1 else ()
    return outer + (o,) * d + inner, len(outer)


def _blocks(case):
    """Shapes of the blocks of a batched case and their offsets in one
    buffer (every block on a 256-byte boundary, as an allocator gives)."""
    rng = np.random.default_rng(case["block_seed"])
    v = workloads.power_law(rng, 4, case["v"], 1.75, case["blocks"])
    o = workloads.power_law(rng, 2, case["o"], 1.75, case["blocks"])
    shapes, offs, pos = [], [], 0
    step = 256 // (8 if case["dtype"] == "f64" else 4)
    for a, b in zip(v, o):
        s = (int(a),) * 3 + (int(b),) * 3
        shapes.append(s)
        offs.append(pos)
        pos += -(-math.prod(s) // step) * step
    return shapes, offs, pos


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) + 1)
    return g


def _uniform(shape, dtype, g):
    return torch.empty(shape, dtype=dtype, device="cuda").uniform_(-1.0, 1.0, generator=g)


def _packed_shape(shape, first, d):
    return shape[:first] + (math.comb(shape[first], d),) + shape[first + d:]


def _inputs(case, seed):
    """The input tensors of a case, from the seed alone."""
    dt, g = _DTYPE[case["dtype"]], _generator(seed)
    kind = case["kind"]
    if kind == "batched":
        shapes, offs, total = _blocks(case)
        flat = torch.zeros(total, dtype=dt, device="cuda")
        for s, at in zip(shapes, offs):
            flat[at:at + math.prod(s)].uniform_(-1.0, 1.0, generator=g)
        return [flat]
    shape, first = _shape(case)
    if kind == "unpack":
        return [_uniform(_packed_shape(shape, first, case["d"]), dt, g)]
    n = 2 if kind in ("vjp", "train", "cgrad") else 1
    return [_uniform(shape, dt, g) for _ in range(n)]


# ------------------------------------------------------------------ the cases
def _case(name, kind, d, o, outer="", dtype="f64", inplace=False, adjoint=False, op="spin",
          inner=1, v=0, blocks=0, block_seed=0):
    return {"name": name, "kind": kind, "d": d, "o": o, "outer": outer, "dtype": dtype,
            "inplace": inplace, "adjoint": adjoint, "op": op, "inner": inner, "v": v,
            "blocks": blocks, "block_seed": block_seed}


def listed():
    return [
        # one small amplitude tensor (v = 16, o = 8) inside an autograd
        # program: forward and backward, 34 MB each; launches count
        _case("vjp_3d_v16_o8", "vjp", 3, 8, "16x16x16"),
        # the headline workload: one slab of the v = 64, o = 32 triples
        # amplitudes, 8.6 GB in place
        _case("slab_3d_v64_o32_inplace", "exec", 3, 32, "64x64x8", inplace=True),
        # out of place in the other direction: v = 48, o = 24, a slab of six
        _case("adjoint_3d_v48_o24", "exec", 3, 24, "48x48x8", adjoint=True, op="factored"),
        # single precision, v = 48, o = 24
        _case("forward_3d_v48_o24_f32", "exec", 3, 24, "48x48x16", dtype="f32", op="factored"),
        # an odd number of occupied orbitals: no row is a whole 16-byte chunk
        _case("odd_3d_v40_o33_inplace", "exec", 3, 33, "40x40x4", inplace=True),
        # quadruples: one a-slab of v = 24, o = 12, 24 coefficients, 2.3 GB
        _case("slab_4d_v24_o12_inplace", "exec", 4, 12, "1x24x24x24", inplace=True, op="dense"),
        # the paper's own benchmark, medium size: one cube without spectators
        _case("cube_4d_n80_inplace", "exec", 4, 80, "", inplace=True),
        _case("cube_3d_n352_inplace", "exec", 3, 352, "", inplace=True),
        # symmetry blocks of very different sizes in one graph launch, 2 GB
        _case("batched_200_blocks", "batched", 3, 16, v=40, blocks=200, block_seed=7,
              inplace=True),
        # a training step that learns the coefficients: output, gradient of
        # the tensor, gradient of the coefficients
        _case("train_3d_v32_o16", "train", 3, 16, "32x32x32"),
        # an antisymmetric tensor unpacked from its strictly increasing
        # entries, 4.3 GB written
        _case("unpack_3d_v64_o32", "unpack", 3, 32, "64x64x4", op="anti"),
        # triples amplitudes with (a,i), (b,j), (c,k) as pairs, v = 48,
        # o = 24, 12.2 GB in place
        _case("pairs_3d_v48_o24_inplace", "pairs", 3, 24, v=48, inplace=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _outer(rng, cubes):
    """Two or three outer extents whose product is about `cubes`."""
    a = max(1, _log_int(rng, 1, max(1, cubes)))
    b = max(1, cubes // a)
    return "%dx%d" % (a, b)


def _aligned(rng, d, dtype):
    """An extent for the forms that need the direct layout: a cube of which
    two fit a CU, or rows of whole 16-byte chunks."""
    step = 2 if dtype == "f64" else 4
    small, large = (20, 48) if d == 3 else (8, 24)
    if rng.random() < 0.5:
        return rng.randint(d, small)
    return step * rng.randint(-(-small // step), large // step)


def draw(rng):
    """One more case: the listed kinds over d = 2..4, extents 3..48 (4D to
    24, 2D to 160) with odd ones among them, 1 MB to 4 GB a tensor, both
    types, in place or out of place, forward or adjoint, trailing groups or
    inner runs; single cubes of 30 MB to 1.3 GB; batches of 8 to 200 blocks."""
    kind = rng.choice(["exec", "exec", "exec", "exec", "cube", "vjp", "train", "cgrad", "unpack",
                       "pack", "pairs", "batched"])
    dtype = rng.choice(["f64", "f64", "f32"])
    esz = 8 if dtype == "f64" else 4
    elems = _log_int(rng, 1 << 18, 1 << 29)
    if kind == "cube":
        d = rng.choice([3, 4])
        o = rng.randint(200, 544) if d == 3 else 2 * rng.randint(26, 56)
        return _case("", "exec", d, o, "", dtype, inplace=True)
    if kind == "batched":
        blocks = _log_int(rng, 8, 200)
        return _case("", "batched", 3, rng.randint(8, 16), v=rng.randint(12, 40), blocks=blocks,
                     block_seed=rng.randint(0, 1 << 20), dtype=dtype, inplace=True)
    if kind == "pairs":
        o = rng.randint(4, 12) if rng.random() < 0.5 else 4 * rng.randint(3, 6)
        v = max(2, min(48, int((elems / o ** 3) ** (1 / 3))))
        return _case("", "pairs", 3, o, v=v, dtype=dtype, inplace=rng.random() < 0.7)
    d = rng.choice([2, 3, 3, 3, 4, 4])
    if kind in ("exec", "vjp"):
        o = _log_int(rng, 8, 160) if d == 2 else rng.randint(4, 48) if d == 3 else rng.randint(3, 24)
        ops = {2: ["spin"], 3: ["spin", "factored", "anti", "subgroup"], 4: ["spin", "dense", "anti"]}
        op = rng.choice(ops[d])
        inner = rng.choice([1, 1, 1, 2, 3, 8]) if o ** d < 50000 else 1
        cubes = max(1, elems // (o ** d * inner))
        return _case("", kind, d, o, _outer(rng, cubes), dtype,
                     inplace=kind == "exec" and rng.random() < 0.6,
                     adjoint=kind == "exec" and rng.random() < 0.3, op=op, inner=inner)
    d = max(d, 3)
    o = _aligned(rng, d, dtype)
    cubes = max(1, elems // o ** d)
    op = "anti" if kind in ("unpack", "pack") else "spin" if d == 3 else "dense"
    return _case("", kind, d, o, _outer(rng, cubes), dtype, op=op)


# -------------------------------------------------------------------- running
def prepare(case, seed):
    xs = _inputs(case, seed)
    kind, d, inplace = case["kind"], case["d"], case["inplace"]
    stages = operator(case["op"], d)
    st = {"case": case, "xs": xs}
    if kind == "batched":
        shapes, offs, _ = _blocks(case)
        ts = [xs[0][at:at + math.prod(s)].view(s) for s, at in zip(shapes, offs)]
        plan = ss.spinsum_plan_batched(shapes, d, stages, dtype=case["dtype"], inplace=True)
        st["graph"] = ss.spinsum_graph_create(plan, ts, ts)
        return st
    shape, first = _shape(case)
    if kind == "train":
        st["perms"] = [p for p, _ in stages[0]]
        st["alpha"] = torch.tensor([a for _, a in stages[0]], dtype=_DTYPE[case["dtype"]],
                                   device="cuda", requires_grad=True)
        xs[0].requires_grad_(True)
        st["first"] = first
        return st
    flags = ss.SPINSUM_FLAG_INDEX_PAIRS if kind == "pairs" else 0
    st["plan"] = ss.spinsum_plan(shape, first, d, stages, dtype=case["dtype"], inplace=inplace,
                                 flags=flags)
    if kind == "vjp":
        xs[0].requires_grad_(True)
    elif kind == "unpack":
        st["out"] = torch.empty(shape, dtype=xs[0].dtype, device="cuda")
    elif kind == "pack":
        st["out"] = torch.empty(_packed_shape(shape, first, d), dtype=xs[0].dtype, device="cuda")
    elif kind in ("exec", "pairs"):
        st["out"] = xs[0] if inplace else torch.empty_like(xs[0])
    return st


def run(state):
    case, xs = state["case"], state["xs"]
    kind = case["kind"]
    if kind == "batched":
        ss.spinsum_graph_launch(state["graph"])
        return xs[0]
    if kind == "vjp":
        y = ss.SpinSumFunction.apply(xs[0], state["plan"])
        (gx,) = torch.autograd.grad(y, (xs[0],), xs[1])
        return y.detach(), gx
    if kind == "train":
        y = ss.SpinSumCoefFunction.apply(xs[0], state["alpha"], state["perms"], state["first"])
        gx, ga = torch.autograd.grad(y, (xs[0], state["alpha"]), xs[1])
        return y.detach(), gx, ga
    plan = state["plan"]
    if kind == "cgrad":
        return ss.spinsum_coef_grad(plan, xs[0], xs[1])
    if kind == "unpack":
        return ss.spinsum_unpack(plan, xs[0], state["out"])
    if kind == "pack":
        return ss.spinsum_pack(plan, xs[0], state["out"])
    if case["adjoint"]:
        return ss.spinsum_adjoint(plan, xs[0], state["out"])
    return ss.spinsum_exec(plan, xs[0], state["out"])


def _increasing(o, d):
    """Linear index, in a cube of edge o, of every strictly increasing tuple,
    in lexicographic order."""
    grids = torch.meshgrid(*[torch.arange(o, device="cuda")] * d, indexing="ij")
    ok = torch.ones_like(grids[0], dtype=torch.bool)
    for m in range(d - 1):
        ok &= grids[m] < grids[m + 1]
    return ok.reshape(-1).nonzero().reshape(-1)


def exact(case, seed):
    xs = [x.double() for x in _inputs(case, seed)]
    kind, d = case["kind"], case["d"]
    stages = operator(case["op"], d)
    if kind == "batched":
        shapes, offs, total = _blocks(case)
        out = torch.zeros_like(xs[0])
        for s, at in zip(shapes, offs):
            n = math.prod(s)
            out[at:at + n] = _apply(xs[0][at:at + n].view(s), stages, 3, d).reshape(-1)
        return out
    shape, first = _shape(case)
    if kind in ("exec", "pairs"):
        return _apply(xs[0], stages, first, d, case["adjoint"], kind == "pairs")
    if kind == "vjp":
        return (_apply(xs[0], stages, first, d), _apply(xs[1], stages, first, d, adjoint=True))
    if kind in ("train", "cgrad"):
        perms = [p for p, _ in stages[0]] if kind == "train" else itertools.permutations(range(d))
        g = xs[1].reshape(-1)
        ga = torch.stack([torch.dot(g, xs[0].permute(_axes(p, first, xs[0].dim())).reshape(-1))
                          for p in perms])
        if kind == "cgrad":
            return ga
        # the coefficients in the type the program holds them in
        al = torch.tensor([a for _, a in stages[0]], dtype=_DTYPE[case["dtype"]]).double().tolist()
        st = [[(p, a) for (p, _), a in zip(stages[0], al)]]
        return _apply(xs[0], st, first, d), _apply(xs[1], st, first, d, adjoint=True), ga
    at = _increasing(case["o"], d)
    outer = math.prod(shape[:first])
    if kind == "unpack":
        full = torch.zeros((outer, case["o"] ** d), dtype=torch.float64, device="cuda")
        full[:, at] = xs[0].reshape(outer, -1)
        return _apply(full.view(shape), stages, first, d)
    y = _apply(xs[0], stages, first, d, adjoint=True)
    return y.reshape(outer, -1)[:, at].reshape(_packed_shape(shape, first, d))


def work(case):
    esz = 8 if case["dtype"] == "f64" else 4
    kind, d = case["kind"], case["d"]
    terms = len(_expanded(operator(case["op"], d), d))
    if kind == "batched":
        n = sum(math.prod(s) for s in _blocks(case)[0])
        return {"bytes": 2 * n * esz, "flops": 2 * terms * n}
    shape, first = _shape(case)
    n = math.prod(shape)
    if kind in ("unpack", "pack"):
        packed = math.prod(_packed_shape(shape, first, d))
        return {"bytes": (n + packed) * esz,
                "flops": n if kind == "unpack" else 2 * terms * packed}
    if kind == "vjp":
        return {"bytes": 4 * n * esz, "flops": 4 * terms * n}
    if kind == "train":
        # the tensor and the gradient read once, the output and the tensor's
        # gradient written once
        return {"bytes": 4 * n * esz, "flops": 6 * terms * n}
    if kind == "cgrad":
        return {"bytes": 2 * n * esz, "flops": 2 * math.factorial(d) * n}
    return {"bytes": 2 * n * esz, "flops": 2 * terms * n}
