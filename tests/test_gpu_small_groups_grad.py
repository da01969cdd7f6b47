"""Both gradients of a backward pass on the smallest groups, whose tiles take
fewer bytes of LDS than the sums of a workgroup's waves: the tensor's gradient
bit for bit that of spinsum_adjoint, the coefficients' against the oracle, and
the same through SpinSumCoefFunction.

Bars: coefficient gradients 1e-12 of sum |g| |x|, the bound of every
coefficient (sums in double on the same values, fewer than 1e6 terms)."""
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


def _terms(d):
    return [[(p, 0.5 + 0.25 * i) for i, p in enumerate(itertools.permutations(range(d)))]]


@pytest.mark.parametrize("cubes", [1, 100, 5000])
@pytest.mark.parametrize("dtype", [F64, F32])
@pytest.mark.parametrize("d", [2, 3])
def test_small_groups(d, dtype, cubes):
    for n in (1, 2, 3, 4):
        for inner in ((), (3,)):
            shape = (cubes,) + (n,) * d + inner
            for inplace in (False, True):
                p = ss.spinsum_plan(shape, 1, d, _terms(d), dtype=dtype, inplace=inplace)
                x = workloads.uniform(shape, 9300 + n, device=DEV, dtype=dtype)
                g = workloads.uniform(shape, 9400 + n, device=DEV, dtype=dtype)
                want = g.clone() if inplace else torch.empty_like(g)
                ss.spinsum_adjoint(p, want if inplace else g, want)
                got = g.clone() if inplace else torch.full_like(g, 3.0)
                c = ss.spinsum_adjoint_coef_grad(p, x, got if inplace else g, got)
                torch.cuda.synchronize()
                assert torch.equal(got, want), (shape, inplace)
                xh, gh = x.cpu().to(F64).numpy(), g.cpu().to(F64).numpy()
                ref = oracle.coef_grad(xh, gh, 1, d)
                assert np.max(np.abs(c.cpu().numpy() - ref)) <= 1e-12 * np.sum(np.abs(xh)) * np.max(np.abs(gh))


@pytest.mark.parametrize("n", [2, 3])
def test_small_groups_autograd(n):
    perms = list(itertools.permutations(range(3)))
    shape = (7, n, n, n)
    x = workloads.uniform(shape, 9500, device=DEV, dtype=F32).requires_grad_()
    g = workloads.uniform(shape, 9501, device=DEV, dtype=F32)
    alpha = torch.tensor([0.5 + 0.25 * i for i in range(6)], dtype=F32, device=DEV, requires_grad=True)
    ss.SpinSumCoefFunction.apply(x, alpha, perms, 1).backward(g)
    p = ss.spinsum_plan(shape, 1, 3, _terms(3), dtype=F32)
    want = ss.spinsum_adjoint(p, g, torch.empty_like(g))
    torch.cuda.synchronize()
    assert torch.equal(x.grad, want)
