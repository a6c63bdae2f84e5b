"""Every exponent 0..16 on its own, at a point whose powers are exact: past the
kept powers x^1..x^6 a power is a product of two or three of them.  And every
place of a variable among the factors of an equation's monomials, with as many
variables as lanes, one more and the most, so that each lane's list is used.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from paper_1210_0800_amd import api, inputs  # noqa: E402
from tests._exact import EPS  # noqa: E402
from tests._parity import diff  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L", [1, 2, 4])
def test_every_exponent(L):
    exps = np.arange(17).reshape(17, 1, 1)
    coef = np.zeros((L, 2, 17, 1))
    coef[0, 0] = 1.0
    ds = api.PolySystem(np.zeros((17, 1, 1), int), exps, coef, 1, torch.device("cuda:0"))
    X = torch.zeros((1, L, 2, 1), dtype=torch.float64, device="cuda")
    X[0, 0, 0, 0] = 1.5
    J, F = api.poly_eval(ds, X)
    torch.cuda.synchronize()
    d = np.arange(17)
    assert np.array_equal(F[0, 0, 0].cpu().numpy(), 1.5 ** d)
    assert np.array_equal(J[0, 0, 0, 0].cpu().numpy(), d * 1.5 ** (d - 1.0))
    assert bool((F[0, 1:] == 0).all()) and bool((J[0, :, 1] == 0).all())


@pytest.mark.parametrize("L,nvar,nmon,nvpm", [(1, 32, 32, 4), (2, 33, 32, 3), (1, 63, 64, 8), (4, 63, 33, 2), (1, 1, 64, 8)])
def test_every_variable_and_place(L, nvar, nmon, nvpm):
    neq = 3
    s = inputs.polysys(neq=neq, nvar=nvar, nmon=nmon, nvpm=min(nvpm, nvar), maxdeg=2, L=L, system=9)
    e, m, t = np.meshgrid(np.arange(neq), np.arange(nmon), np.arange(nvpm), indexing="ij")
    s["vars"] = ((e + m * nvpm + t) % nvar).astype(np.int32)  # repeated within a monomial where nvar < nvpm
    s["exps"] = (1 + (e + m + t) % 2).astype(np.int32)
    x = inputs.near_root(s, 1e-2, L=L, system=9)
    Fo, Jo = oracle.poly_eval(s, x)
    ds = api.PolySystem(s["vars"], s["exps"], s["coef"], nvar, torch.device("cuda:0"))
    J, F = api.poly_eval(ds, torch.from_numpy(x[None]).cuda())
    torch.cuda.synchronize()
    # 4096 units times the terms of an entry (64 monomials, 8 factors of degree
    # 2), products up to 1.015^16 and coefficients up to 64 / 64 and the first
    tol = 4096 * EPS[L] * 64 * 16 * 2 * max(1.0, float(np.abs(s["coef"][0]).max()))
    assert np.max(np.abs(diff(F[0].cpu().numpy(), Fo))) <= tol
    assert np.max(np.abs(diff(J[0].cpu().numpy(), Jo))) <= tol
