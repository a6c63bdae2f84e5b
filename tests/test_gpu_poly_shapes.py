"""Polynomial evaluation over its launch shapes: half-wave and whole-wave
equations (32 / 33 monomials), more variables than a half wave, exponents
past the power table, repeated variables in a monomial, odd equation counts;
against the oracle, and bitwise the same in a large batch.

Bar: that of the other evaluation tests (4096 units of the precision times
the 64 terms an entry may sum), times 4 for products up to 1.015^48 and the
first coefficients, and times the degree for the derivatives.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from paper_1210_0800_amd import api, inputs  # noqa: E402
from tests._exact import EPS  # noqa: E402
from tests._parity import diff  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,neq,nvar,nmon,nvpm,maxdeg", [
    (4, 3, 2, 1, 1, 9), (4, 5, 33, 32, 2, 7), (2, 33, 40, 32, 3, 8), (2, 5, 63, 33, 8, 2), (1, 64, 33, 64, 2, 16),
    (2, 1, 1, 5, 1, 3)])
def test_shapes_against_the_oracle(L, neq, nvar, nmon, nvpm, maxdeg):
    s = inputs.polysys(neq=neq, nvar=nvar, nmon=nmon, nvpm=nvpm, maxdeg=maxdeg, L=L, system=8)
    if nvpm > 1:
        s["vars"][0, 0, 1] = s["vars"][0, 0, 0]  # a repeated variable
        s["exps"][0, -1, 0] = 0
    X = np.stack([inputs.near_root(s, 1e-2, L=L, system=k) for k in range(3)])
    ds = api.PolySystem(s["vars"], s["exps"], s["coef"], nvar, torch.device("cuda:0"))
    Xt = torch.from_numpy(X).cuda()
    J, F = api.poly_eval(ds, Xt)
    idx = torch.arange(600, device="cuda") % 3
    Jb, Fb = api.poly_eval(ds, Xt[idx])
    torch.cuda.synchronize()
    assert torch.equal(Jb, J[idx]) and torch.equal(Fb, F[idx])
    tol = 4096 * EPS[L] * 64 * 4
    for p in range(3):
        Fo, Jo = oracle.poly_eval(s, X[p])
        assert np.max(np.abs(diff(F[p].cpu().numpy(), Fo))) <= tol
        assert np.max(np.abs(diff(J[p].cpu().numpy(), Jo))) <= tol * maxdeg
