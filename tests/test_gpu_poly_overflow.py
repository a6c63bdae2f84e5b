"""Polynomial evaluation where one monomial overflows: what does not contain
it stays finite and agrees with the oracle (the lanes without a monomial add
nothing), and a derivative whose coefficient brings it back in range is
finite although its power times its exponent is not.

Bar: that of the other evaluation tests (4096 units of the precision times
the 64 terms an entry may sum).
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
@pytest.mark.parametrize("nmon", [5, 33])
@pytest.mark.parametrize("value", [2.0 ** 200, np.inf, np.nan])
def test_an_overflowing_monomial_stays_alone(L, nmon, value):
    s = inputs.polysys(neq=5, nvar=6, nmon=nmon, nvpm=2, maxdeg=3, L=L, system=2)
    s["vars"][s["vars"] == 0] = 3
    s["vars"][0, 0, 0], s["exps"][0, 0, 0] = 0, 16
    x = inputs.near_root(s, 1e-2, L=L, system=2)
    Fo, Jo = oracle.poly_eval(s, x)
    x[:, :, 0] = 0.0
    x[0, 0, 0] = value
    ds = api.PolySystem(s["vars"], s["exps"], s["coef"], 6, torch.device("cuda:0"))
    for batch in (1, 600):
        X = torch.from_numpy(x).cuda().expand(batch, *x.shape).contiguous()
        J, F = api.poly_eval(ds, X)
        torch.cuda.synchronize()
        J, F = J[-1].cpu().numpy(), F[-1].cpu().numpy()
        tol = 4096 * EPS[L] * 64
        assert np.max(np.abs(diff(F[:, :, 1:], Fo[:, :, 1:]))) <= tol
        assert np.max(np.abs(diff(J[:, :, :, 1:], Jo[:, :, :, 1:]))) <= tol * 3
        assert not np.isfinite(F[0, 0, 0])


@pytest.mark.parametrize("L", [1, 2, 4])
def test_a_derivative_brought_back_by_its_coefficient(L):
    # c x^16 with x = 2^68, c = 2^-100: 16 x^15 is 2^1024, c 16 x^15 is 2^924
    coef = np.zeros((L, 2, 1, 1))
    coef[0, 0] = 2.0 ** -100
    ds = api.PolySystem(np.zeros((1, 1, 1), int), np.full((1, 1, 1), 16), coef, 1, torch.device("cuda:0"))
    X = torch.zeros((1, L, 2, 1), dtype=torch.float64, device="cuda")
    X[0, 0, 0, 0] = 2.0 ** 68
    J, _ = api.poly_eval(ds, X)
    torch.cuda.synchronize()
    want = np.zeros((L, 2, 1, 1))
    want[0, 0] = 2.0 ** 924
    assert np.array_equal(J[0].cpu().numpy(), want)
