"""The triangular solves at the edges of their shapes (32 rows per wave, 256
per workgroup): back substitution in every precision and, through the
adjoint, the forward substitution, against the oracle; bitwise under timing
jitter across workgroups; first bad diagonal entry.

R is 2 on the diagonal plus entries of size 1 / n above it, so kappa is below
10 and the solutions agree to the precision's parity bar.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from paper_1210_0800_amd import api, inputs  # noqa: E402
from tests._parity import TAU, diff  # noqa: E402

pytestmark = pytest.mark.gpu


def T(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def triangular(prec, n, seed):
    g = inputs.rng(94, seed, 0)
    R = inputs.random_complex(g, (n, n), prec) * 2.0 ** -int(np.ceil(np.log2(n)) if n > 1 else 0)
    for j in range(n):
        R[:, :, j, j:] = 0.0  # column j, rows from j on
        R[0, 0, j, j] = 2.0
    return np.ascontiguousarray(R), inputs.random_complex(inputs.rng(94, seed, 2), (n,), prec)


def rel(x, xo):
    return np.sqrt(np.sum(diff(x, xo) ** 2) / np.sum(xo[0] ** 2))


@pytest.mark.parametrize("prec", [1, 2, 4])
@pytest.mark.parametrize("n", [1, 2, 31, 32, 33, 65, 127, 128, 129, 300, 513])
def test_back_substitution(prec, n):
    R, y = triangular(prec, n, n)
    x, info = api.ls_backsolve(T(R), T(y))
    torch.cuda.synchronize()
    assert int(info.item()) == 0
    xo, _ = oracle.backsolve(R, y)
    assert rel(x.cpu().numpy(), xo) <= TAU[prec]


@pytest.mark.parametrize("prec,n", [(2, 1), (2, 33), (2, 129), (2, 300), (4, 31), (4, 65), (4, 270)])
def test_forward_substitution_by_the_adjoint(prec, n):
    # Q = [I 0]^T: gb = Q w is (w, 0), w = R^{-H} g
    m = n + 3
    R, g = triangular(prec, n, 1000 + n)
    Q = np.zeros((prec, 2, n, m))
    Q[0, 0, np.arange(n), np.arange(n)] = 1.0
    A = np.zeros_like(Q)
    A[:, :, :, :n] = R
    b = np.zeros((prec, 2, m))
    x = np.zeros((prec, 2, n))
    _, gb, info = api.ls_adjoint(T(A), T(b), T(Q), T(R), T(x), T(g))
    torch.cuda.synchronize()
    assert int(info.item()) == 0
    # R^H w = g is the back substitution of the flipped, conjugated system
    F = np.ascontiguousarray(np.transpose(R, (0, 1, 3, 2))[:, :, ::-1, ::-1]).copy()
    F[:, 1] = -F[:, 1]
    F = np.ascontiguousarray(F)
    wo, _ = oracle.backsolve(F, np.ascontiguousarray(g[:, :, ::-1]))
    wo = np.ascontiguousarray(wo[:, :, ::-1])
    w = gb.cpu().numpy()
    assert rel(w[:, :, :n], wo) <= TAU[prec] and np.all(w[:, :, n:] == 0)


@pytest.mark.parametrize("prec", [1, 2, 4])
def test_bitwise_under_jitter(prec):
    R, y = triangular(prec, 600, 77)
    Rt, yt = T(R), T(y)
    try:
        out = []
        for seed in (0, 1, 0xDEADBEEF):
            api.set_jitter(seed)
            out.append(api.ls_backsolve(Rt, yt)[0])
            torch.cuda.synchronize()
    finally:
        api.set_jitter(0)
    assert torch.equal(out[0], out[1]) and torch.equal(out[0], out[2])


@pytest.mark.parametrize("n,bad", [(40, 0), (40, 39), (300, 17), (300, 280)])
def test_first_bad_diagonal(n, bad):
    R, y = triangular(2, n, 5)
    R[:, :, bad, bad] = 0.0
    R[0, 0, n - 1, n - 1] = np.nan if bad < n - 1 else 0.0
    _, info = api.ls_backsolve(T(R), T(y))
    torch.cuda.synchronize()
    assert int(info.item()) == bad + 1


@pytest.mark.parametrize("prec,m,n", [(1, 1, 1), (1, 512, 9), (1, 513, 7), (1, 1025, 6), (1, 2049, 5), (2, 512, 6),
                                      (2, 1025, 5), (2, 2049, 3), (4, 65, 7), (4, 600, 5), (4, 1100, 3)])
def test_projections_of_a_new_right_hand_side(prec, m, n):
    p = inputs.random_problem(prec, m, n, seed=m + n, config=93)
    o = oracle.mgs(p["A"], p["b"])
    x, info = api.ls_solve(T(o["Q"]), T(o["R"]), T(p["b"]))
    torch.cuda.synchronize()
    assert int(info.item()) == 0
    xo, _ = oracle.ls_solve(o["Q"], o["R"], p["b"])
    # kappa below 100 at these shapes, relative to ||x|| + ||b|| / sigma_min
    assert rel(x.cpu().numpy(), xo) <= 100 * TAU[prec]
