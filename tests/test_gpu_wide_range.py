"""Entries of one column, or of the right-hand side, that are hundreds of
powers of two apart: every entry of R, y and x keeps its own relative
accuracy where the projections do not mix them.

A is diagonal with a wide right-hand side (Q = I, R = A, y = b, x = b / a), or
upper triangular with one tiny entry above a huge diagonal one in its last
columns (Q = I, R = A).  Bar: 64 units of the precision per entry (a product
with a reciprocal, a projection and a division: fewer than 16 roundings).
"""
from fractions import Fraction as F

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1210_0800_amd import api, inputs  # noqa: E402
from tests._exact import EPS  # noqa: E402
from tests._parity import diff  # noqa: E402

pytestmark = pytest.mark.gpu


def one(g, prec):
    """A random real number in 1 .. 2 with all its limbs."""
    v = np.array([1.0] + [0.0] * (prec - 1))
    v[0] += g.uniform(0.0, 1.0)
    for l in range(1, prec):
        v[l] = v[l - 1] * 2.0 ** -54 * g.uniform(0.5, 1.0)
    return v


def diagonal(prec, m, n):
    g = inputs.rng(94, m + n, 5)
    A, b = np.zeros((prec, 2, n, m)), np.zeros((prec, 2, m))
    for j in range(n):
        A[:, 0, j, j] = one(g, prec)
        b[:, 0, j] = one(g, prec) * 2.0 ** (650 - 1300 * j // max(n - 1, 1))
    return A, b


def with_far_columns(prec, m, n):
    A, b = diagonal(prec, m, n)
    g = inputs.rng(94, m + n, 6)
    A[:, 0, n - 1, n - 1] *= 2.0 ** 300
    A[:, 0, n - 1, 0] = one(g, prec) * 2.0 ** -700
    A[:, 0, n - 2, n - 2] *= 2.0 ** 350
    A[:, 0, n - 2, 1] = one(g, prec) * 2.0 ** -600
    b[0, 0], b[1:] = 1.0, 0.0
    return A, b


def close(got, want, prec):
    d, w = np.abs(diff(got, want)), np.abs(want[0])
    assert np.all(d <= 64 * EPS[prec] * w), "%.3e" % np.max(d / np.where(w > 0, w, 1.0))


def check(A, b, Q, R, y, x, prec):
    n, m = A.shape[2:]
    I = np.zeros((prec, 2, n, m))
    I[0, 0, np.arange(n), np.arange(n)] = 1.0
    assert np.max(np.abs(diff(Q, I))) <= 64 * EPS[prec]
    close(R, A[:, :, :, :n], prec)
    if y is None:
        return
    close(y, b[:, :, :n], prec)
    k = np.arange(n)
    got, want, a = ([[F(float(v[i, 0, j])) for i in range(prec)] for j in k] for v in (x, b, A[:, :, k, k]))
    for xj, bj, aj in zip(got, want, a):
        assert abs(sum(xj) * sum(aj) - sum(bj)) <= 64 * F(EPS[prec]) * abs(sum(bj))


def N(t):
    return t.cpu().numpy()


@pytest.mark.parametrize("prec,m,n", [(1, 8, 8), (1, 30, 20), (1, 40, 35), (1, 64, 12), (2, 14, 14), (2, 32, 24),
                                      (2, 50, 20), (4, 30, 20)])
@pytest.mark.parametrize("batch", [1, 600])
@pytest.mark.parametrize("kind", [diagonal, with_far_columns])
def test_batched(prec, m, n, batch, kind):
    A, b = kind(prec, m, n)
    At = torch.from_numpy(A).cuda().expand(batch, *A.shape).contiguous()
    bt = torch.from_numpy(b).cuda().expand(batch, *b.shape).contiguous()
    f = api.lstsq_batched(At, bt, with_y=True, with_rho=True)
    torch.cuda.synchronize()
    assert int((f["info"] != 0).sum().item()) == 0
    Q, R, y, x = (N(f[k][-1]) for k in ("Q", "R", "y", "x"))
    check(A, b, Q, R, y if kind is diagonal else None, x, prec)


@pytest.mark.parametrize("m,n", [(20, 12), (100, 30), (300, 8), (700, 9)])
@pytest.mark.parametrize("kind", [diagonal, with_far_columns])
def test_qd_launch(m, n, kind):
    A, b = kind(4, m, n)
    f = api.lstsq(torch.from_numpy(A).cuda(), torch.from_numpy(b).cuda())
    torch.cuda.synchronize()
    assert int(f["info"].item()) == 0 and int(f["info_backsolve"].item()) == 0
    Q, R, y, x = (N(f[k]) for k in ("Q", "R", "y", "x"))
    check(A, b, Q, R, y if kind is diagonal else None, x, 4)


@pytest.mark.parametrize("prec,m,n", [(1, 20, 12), (2, 20, 12), (2, 50, 20), (4, 20, 12), (4, 300, 8)])
def test_right_hand_sides_at_the_ends_of_the_range(prec, m, n):
    p = inputs.random_problem(prec, m, n, seed=3, config=94)
    A = torch.from_numpy(p["A"]).cuda()
    ref = api.mgs_qr(A, torch.from_numpy(p["b"]).cuda())
    for e in (1015, -700):
        f = api.mgs_qr(A, torch.from_numpy(p["b"] * 2.0 ** e).cuda())
        torch.cuda.synchronize()
        assert int(f["info"].item()) == 0
        # (a power of two moves every operation's result by that power)
        assert torch.equal(f["y"] * 2.0 ** -e, ref["y"])
        assert torch.equal(f["Q"], ref["Q"]) and torch.equal(f["R"], ref["R"])
