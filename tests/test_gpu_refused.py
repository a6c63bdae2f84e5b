"""A column whose squared norm is out of range (infinite, or zero) is refused
by the factorisation; its diagonal entry of R is then no pivot, so that a
solve, a new right-hand side or a gradient with those factors is refused too,
naming the same column.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1210_0800_amd import api, inputs  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,m,n", [(1, 20, 12), (1, 50, 40), (1, 64, 10), (1, 90, 70), (2, 20, 12), (2, 50, 30),
                                      (2, 90, 70), (4, 20, 12), (4, 90, 70), (4, 300, 20)])
@pytest.mark.parametrize("scale", [2.0 ** 530, 2.0 ** -560, 0.0])
def test_factors_of_a_refused_matrix(prec, m, n, scale):
    p = inputs.random_problem(prec, m, n, seed=41, config=98)
    A, c = p["A"].copy(), n - 1  # the last one: what comes after it is unspecified
    A[:, :, c] *= scale
    At, b = torch.from_numpy(A).cuda(), torch.from_numpy(p["b"]).cuda()
    f = api.lstsq(At, b)
    _, info = api.ls_solve(f["Q"], f["R"], b)
    infos = [f["info"], f["info_backsolve"], info]
    if prec > 1:
        infos.append(api.ls_adjoint(At, b, f["Q"], f["R"], f["x"], f["x"])[2])
    torch.cuda.synchronize()
    assert [int(i.item()) for i in infos] == [c + 1] * len(infos)
