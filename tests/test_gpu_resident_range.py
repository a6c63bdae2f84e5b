"""The register-resident launch (dd, 64 < m <= 1024) on columns whose squared
norms are near the end of the range: its chain then goes by way of the
normalised column instead of the squared norm's reciprocal.

Bar: the same Q, R and y as without the powers of two, up to those, to the
rounding of n projections of a well-conditioned matrix (n columns, 4 eps
each, condition about 4, one factor 2 for either side).
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1210_0800_amd import api, inputs  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n", [(65, 12), (200, 20), (600, 9)])
def test_columns_near_the_end_of_the_range(m, n):
    p = inputs.random_problem(2, m, n, seed=21, config=98)
    e = np.zeros(n, int)
    e[0], e[3], e[4], e[n - 1] = 470, 440, -440, 480
    A2 = p["A"] * np.ldexp(1.0, e)[None, None, :, None]
    b = torch.from_numpy(p["b"]).cuda()
    f, g = api.mgs_qr(torch.from_numpy(p["A"]).cuda(), b), api.mgs_qr(torch.from_numpy(A2).cuda(), b)
    torch.cuda.synchronize()
    assert int(g["info"].item()) == 0
    back = {k: g[k].cpu().numpy() for k in ("Q", "R", "y")}
    back["R"] = back["R"] / np.ldexp(1.0, e)[None, None, :, None]
    for k, v in back.items():
        w = f[k].cpu().numpy()
        d = np.abs(sum(v[i] - w[i] for i in range(2)))
        assert float(d.max()) <= 32 * n * 2.0**-104 * max(1.0, float(np.abs(w[0]).max())), k
    for bad in (2.0**530, 0.0):
        A2 = p["A"].copy()
        A2[:, :, 5] *= bad
        h = api.mgs_qr(torch.from_numpy(A2).cuda(), b)
        torch.cuda.synchronize()
        assert int(h["info"].item()) == 6
