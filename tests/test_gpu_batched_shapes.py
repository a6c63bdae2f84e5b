"""mgs_lstsq_batched picks its workgroup shape (waves per system, column slots
per wave) by batch size, rows and columns: a system's results must be
bitwise the same in every shape, with and without b, and the last system of
a large batch must be complete.  Sizes: one and the full number of row
groups and slots, and one past each.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1210_0800_amd import api, inputs  # noqa: E402

pytestmark = pytest.mark.gpu

SIZES = [(1, 1), (16, 16), (17, 4), (32, 32), (33, 32), (34, 33), (48, 40), (64, 63)]
CASES = [(p, m, n) for p in (1, 2, 4) for m, n in SIZES if 64 * m * n <= 162816 or p < 4]


@pytest.mark.parametrize("prec,m,n", CASES)
def test_results_do_not_depend_on_the_shape(prec, m, n):
    probs = [inputs.random_problem(prec, m, n, seed=s, config=97) for s in range(3)]
    A = torch.from_numpy(np.stack([p["A"] for p in probs])).cuda()
    b = torch.from_numpy(np.stack([p["b"] for p in probs])).cuda()
    ref = api.lstsq_batched(A, b, with_y=True, with_rho=True)
    qr = api.lstsq_batched(A)
    torch.cuda.synchronize()
    assert int((ref["info"] != 0).sum().item()) == 0
    for batch in (300, 515):
        idx = torch.arange(batch, device="cuda") % 3
        f = api.lstsq_batched(A[idx], b[idx], with_y=True, with_rho=True)
        g = api.lstsq_batched(A[idx])
        torch.cuda.synchronize()
        for k in ("Q", "R", "x", "y", "rho", "info"):
            assert torch.equal(f[k], ref[k][idx]), (batch, k)
        for k in ("Q", "R", "info"):
            assert torch.equal(g[k], qr[k][idx]), (batch, k)


@pytest.mark.parametrize("prec,m,n", [(1, 20, 12), (1, 42, 42), (1, 64, 63), (2, 32, 32), (2, 48, 40), (4, 30, 20)])
def test_powers_of_two(prec, m, n):
    """Columns and b times powers of two whose squares are still in range:
    the same Q, x, y and R up to those powers, to the precision's error bar
    (64 eps: no operation rounds differently but at the ends of the range);
    a column whose squares are out of range is refused, as is one after it
    that is fine."""
    eps = {1: 2.0**-52, 2: 2.0**-104, 4: 2.0**-208}[prec]
    p = inputs.random_problem(prec, m, n, seed=5, config=97)
    e = np.zeros(n, int)
    e[1], e[n // 2], e[n - 2], e[n - 1], eb = 480, 300, -350, 150, 400
    A2, b2 = p["A"] * np.ldexp(1.0, e)[None, None, :, None], p["b"] * 2.0**eb
    one = torch.from_numpy(np.stack([p["A"]])).cuda(), torch.from_numpy(np.stack([p["b"]])).cuda()
    f = api.lstsq_batched(*one, with_y=True, with_rho=True)
    for batch in (1, 300, 600):
        A = torch.from_numpy(A2).cuda().expand(batch, *A2.shape).contiguous()
        b = torch.from_numpy(b2).cuda().expand(batch, *b2.shape).contiguous()
        g = api.lstsq_batched(A, b, with_y=True, with_rho=True)
        torch.cuda.synchronize()
        assert int((g["info"] != 0).sum().item()) == 0
        back = {k: g[k][-1].cpu().numpy() for k in ("Q", "R", "x", "y", "rho")}
        back["R"] = back["R"] / np.ldexp(1.0, e)[None, None, :, None]
        back["x"] = back["x"] * np.ldexp(1.0, e - eb)
        back["y"], back["rho"] = back["y"] * 2.0**-eb, back["rho"] * 2.0**-eb
        for k, v in back.items():
            # limb by limb from the leading one: the difference is exact
            d = np.abs(sum(v[i] - f[k][0].cpu().numpy()[i] for i in range(prec)))
            assert float(d.max()) <= 64 * eps * max(1.0, float(np.abs(f[k][0].cpu().numpy()[0]).max())), (batch, k)
    A2 = p["A"].copy()
    A2[:, :, n // 2] *= 2.0**530
    for batch in (1, 600):
        A = torch.from_numpy(A2).cuda().expand(batch, *A2.shape).contiguous()
        assert int(api.lstsq_batched(A)["info"][-1].item()) == n // 2 + 1
