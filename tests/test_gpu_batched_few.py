"""Small systems of few columns on many rows (their own lane grids: at most 8
columns past the first on 17 to 32 and on more rows, 9 to 16 on more than 32):
at the edges of each and one past, against the oracle, bitwise the same in
every batch size, and bitwise under timing jitter.

Bars: the parity bars of the other small systems.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from paper_1210_0800_amd import api, inputs  # noqa: E402
from tests._parity import assert_parity, errors  # noqa: E402

pytestmark = pytest.mark.gpu

SIZES = [(17, 1), (17, 8), (32, 8), (32, 9), (33, 1), (33, 8), (33, 9), (33, 16), (33, 17), (64, 2), (64, 8), (64, 9),
         (64, 16)]


@pytest.mark.parametrize("prec", [1, 2, 4])
@pytest.mark.parametrize("m,n", SIZES)
def test_few_columns(prec, m, n):
    probs = [inputs.random_problem(prec, m, n, seed=s, config=97) for s in range(3)]
    A = torch.from_numpy(np.stack([p["A"] for p in probs])).cuda()
    b = torch.from_numpy(np.stack([p["b"] for p in probs])).cuda()
    ref = api.lstsq_batched(A, b, with_y=True, with_rho=True)
    qr = api.lstsq_batched(A)
    torch.cuda.synchronize()
    assert int((ref["info"] != 0).sum().item()) == 0
    for s, p in enumerate(probs):
        o = oracle.mgs(p["A"], p["b"])
        xo, _ = oracle.backsolve(o["R"], o["y"])
        Q, R, x = (ref[k][s].cpu().numpy() for k in ("Q", "R", "x"))
        assert_parity(errors(p["A"], Q, R, o["Q"], o["R"], x, xo, o["rho"]), prec)
    for batch in (300, 515):
        idx = torch.arange(batch, device="cuda") % 3
        f = api.lstsq_batched(A[idx], b[idx], with_y=True, with_rho=True)
        g = api.lstsq_batched(A[idx])
        torch.cuda.synchronize()
        for k in ("Q", "R", "x", "y", "rho", "info"):
            assert torch.equal(f[k], ref[k][idx]), (batch, k)
        for k in ("Q", "R", "info"):
            assert torch.equal(g[k], qr[k][idx]), (batch, k)
    try:
        api.set_jitter(0xDEADBEEF)
        f = api.lstsq_batched(A, b, with_y=True, with_rho=True)
        torch.cuda.synchronize()
    finally:
        api.set_jitter(0)
    for k in ("Q", "R", "x", "y", "rho", "info"):
        assert torch.equal(f[k], ref[k]), k
