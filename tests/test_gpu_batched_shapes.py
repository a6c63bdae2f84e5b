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
