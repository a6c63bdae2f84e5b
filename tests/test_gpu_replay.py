"""The refinement's projections of a residual, in one launch per step: rows at
the edges of its workgroups (64 rows each), columns at the edges of its waves'
shares and panels (16, 64), one workgroup and several, one panel to more than
its three exchange buffers.

Bar: x back from b = A x (exact in FP64) to the bar of the other refinement
tests; bitwise the same under timing jitter.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1210_0800_amd import api, inputs  # noqa: E402
from tests._parity import diff  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n", [(1, 1), (64, 64), (64, 15), (65, 17), (66, 66), (127, 64), (129, 128), (300, 257),
                                 (2049, 40)])
def test_replay_edges(m, n):
    p = inputs.random_problem(2, m, n, seed=m, config=96)
    # entries of 20 bits and x of 6: b = A x is exact in FP64
    A0, x0 = np.round(p["A"][0] * 2.0**20) / 2.0**20, np.round(p["b"][0][:, np.arange(n) % m] * 64.0) / 64.0
    x0[0, 0] = 0.5
    Ac, xc = A0[0] + 1j * A0[1], x0[0] + 1j * x0[1]  # Ac[j, i] is A(i, j)
    bc = (Ac * xc[:, None]).sum(axis=0)
    A, b, x = np.zeros((2, 2, n, m)), np.zeros((2, 2, m)), np.zeros((2, 2, n))
    A[0], b[0], x[0] = A0, np.stack([bc.real, bc.imag]), x0
    A, b = torch.from_numpy(A).cuda(), torch.from_numpy(b).cuda()
    f = api.refine_lstsq(A, b, max_iter=20)
    torch.cuda.synchronize()
    assert int(f["info"].item()) == 0
    err = np.abs(diff(f["x"].cpu().numpy(), x)).max() / np.abs(x[0]).max()
    assert err <= 1e-27
    try:
        for seed in (1, 0xDEADBEEF):
            api.set_jitter(seed)
            h = api.refine_lstsq(A, b, max_iter=20)
            torch.cuda.synchronize()
            assert torch.equal(h["x"], f["x"]) and torch.equal(h["iters"], f["iters"])
    finally:
        api.set_jitter(0)
