"""qd columns that cancel against an earlier one by 2^-k, k past one, near two
and past two limbs: the sums that stay in level words until their value is
taken must still give normalised limbs whose leading one is the rounded
value, on every schedule.

Bar: kappa_2 of the scaled columns is about 2^k (within 2^4 for these
sizes), so Q and R agree with the oracle's to the parity bar times 2^(k+4).
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from paper_1210_0800_amd import api, inputs  # noqa: E402
from tests._parity import TAU, col_norms, diff  # noqa: E402

pytestmark = pytest.mark.gpu


def near_dependent(m, n, k):
    """Column n-1 = column 0 / 2 + 2^-k times a random column, exact in qd."""
    p = inputs.random_problem(4, m, n, seed=k, config=95)
    A = p["A"]
    A[2:] = 0.0  # two limbs: the sum below fits four
    d = inputs.random_problem(1, m, 1, seed=k, config=96)["A"][0, :, 0]
    for part in range(2):
        limbs = [0.5 * A[0, part, 0], 0.5 * A[1, part, 0], d[part] * 2.0 ** -k, np.zeros(m)]
        limbs.sort(key=lambda v: -np.max(np.abs(v)))
        A[:, part, n - 1] = np.stack(inputs.normalize(limbs))
    return A, p["b"]


def assert_normalised(X):
    for i in range(X.shape[0] - 1):
        assert np.all(np.abs(X[i + 1]) <= np.spacing(np.abs(X[i])))


@pytest.mark.parametrize("m,n", [(24, 6), (70, 5)])
@pytest.mark.parametrize("k", [60, 104, 130])
def test_near_dependent_columns(m, n, k):
    A, b = near_dependent(m, n, k)
    o = oracle.mgs(A, b)
    assert o["info"] == 0
    for sched in ("panel",) if m > 64 else ("panel", "small"):
        f = api.mgs_qr(torch.from_numpy(A).cuda(), torch.from_numpy(b).cuda(), schedule=sched)
        torch.cuda.synchronize()
        assert int(f["info"].item()) == 0
        Q, R = f["Q"].cpu().numpy(), f["R"].cpu().numpy()
        assert_normalised(Q)
        assert_normalised(R)
        tol = TAU[4] * 2.0 ** (k + 4)
        dQ, dR = diff(Q, o["Q"]), diff(R, o["R"])
        assert np.max(np.sqrt(np.sum(dQ ** 2, axis=(0, 2)))) <= tol
        assert np.max(np.sqrt(np.sum(dR ** 2, axis=(0, 2))) / col_norms(A)) <= tol
