"""The left-looking single launch (qd, m <= 1024, the automatic schedule):
against the oracle at the edges of its shapes (rows 64 / 65, 128 / 129, 256 /
257, 512 / 513; one column, more columns than workgroups), in place (its
other hand-off), with leading dimensions beyond m, bitwise under timing
jitter, and with a bad column.

Bars: those of the other qd parity tests.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from paper_1210_0800_amd import _lib, api, inputs  # noqa: E402
from tests._parity import assert_parity, diff, errors  # noqa: E402

pytestmark = pytest.mark.gpu


def T(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def N(t):
    return t.cpu().numpy()


@pytest.mark.parametrize("m,n", [(1, 1), (7, 1), (64, 30), (65, 30), (129, 20), (257, 12), (513, 6), (300, 290)])
def test_against_oracle_and_in_place(m, n):
    p = inputs.random_problem(4, m, n, seed=m + n, config=98)
    A, b = p["A"], p["b"]
    o = oracle.mgs(A, b)
    xo, _ = oracle.backsolve(o["R"], o["y"])
    f = api.lstsq(T(A), T(b))
    torch.cuda.synchronize()
    assert int(f["info"].item()) == 0
    Q, R = N(f["Q"]), N(f["R"])
    assert_parity(errors(A, Q, R, o["Q"], o["R"], N(f["x"]), xo, o["rho"]), 4)
    il = np.tril_indices(n, -1)
    assert np.all(R[:, :, il[1], il[0]] == 0) and np.all(R[:, 1, np.arange(n), np.arange(n)] == 0)
    nb = np.sqrt(np.sum(b[0] ** 2))
    assert abs(float(diff(N(f["rho"])[:, None], o["rho"][:, None])[0])) <= 1e-57 * nb
    # in place, without b: the other hand-off, the same bits
    At = T(A)
    g = api.mgs_qr(At, Q=At)
    torch.cuda.synchronize()
    assert torch.equal(At, f["Q"]) and torch.equal(g["R"], f["R"])


def test_more_columns_than_workgroups():
    m, n = 600, 560  # two workgroups per compute unit, 512 of them
    p = inputs.random_problem(4, m, n, seed=3, config=98)
    A, b = T(p["A"]), T(p["b"])
    f = api.mgs_qr(A, b)
    g = api.mgs_qr(A, b, schedule="panel")
    torch.cuda.synchronize()
    assert int(f["info"].item()) == 0
    assert_parity(errors(p["A"], N(f["Q"]), N(f["R"]), N(g["Q"]), N(g["R"])), 4, what=("err_q", "err_r"))
    At = A.clone()
    api.mgs_qr(At, b, Q=At)
    torch.cuda.synchronize()
    assert torch.equal(At, f["Q"])


def test_leading_dimensions():
    m, n, ld = 70, 9, 75
    p = inputs.random_problem(4, m, n, seed=5, config=98)
    Ap = torch.full((4, 2, n, ld), 7.0, dtype=torch.float64, device="cuda")
    Ap[..., :m] = T(p["A"])
    Q = torch.full_like(Ap, -3.0)
    R = torch.full((4, 2, n, n + 2), -3.0, dtype=torch.float64, device="cuda")
    info = torch.empty(1, dtype=torch.int32, device="cuda")
    work = api.workspace(m, n, 4, _lib.MGS_OP_QR, Ap.device)
    st = _lib.lib().mgs_qr(m, n, 4, Ap.data_ptr(), ld, Q.data_ptr(), ld, R.data_ptr(), n + 2, None, None, None,
                           work.data_ptr(), work.numel() * 8, info.data_ptr(), torch.cuda.current_stream().cuda_stream)
    assert st == 0
    f = api.mgs_qr(T(p["A"]))
    torch.cuda.synchronize()
    assert torch.equal(Q[..., :m], f["Q"]) and bool((Q[..., m:] == -3.0).all())
    assert torch.equal(R[..., :n], f["R"]) and bool((R[..., n:] == -3.0).all())


def test_bitwise_under_jitter():
    p = inputs.random_problem(4, 140, 90, seed=9, config=98)
    A, b = T(p["A"]), T(p["b"])
    try:
        out = []
        for seed in (0, 1, 0xDEADBEEF):
            api.set_jitter(seed)
            out.append(api.mgs_qr(A, b))
            torch.cuda.synchronize()
    finally:
        api.set_jitter(0)
    for f in out[1:]:
        for k in ("Q", "R", "y", "rho", "info"):
            assert torch.equal(f[k], out[0][k]), k


def test_bad_columns():
    p = inputs.random_problem(4, 100, 30, seed=11, config=98)
    for col, value in ((0, 0.0), (17, 0.0), (29, np.nan)):
        A = p["A"].copy()
        A[:, :, col] = 0.0
        A[0, 0, col, 3] = value
        f = api.mgs_qr(T(A), T(p["b"]))
        torch.cuda.synchronize()
        assert int(f["info"].item()) == col + 1
    # a raw entry with the bits of the hand-off's empty marker
    A = p["A"].copy()
    A[0, 0, 0, 5] = np.array([0x7FF4A5A5A5A5A5A5], dtype=np.uint64).view(np.float64)[0]
    f = api.mgs_qr(T(A), T(p["b"]))
    torch.cuda.synchronize()
    assert int(f["info"].item()) == 1


@pytest.mark.parametrize("m,n", [(40, 20), (100, 30), (600, 8)])
def test_columns_near_the_end_of_the_range(m, n):
    # columns times powers of two whose squares are still in range: the same
    # Q, y and R up to those powers (64 eps: no operation rounds differently);
    # a column whose squares are out of range is refused
    p = inputs.random_problem(4, m, n, seed=15, config=98)
    e = np.zeros(n, int)
    e[0], e[n // 2], e[n - 2], e[n - 1] = 490, 480, -250, 300
    A2 = p["A"] * np.ldexp(1.0, e)[None, None, :, None]
    f, g = api.mgs_qr(T(p["A"]), T(p["b"])), api.mgs_qr(T(A2), T(p["b"]))
    torch.cuda.synchronize()
    assert int(g["info"].item()) == 0
    back = {k: N(g[k]) for k in ("Q", "R", "y", "rho")}
    assert np.all(back["R"][:, 1, np.arange(n), np.arange(n)] == 0)
    back["R"] = back["R"] / np.ldexp(1.0, e)[None, None, :, None]
    for k, v in back.items():
        w = N(f[k])
        d = np.abs(sum(v[i] - w[i] for i in range(4)))
        assert float(d.max()) <= 64 * 2.0**-208 * max(1.0, float(np.abs(w[0]).max())), k
    A2 = p["A"].copy()
    A2[:, :, n // 2] *= 2.0**530
    g = api.mgs_qr(T(A2), T(p["b"]))
    torch.cuda.synchronize()
    assert int(g["info"].item()) == n // 2 + 1
