"""The left-looking launch (qd, m <= 1024, what mgs_qr takes by itself) in each
of its shapes: that it is the kernel that runs, columns that cancel against an
earlier one with later columns projected against the remainder, both
hand-offs (Q apart from A, and in place) under timing jitter, several streams
at once, and captured in a graph.

Bars: kappa_2 of the scaled columns is about 2^k (within 2^4 for these
sizes), so Q and R agree with the oracle's to the parity bar times 2^(k+4).
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from paper_1210_0800_amd import api, inputs  # noqa: E402
from tests._parity import TAU, assert_parity, col_norms, diff, errors  # noqa: E402

pytestmark = pytest.mark.gpu

# one per shape: rows up to 64, 128, 256, 512 with few and many columns, 1024
SHAPES = [(60, 20), (100, 40), (200, 30), (400, 20), (400, 300), (600, 12)]


def T(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def N(t):
    return t.cpu().numpy()


@pytest.mark.parametrize("m,n", SHAPES)
def test_the_launch_runs(m, n):
    # its projections round differently from the other schedules'
    p = inputs.random_problem(4, m, n, seed=31, config=98)
    A, b = T(p["A"]), T(p["b"])
    f, g = api.mgs_qr(A, b), api.mgs_qr(A, b, schedule="panel")
    torch.cuda.synchronize()
    assert int(f["info"].item()) == 0
    assert not torch.equal(f["R"], g["R"]) and not torch.equal(f["Q"], g["Q"])
    assert_parity(errors(p["A"], N(f["Q"]), N(f["R"]), N(g["Q"]), N(g["R"])), 4, what=("err_q", "err_r"))


@pytest.mark.parametrize("m,n", [s for s in SHAPES if s[1] <= 40] + [(300, 291)])
@pytest.mark.parametrize("k", [60, 104, 130])
def test_near_dependent_columns(m, n, k):
    """Column n/2 = column 0 / 2 + 2^-k times a random column, exact in qd."""
    p = inputs.random_problem(4, m, n, seed=k, config=95)
    A, b, c = p["A"], p["b"], n // 2
    A[2:] = 0.0  # two limbs: the sum below fits four
    d = inputs.random_problem(1, m, 1, seed=k, config=96)["A"][0, :, 0]
    for part in range(2):
        limbs = [0.5 * A[0, part, 0], 0.5 * A[1, part, 0], d[part] * 2.0 ** -k, np.zeros(m)]
        limbs.sort(key=lambda v: -np.max(np.abs(v)))
        A[:, part, c] = np.stack(inputs.normalize(limbs))
    if n <= 40:
        o = oracle.mgs(A, b)
        assert o["info"] == 0
    else:  # (the per-panel schedule is checked on such columns elsewhere)
        g = api.mgs_qr(T(A), T(b), schedule="panel")
        o = dict(Q=N(g["Q"]), R=N(g["R"]))
    f = api.mgs_qr(T(A), T(b))
    torch.cuda.synchronize()
    assert int(f["info"].item()) == 0
    Q, R = N(f["Q"]), N(f["R"])
    for X in (Q, R):
        for i in range(3):
            assert np.all(np.abs(X[i + 1]) <= np.spacing(np.abs(X[i])))
    tol = TAU[4] * 2.0 ** (k + 4)
    dQ, dR = diff(Q, o["Q"]), diff(R, o["R"])
    assert np.max(np.sqrt(np.sum(dQ ** 2, axis=(0, 2)))) <= tol
    assert np.max(np.sqrt(np.sum(dR ** 2, axis=(0, 2))) / col_norms(A)) <= tol


@pytest.mark.parametrize("m,n", SHAPES)
@pytest.mark.parametrize("in_place", [False, True])
def test_bitwise_under_jitter(m, n, in_place):
    p = inputs.random_problem(4, m, n, seed=33, config=98)
    A, b = T(p["A"]), T(p["b"])

    def run():
        At = A.clone()
        f = api.mgs_qr(At, b, Q=At if in_place else None)
        torch.cuda.synchronize()
        return f

    try:
        out = []
        for seed in (0, 1, 0xDEADBEEF):
            api.set_jitter(seed)
            out.append(run())
    finally:
        api.set_jitter(0)
    for f in out[1:]:
        for k in ("Q", "R", "y", "rho", "info"):
            assert torch.equal(f[k], out[0][k]), k


def test_several_streams_at_once():
    shapes = [(60, 50), (100, 90), (300, 290), (600, 40)]
    probs = [inputs.random_problem(4, m, n, seed=35, config=98) for m, n in shapes]
    data = [(T(p["A"]), T(p["b"])) for p in probs]
    ref = [api.lstsq(A, b) for A, b in data]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in data]
    out = []
    for _ in range(3):
        for s, (A, b) in zip(streams, data):
            with torch.cuda.stream(s):
                out.append(api.lstsq(A, b))
    torch.cuda.synchronize()
    for i, f in enumerate(out):
        for k in ("Q", "R", "y", "x", "rho", "info"):
            assert torch.equal(f[k], ref[i % len(ref)][k]), (i, k)


def test_captured():
    m, n = 150, 140
    probs = [inputs.random_problem(4, m, n, seed=s, config=98) for s in (37, 38, 39)]
    ref = [api.mgs_qr(T(p["A"]), T(p["b"])) for p in probs]
    A, b = T(probs[0]["A"]), T(probs[0]["b"])
    out = api.mgs_qr_noalloc(A, b)
    x, info = api.ls_backsolve(out["R"], out["y"])
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        api.mgs_qr_noalloc(A, b, Q=out["Q"], R=out["R"], y=out["y"], rho=out["rho"], info=out["info"])
        api.ls_backsolve(out["R"], out["y"], x=x, info=info)
    for i in (0, 1, 2, 1, 0):
        A.copy_(T(probs[i]["A"]))
        b.copy_(T(probs[i]["b"]))
        out["R"].fill_(7.0)
        graph.replay()
        torch.cuda.synchronize()
        for k in ("Q", "R", "y", "rho", "info"):
            assert torch.equal(out[k], ref[i][k]), (i, k)
        assert torch.equal(x, api.ls_backsolve(ref[i]["R"], ref[i]["y"])[0])
