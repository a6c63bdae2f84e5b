"""The work that programs have this library do, as cases to be timed.

A case is one call (or one call and its gradient) through the public entry
points of `paper_1210_0800_amd.api`:

* ``lstsq``    x = argmin ||b - A x|| by MGS on [A b] and back substitution,
* ``grad``     the same through autograd, with the gradients of A and b,
* ``solve``    a new right-hand side against factors that are kept,
* ``refine``   the precision form (FP64 factors, dd / qd refinement),
* ``batched``  many independent small systems in one call,
* ``newton``   Newton corrector steps of a polynomial system at a batch of
  points (the path tracker's inner loop),

in complex double (prec 1), double-double (2) and quad-double (4).
"""
import math

import numpy as np
import torch

from paper_1210_0800_amd import api, inputs


def listed():
    return [
        # The smallest system in use (the paper's smallest size) in double:
        # nothing but latency and launches.
        dict(name="lstsq_d_32", op="lstsq", prec=1, m=32, n=32, spread=0.0),
        # The corrector of one path in double-double: a serial chain of 32 x 32
        # solves, each needed before the next can start.
        dict(name="newton_dd_1path", op="newton", prec=2, n=32, batch=1, iters=5),
        # The paper's middle size, quad-double.
        dict(name="lstsq_qd_80", op="lstsq", prec=4, m=80, n=80, spread=0.0),
        # A new right-hand side for kept factors, odd tall shape, double.
        dict(name="solve_d_700x500", op="solve", prec=1, m=700, n=500, spread=0.0),
        # Fitting inside a differentiable program: forward and adjoint.
        dict(name="grad_dd_512x384", op="grad", prec=2, m=512, n=384, spread=0.0),
        # Overdetermined fit in quad-double.
        dict(name="lstsq_qd_320x256", op="lstsq", prec=4, m=320, n=256, spread=0.0),
        # The Jacobian of a system of high degree (columns of very different
        # size), the benchmark's own workload.
        dict(name="lstsq_dd_1024", op="lstsq", prec=2, m=1024, n=1024, spread=12.0),
        # The largest plain solve: quad-double, 1024 columns.
        dict(name="lstsq_qd_1024", op="lstsq", prec=4, m=1024, n=1024, spread=0.0),
        # The precision form at its benchmark's size and condition, and at an
        # odd size in quad-double.
        dict(name="refine_dd_2048", op="refine", prec=2, n=2048, cond=1e10),
        dict(name="refine_qd_1025", op="refine", prec=4, n=1025, cond=1e6),
        # Many small independent systems: throughput of the whole card.
        dict(name="batched_dd_32", op="batched", prec=2, m=32, n=32, batch=10000),
        # The corrector over many paths at once in quad-double.
        dict(name="newton_qd_1024paths", op="newton", prec=4, n=32, batch=1024, iters=3),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["lstsq", "lstsq", "grad", "solve", "refine", "batched", "newton"])
    prec = rng.choice([1, 2, 4])
    if op in ("lstsq", "solve", "grad"):
        if op == "grad":
            prec = rng.choice([2, 4])
        n = _log(rng, 8, {1: 1400, 2: 1024, 4: 600}[prec])
        m = min(int(n * rng.choice([1.0, rng.uniform(1.0, 1.6)])), {1: 2048, 2: 1400, 4: 900}[prec])
        return dict(op=op, prec=prec, m=m, n=n, spread=rng.choice([0.0, 6.0]) if op == "lstsq" else 0.0)
    if op == "refine":
        return dict(op=op, prec=rng.choice([2, 4]), n=_log(rng, 100, 2048), cond=10.0 ** rng.randint(2, 9))
    if op == "batched":
        n = rng.randint(6, 48)
        return dict(op=op, prec=prec, m=min(n + rng.choice([0, 0, rng.randint(1, 12)]), 52), n=n,
                    batch=_log(rng, 50, {1: 10000, 2: 8000, 4: 2500}[prec]))
    return dict(op=op, prec=prec, n=rng.randint(8, 44), batch=_log(rng, 1, {1: 1024, 2: 1024, 4: 512}[prec]),
                iters=rng.randint(1, 5))


# ------------------------------------------------------------------ inputs --
def _gen(seed, dev):
    g = torch.Generator(device=dev)
    g.manual_seed(int(seed))
    return g


def _uniform(g, shape, dev):
    return torch.rand(shape, generator=g, device=dev, dtype=torch.float64) * 2.0 - 1.0


def _limbs(hi, prec, g):
    """Planar limbs [prec, ...] under leading limbs `hi`: each at most half a
    unit in the last place of the one above."""
    out = [hi]
    for _ in range(1, prec):
        out.append(out[-1] * 2.0 ** -54 * _uniform(g, hi.shape, hi.device))
    return torch.stack(out).contiguous()


def _system(case, seed, dev):
    g = _gen(seed, dev)
    m, n, prec = case["m"], case["n"], case["prec"]
    hi = _uniform(g, (2, n, m), dev)
    if case["spread"]:
        s = 10.0 ** (_uniform(g, (1, n, 1), dev) * case["spread"])
        hi = hi * s
    return _limbs(hi, prec, g), _limbs(_uniform(g, (2, m), dev), prec, g), g


def _poly(case, seed):
    n, prec = case["n"], case["prec"]
    s = inputs.polysys(neq=n, nvar=n, nmon=32, nvpm=5, maxdeg=5, L=prec, system=int(seed))
    r = np.random.default_rng([12100800, 77, int(seed)])
    x = np.zeros((case["batch"], prec, 2, n))
    x[:, 0] = s["root"][0] + 1e-3 * r.uniform(-1.0, 1.0, (case["batch"], 2, n))
    return s, x


def prepare(case, seed):
    dev = torch.device("cuda:0")
    op, prec = case["op"], case["prec"]
    if op == "newton":
        s, x = _poly(case, seed)
        return dict(case=case, system=api.PolySystem(s["vars"], s["exps"], s["coef"], s["nvar"], dev),
                    x0=torch.from_numpy(x).to(dev))
    if op == "batched":
        g = _gen(seed, dev)
        B, m, n = case["batch"], case["m"], case["n"]
        A = _limbs(_uniform(g, (B, 2, n, m), dev), prec, g).transpose(0, 1).contiguous()
        b = _limbs(_uniform(g, (B, 2, m), dev), prec, g).transpose(0, 1).contiguous()
        return dict(case=case, A=A, b=b)
    if op == "refine":
        g, n = _gen(seed, dev), case["n"]
        sig = torch.pow(torch.tensor(case["cond"], dtype=torch.float64, device=dev),
                        -torch.arange(n, device=dev, dtype=torch.float64) / (n - 1.0))
        M = torch.diag(sig).to(torch.complex128)
        for k in range(6):  # Householder reflectors on both sides: M keeps the singular values
            v = torch.complex(_uniform(g, (n, 1), dev), _uniform(g, (n, 1), dev))
            c = 2.0 / (v.real.square() + v.imag.square()).sum()
            M = M - c * (M @ v) @ v.conj().T if k % 2 else M - c * v @ (v.conj().T @ M)
        hi = torch.stack([M.real.T, M.imag.T]).contiguous()  # [2, column, row]
        return dict(case=case, A=_limbs(hi, prec, g), b=_limbs(_uniform(g, (2, n), dev), prec, g))
    A, b, g = _system(case, seed, dev)
    if op == "solve":  # the factors a program keeps
        f = api.mgs_qr(A)
        return dict(case=case, Q=f["Q"], R=f["R"], b=b)
    if op == "grad":
        A.requires_grad_(True)
        b.requires_grad_(True)
        return dict(case=case, A=A, b=b, gx=_limbs(_uniform(g, (2, case["n"]), dev), prec, g))
    return dict(case=case, A=A, b=b)


# ------------------------------------------------------------------- calls --
def run(state):
    case = state["case"]
    op = case["op"]
    if op == "lstsq":
        f = api.lstsq(state["A"], state["b"])
        out = dict(x=f["x"], Q=f["Q"], R=f["R"], y=f["y"], info=f["info"], info_backsolve=f["info_backsolve"])
        if case["m"] > case["n"]:
            out["rho"] = f["rho"]  # (of a square system it is rounding noise)
        return out
    if op == "grad":
        x = api.LstsqFn.apply(state["A"], state["b"])
        gA, gb = torch.autograd.grad(x, (state["A"], state["b"]), state["gx"])
        return dict(x=x, gA=gA, gb=gb)
    if op == "solve":
        x, info = api.ls_solve(state["Q"], state["R"], state["b"])
        return dict(x=x, info=info)
    if op == "refine":
        # (iters and err_est tell how it went, not the answer)
        f = api.refine_lstsq(state["A"], state["b"], max_iter=20)
        return dict(x=f["x"], info=f["info"])
    if op == "batched":
        f = api.lstsq_batched(state["A"], state["b"], with_rho=case["m"] > case["n"])
        out = dict(x=f["x"], Q=f["Q"], R=f["R"], info=f["info"])
        if case["m"] > case["n"]:
            out["rho"] = f["rho"]
        return out
    x = state["x0"].clone()  # the corrector updates its points in place
    f = api.newton_batched(state["system"], x, case["iters"])
    return dict(x=f["x"], dnorm=f["dnorm"], info=f["info"])


# -------------------------------------------------------------------- work --
# FP64 operations of one complex multiply-add (the inner product's and the
# update's) in each precision, FMA = 2.  Double: 4 FMA.  Double-double: 60 /
# 66 with error-free transformations.  Quad-double: per real part two
# products, each of 6 exact and 7 plain products of limbs, and about 28 exact
# sums of two words.
F_MULADD = {1: 8, 2: 63, 4: 440}


def _qr_flops(m, n, cols, prec):
    return 2 * F_MULADD[prec] * m * (n * (cols - 1) - n * (n - 1) // 2)


def work(case):
    op, prec, n = case["op"], case["prec"], case["n"]
    m = case.get("m", n)
    f, el = F_MULADD[prec], 16 * prec  # bytes of a complex element
    if op == "lstsq":
        return dict(bytes=el * (2 * m * n + n * n + m + 2 * n), flops=_qr_flops(m, n, n + 1, prec) + f * n * n // 2)
    if op == "grad":
        return dict(bytes=el * (2 * m * n + 2 * m + 2 * n),
                    flops=_qr_flops(m, n, n + 1, prec) + f * (3 * n * n // 2 + 4 * m * n))
    if op == "solve":
        return dict(bytes=el * (m * n + n * n // 2 + m + n), flops=f * (2 * m * n + n * n // 2))
    if op == "refine":  # FP64 factorisation, then at least one residual in twice the precision
        return dict(bytes=el * (n * n + 2 * n), flops=_qr_flops(n, n, n + 1, 1) + F_MULADD[4] * n * n)
    if op == "batched":
        one = _qr_flops(m, n, n + 1, prec) + f * n * n // 2
        return dict(bytes=case["batch"] * el * (2 * m * n + n * n + m + n), flops=case["batch"] * one)
    mono = 32 * (2 * 3 * 5 + 2 * 5)  # powers, prefix and suffix products of 32 monomials of 5 variables
    one = n * mono * f + _qr_flops(n, n, n + 1, prec) + f * n * n // 2
    return dict(bytes=el * 2 * n * case["batch"] + n * 32 * (el + 40),
                flops=case["batch"] * case["iters"] * one)


# ------------------------------------------------------------------- exact --
def _complex(t):
    """Leading limbs of planar [prec, 2, ...] as complex128."""
    t = t.detach().cpu().numpy()
    return t[0, 0] + 1j * t[0, 1]


def _planar(z, prec):
    """complex128 [...] as planar [prec, 2, ...], the lower limbs zero."""
    out = np.zeros((prec, 2) + z.shape)
    out[0, 0], out[0, 1] = z.real, z.imag
    return out


def _qr(A):
    Q, R = np.linalg.qr(A)
    d = np.einsum("...ii->...i", R)
    ph = d / np.abs(d)
    return Q * ph[..., None, :], R * ph.conj()[..., :, None]


def _newton64(s, x0, iters):
    """x and the norm of each step's correction, complex128."""
    root = x0[:, 0, 0] + 1j * x0[:, 0, 1]
    c = s["coef"][0, 0] + 1j * s["coef"][0, 1]
    v, d, n = s["vars"], s["exps"], s["nvar"]
    x, norms = root.copy(), []
    for _ in range(iters):
        F = np.zeros(x.shape, complex)
        J = np.zeros((x.shape[0], n, n), complex)
        for i in range(x.shape[0]):
            xv = x[i][v]
            p = xv ** d
            F[i] = (c * p.prod(axis=2)).sum(axis=1)
            for t in range(v.shape[2]):
                rest = c * d[:, :, t] * xv[:, :, t] ** (d[:, :, t] - 1) * np.delete(p, t, axis=2).prod(axis=2)
                np.add.at(J[i], (np.arange(n)[:, None], v[:, :, t]), rest)
        dx = np.linalg.solve(J, -F[..., None])[..., 0]
        x = x + dx
        norms.append(np.linalg.norm(dx, axis=1))
    return x, np.array(norms)


def exact(case, seed):
    op, prec = case["op"], case["prec"]
    if op == "newton":
        s, x0 = _poly(case, seed)
        x, norms = _newton64(s, x0, case["iters"])
        out = np.zeros(x0.shape)
        out[:, 0, 0], out[:, 0, 1] = x.real, x.imag
        return dict(x=out, dnorm=norms, info=None)
    if op == "solve":
        A, b, _ = _system(case, seed, torch.device("cuda:0"))
        Q, R = _qr(_complex(A).T)
        x = np.linalg.solve(R, Q.conj().T @ _complex(b))
        return dict(x=_planar(x, prec), info=None)
    st = prepare(case, seed)
    if op == "batched":
        A = st["A"].cpu().numpy()
        b = st["b"].cpu().numpy()
        A = np.swapaxes(A[:, 0, 0] + 1j * A[:, 0, 1], 1, 2)
        b = b[:, 0, 0] + 1j * b[:, 0, 1]
        Q, R = _qr(A)
        y = np.swapaxes(Q.conj(), 1, 2) @ b[..., None]
        x = np.linalg.solve(R, y)[..., 0]
        move = lambda z: np.ascontiguousarray(np.swapaxes(_planar(z, prec), 0, 2).swapaxes(1, 2))  # noqa: E731
        out = dict(x=move(x), Q=move(np.swapaxes(Q, 1, 2)), R=move(np.swapaxes(R, 1, 2)), info=None)
        if case["m"] > case["n"]:
            out["rho"] = np.zeros((case["batch"], prec))
            out["rho"][:, 0] = np.linalg.norm(b - (A @ x[..., None])[..., 0], axis=1)
        return out
    A, b = _complex(st["A"]).T, _complex(st["b"])
    if op == "refine":
        return dict(x=_planar(np.linalg.solve(A, b), prec), info=None)
    Q, R = _qr(A)
    y = Q.conj().T @ b
    x = np.linalg.solve(R, y)
    if op == "grad":
        g = _complex(st["gx"])
        z = np.linalg.solve(R, np.linalg.solve(R.conj().T, g))
        gb = A @ z
        r = b - A @ x
        gA = np.outer(r, z.conj()) - np.outer(gb, x.conj())
        return dict(x=_planar(x, prec), gA=_planar(gA.T, prec), gb=_planar(gb, prec))
    out = dict(x=_planar(x, prec), Q=_planar(Q.T, prec), R=_planar(R.T, prec), y=_planar(y, prec), info=None,
               info_backsolve=None)
    if case["m"] > case["n"]:
        out["rho"] = np.zeros(prec)
        out["rho"][0] = np.linalg.norm(b - A @ x)
    return out
