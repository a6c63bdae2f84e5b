"""A triangular solve that times out inside a longer call must show in that
call's info, whatever comes after it: in the adjoint (whose second solve
shares the status word), in the Newton step of one qd point (whose x must
then stay as it is) and in the refinement (first solution and correction).

The time-out is forced by a tiny limit on one launch's own bounded waits, so
every kernel ends normally; a call without it must then succeed again.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1210_0800_amd import api, inputs  # noqa: E402

pytestmark = pytest.mark.gpu
TIMEOUT = -9


def T(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def limited(launch, run):
    """run() with the launch-th waiting launch timed out, then without."""
    torch.cuda.synchronize()
    api.set_wait_limit(launch)
    try:
        out = run()
        torch.cuda.synchronize()
    finally:
        api.set_wait_limit(0)
    return out, run()


@pytest.mark.parametrize("launch", [1, 2])
def test_adjoint(launch):
    p = inputs.random_problem(2, 320, 300, seed=1, config=94)
    A, b = T(p["A"]), T(p["b"])
    f = api.lstsq(A, b)
    gx = f["x"].clone()
    cut, whole = limited(launch, lambda: api.ls_adjoint(A, b, f["Q"], f["R"], f["x"], gx))
    torch.cuda.synchronize()
    assert int(cut[2].item()) == TIMEOUT
    assert int(whole[2].item()) == 0 and bool(torch.isfinite(whole[0]).all())


def test_newton_step_of_one_qd_point():
    s = inputs.polysys(neq=40, nvar=40, nmon=16, nvpm=3, maxdeg=3, L=4, system=1)
    ds = api.PolySystem(s["vars"], s["exps"], s["coef"], 40, torch.device("cuda:0"))
    X = T(np.stack([inputs.near_root(s, 1e-3, L=4, system=1)]))

    def step():
        return api.newton_batched(ds, X.clone(), 1)

    cut, whole = limited(2, step)  # 1: the factorisation, 2: the back substitution
    torch.cuda.synchronize()
    assert int(cut["info"].item()) == TIMEOUT
    assert torch.equal(cut["x"], X) and bool(torch.isnan(cut["dnorm"]).all())
    assert int(whole["info"].item()) == 0 and bool(torch.isfinite(whole["x"]).all())
    # with two steps, the time-out of the first one is not the last status
    again, _ = limited(2, lambda: api.newton_batched(ds, X.clone(), 2))
    torch.cuda.synchronize()
    assert int(again["info"].item()) == 0 and torch.equal(again["x"], whole["x"])


@pytest.mark.parametrize("prec", [2, 4])
@pytest.mark.parametrize("launch,max_iter", [(6, 0), (6, 3), (8, 3)])
def test_refinement(prec, launch, max_iter):
    # 1..5: the panels, 6: the first solution, 7: the projections of the
    # residual, 8: the first correction's solve
    p = inputs.random_problem(prec, 300, 300, seed=2, config=94)
    A, b = T(p["A"]), T(p["b"])
    cut, whole = limited(launch, lambda: api.refine_lstsq(A, b, max_iter=max_iter))
    torch.cuda.synchronize()
    assert int(cut["info"].item()) == TIMEOUT
    assert int(whole["info"].item()) != TIMEOUT and bool(torch.isfinite(whole["x"]).all())
