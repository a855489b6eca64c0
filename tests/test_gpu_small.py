"""Solves of small grids in one work-group, at the edges of their cells per thread, tiles and
limits, against the oracle and against the same solves by launches over the chip (which run
while the kernels are being timed)."""
import numpy as np
import pytest
import torch

from oracle.adjoint import step_vjp
from oracle.piso import Geometry, step as oracle_step
from tests.gpu_common import dev, host, random_state, rel, rel_p, say, tight_opts
from tests.test_gpu_fdm import _api, _blocks, _case

pytestmark = pytest.mark.gpu

# dims, periodic axes: one wave; one cell short of, at and beyond a work-group's threads; the
# largest grid in each form; 8 tiles of a dense axis and (launched) 9; bases too large for the
# LDS beside the fields; long and short lines; 3D (velocity only) at its limits
SHAPES = [((8, 8), ()), ((17, 15), (0,)), ((16, 16), (0, 1)), ((19, 27), ()), ((64, 32), (0,)), ((64, 32), (0, 1)),
          ((45, 45), (0, 1)), ((49, 17), (0,)), ((128, 16), (0,)), ((129, 15), (0,)), ((12, 170), (0,)),
          ((96, 21), (0, 1)), ((683, 3), (1,)), ((64, 33), (0,)),
          ((9, 7, 5), (0, 2)), ((16, 8, 8), (0, 2)), ((16, 16, 8), (0, 1, 2))]


def _step(ctx, case, state, opts):
    u, p, S, ub, nu = [dev(x, ctx.dtype) for x in state]
    tape = ctx.new_tape()
    u1, p1, info = ctx.step(u, p, nu, S, ub, case.dt, opts, tape=tape, info=True)
    g = ctx.step_backward(tape, u, p, nu, ub, case.dt, torch.sin(u), torch.cos(p), opts)
    return host(u1), host(p1), host(g["S"]), host(torch.sin(u)), host(torch.cos(p)), info


@pytest.mark.parametrize("prec", ["f64", "mixed", "f32"])
@pytest.mark.parametrize("dims,periodic", SHAPES + [("cylinder", None)])
def test_step_and_adjoint(dims, periodic, prec):
    """Bounds as in the other parity tests of each form."""
    api = _api()
    say(dims, periodic, prec)
    if dims == (683, 3) and prec == "f32":
        # beyond the limits, so launched on both sides (bit for bit equal); the FP32 multigrid
        # solve of this stretched axis, 450 iterations, ends 3.4e-5 from the oracle
        pytest.skip("conditioning of the launched FP32 solve, not of the kernels under test")
    case = _blocks()[dims] if periodic is None else _case(dims, periodic)
    state = [x.astype(np.float32).astype(np.float64) for x in random_state(case, seed=91)]
    u, p, S, ub, nu = state
    geo = Geometry(case.domain)
    ref = oracle_step(geo, u, p, nu, S, case.dt, ub)
    ctx = api.Context(case.domain, prec)
    o = ctx.default_opts() if prec == "f32" else tight_opts(ctx)
    u1, p1, gS, wu, wp, info = _step(ctx, case, state, o)
    gr = step_vjp(geo, ref, wu, wp)["S"]
    ctx.set_timing(True)
    lu, lp, lg, _, _, linfo = _step(ctx, case, state, o)
    ctx.set_timing(False)
    it, lit = [q["iters"] for q in info["pres"]], [q["iters"] for q in linfo["pres"]]
    say("  iters %s launched %s, oracle u %.1e p %.1e dS %.1e, launched u %.1e p %.1e dS %.1e" %
        (it, lit, rel(u1, ref.u2), rel_p(p1, ref.p2), rel(gS, gr), rel(u1, lu), rel_p(p1, lp), rel(gS, lg)))
    tol_u, tol = (1e-5, 1e-5) if prec == "f32" else (1e-9, 1e-8)
    assert rel(u1, ref.u2) < tol_u and rel_p(p1, ref.p2) < tol and rel(gS, gr) < tol
    assert rel(u1, lu) < tol_u and rel_p(p1, lp) < tol and rel(gS, lg) < tol
    assert max(abs(a - b) for a, b in zip(it, lit)) <= 2   # rounding moves the last iteration


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("dims,periodic", [((18, 16), (0, 1)), ((49, 17), (0,))])
def test_limits_and_outcomes(dims, periodic, prec):
    """A limit of iterations, a zero right-hand side and a state that is not finite end as they
    do when launched."""
    api = _api()
    case = _case(dims, periodic)
    ctx = api.Context(case.domain, prec)
    u, p, S, ub, nu = random_state(case, seed=92)
    o = tight_opts(ctx)
    o.pres.max_iter, o.vel.max_iter, o.vel.precond = 2, 1, 0   # Jacobi alone, without the ILU(0) restart
    for timed in (False, True):
        ctx.set_timing(timed)
        t = ctx.dtype
        _, _, info = ctx.step(dev(u, t), dev(p, t), dev(nu, t), dev(S, t), dev(ub, t), case.dt, o, info=True)
        say(timed, info["vel"], info["pres"])
        assert info["vel"]["status"] == 1 and info["vel"]["iters"] == 1
        assert [q["status"] for q in info["pres"]] == [1, 1] and [q["iters"] for q in info["pres"]] == [2, 2]
        z = tight_opts(ctx)
        u0, p0, info = ctx.step(dev(0 * u, t), dev(0 * p, t), dev(nu, t), dev(0 * S, t), dev(0 * ub, t), case.dt, z,
                                info=True)
        assert not u0.any() and not p0.any() and info["pres"][0]["iters"] == 0 and info["vel"]["iters"] == 0
        bad = u.copy()
        bad[0, 5] = np.nan
        with pytest.raises(RuntimeError):
            ctx.step(dev(bad, t), dev(p, t), dev(nu, t), dev(S, t), dev(ub, t), case.dt, z)
        u1, _, info = ctx.step(dev(u, t), dev(p, t), dev(nu, t), dev(S, t), dev(ub, t), case.dt, ctx.default_opts(),
                               info=True)   # and the context goes on
        assert torch.isfinite(u1).all() and info["vel"]["status"] == 0
    ctx.set_timing(False)
