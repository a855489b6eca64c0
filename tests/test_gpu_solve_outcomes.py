"""What a linear solve returns and leaves behind: the iterate when the call returns, statuses
at and near the limits, the outcome where a recurrence meets an exact zero, and the paths that
an operator or a grid selects."""
import numpy as np
import pytest
import torch

import cases
from oracle.piso import Geometry, step as oracle_step
from tests.gpu_common import dev, host, random_state, rel, rel_p, say, tight_opts
from tests.test_gpu_fdm import _api, _case

pytestmark = pytest.mark.gpu


def _system(ctx, case, state):
    u, p, S, ub, nu = [dev(x, ctx.dtype) for x in state]
    sys = ctx.new_system()
    ctx.assemble(sys, u, p, nu, S, ub, case.dt)
    return sys, u, p, ub


@pytest.mark.parametrize("dims", [(45, 45), (64, 40), (16, 8, 8)])
def test_velocity_is_complete_at_return(dims):
    """Solved on one stream and copied at once on another: the copy is the solution, also of a
    component whose right-hand side is zero (one work-group and launched)."""
    api = _api()
    case = _case(dims, (0,))
    ctx = api.Context(case.domain, "f64")
    sys, u, _, _ = _system(ctx, case, random_state(case, seed=21))
    o = ctx.default_opts().vel
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    last = sys["b"][-1].clone()
    for k in range(40):
        sys["b"][-1] = last * (k % 2)
        x, y = u + k, torch.zeros_like(u)
        torch.cuda.synchronize()
        with torch.cuda.stream(a):
            info = ctx.solve_velocity(sys, x, o)
        with torch.cuda.stream(b):
            y.copy_(x)
        torch.cuda.synchronize()
        assert info["status"] == 0 and torch.equal(x, y), (dims, k)
        assert bool(x[-1].any()) == bool(k % 2)


def _pressure(ctx, sys, u, p, ub, scale, rtol, max_iter):
    s = dict(sys, b_u=sys["b_u"] * scale)
    o = ctx.default_opts().pres
    o.rtol, o.max_iter = rtol, max_iter
    x = torch.zeros_like(p)
    return ctx.solve_pressure(s, u * scale, ub * scale, torch.zeros_like(p), x, o)


@pytest.mark.parametrize("dims,periodic", [((64, 60), (0,)), ((35, 70), ()), ((18, 16), (0, 1)), ((48, 40, 32), (0, 2))])
def test_residual_within_the_tolerance_is_a_solution(dims, periodic):
    """Whichever way a pressure solve ends: stopped by its limit of iterations below the
    tolerance, or (right-hand sides near FP32's smallest numbers, whose residuals stop falling)
    soon after it has met the tolerance instead of running on to the limit."""
    api = _api()
    case = _case(dims, periodic)
    ctx = api.Context(case.domain, "f32")
    sys, u, p, ub = _system(ctx, case, random_state(case, seed=5))
    one_group = dims == (18, 16)   # FP64 residuals, which go on falling at every scale
    for scale, limit in ((1.0, 4),) if one_group else ((1.0, 4), (1e-36, 200)):
        end = _pressure(ctx, sys, u, p, ub, scale, 1e-30, limit)
        got = _pressure(ctx, sys, u, p, ub, scale, 2 * end["rel_residual"], limit)
        say(dims, scale, end, got)
        assert end["status"] == 1 and end["iters"] == limit
        assert got["status"] == 0 and got["rel_residual"] <= 2 * end["rel_residual"]
        assert got["iters"] <= min(limit, 40)


@pytest.mark.parametrize("dims,periodic", [((18, 16), (0, 1)), ((49, 17), (0,)), ((64, 32), (0, 1)), ((45, 44), ())])
def test_one_group_solve_of_any_scale(dims, periodic):
    """A linear solve takes the iterations of the same system at scale one down to right-hand
    sides of FP32's smallest normal numbers (the residual is FP64 in these kernels)."""
    api = _api()
    case = _case(dims, periodic)
    ctx = api.Context(case.domain, "f32")
    sys, u, p, ub = _system(ctx, case, random_state(case, seed=6))
    one = _pressure(ctx, sys, u, p, ub, 1.0, 1e-7, 100)
    for scale in (1e-20, 1e-33, 1e-36, 1e20):
        got = _pressure(ctx, sys, u, p, ub, scale, 1e-7, 100)
        say(dims, scale, one, got)
        assert got["status"] == 0 and abs(got["iters"] - one["iters"]) <= 1


@pytest.mark.parametrize("dims,periodic", [((18, 16), (0, 1)), ((128, 100), ()), ((48, 40, 32), (0, 2)), ((24, 24, 24), (0, 2))])
def test_no_iterations(dims, periodic):
    """A step whose solves may not iterate (piso_step takes max_iter = 0) reports the residual of
    their starts, the same whatever the preconditioner."""
    api = _api()
    case = _case(dims, periodic)
    ctx = api.Context(case.domain, "f64")
    u, p, S, ub, nu = [dev(x, ctx.dtype) for x in random_state(case, seed=7)]
    rels = []
    for precond in (0, 1):
        o = ctx.default_opts()
        o.pres.precond = precond
        ctx.step(u, p, nu, S, ub, case.dt, o)   # leaves its partial sums behind
        o.pres.max_iter = 0
        _, _, info = ctx.step(u, p, nu, S, ub, case.dt, o, info=True)
        assert all(q["status"] == 1 and q["iters"] == 0 for q in info["pres"])
        rels.append([q["rel_residual"] for q in info["pres"]])
    say(dims, rels)
    assert np.allclose(rels[0], rels[1], rtol=1e-8)


def test_easy_velocity_solve_after_a_hard_one():
    """What a solve costs does not hang on the one before: an easy system after one that
    converges in several times its iterations, and after one that fails, takes the time it takes
    by itself (launching the other's iterations made it 3.5 to 5 times that)."""
    api = _api()
    case = _case((96, 96), (0,))
    ctx = api.Context(case.domain, "f64")
    u, p, S, ub, nu = random_state(case, seed=8)
    t = ctx.dtype
    o = ctx.default_opts().vel
    o.precond = 0   # Jacobi alone, without the ILU(0) restart
    x0 = dev(u, t)

    def system(dt, nu):
        sys = ctx.new_system()
        ctx.assemble(sys, x0, dev(p, t), dev(nu, t), dev(S, t), dev(ub, t), dt)
        return sys

    def solve(sys, max_iter=500):
        x = x0.clone()
        o.max_iter = max_iter
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        info = ctx.solve_velocity(sys, x, o)
        b.record()
        b.synchronize()
        return a.elapsed_time(b), info

    easy, hard = system(0.01, nu), system(1e3, 0 * nu + 100.0)
    alone = min(solve(easy)[0] for _ in range(8))
    for limit, status in ((500, 0), (150, 1)):
        after = []
        for _ in range(6):
            _, info = solve(hard, limit)
            assert info["status"] == status
            after.append(solve(easy)[0])
        say("alone %.3f ms, after one of %d iterations (status %d): %.3f" % (alone, info["iters"], status, min(after)))
        assert min(after) < 1.7 * alone


@pytest.mark.parametrize("dims,periodic", [((20, 20), ()), ((9, 7, 5), (0, 2))])
def test_launched_forms_on_request(dims, periodic, monkeypatch):
    """Kernel timing and PISO_CG_GROUPS select the launched velocity solve on small grids: FP32
    vectors there, FP64 ones in one work-group, so the results differ in their last bits."""
    api = _api()
    case = _case(dims, periodic)
    state = random_state(case, seed=9)
    ctx = api.Context(case.domain, "f32")
    monkeypatch.setenv("PISO_CG_GROUPS", "4")
    groups = api.Context(case.domain, "f32")
    sys, u, _, _ = _system(ctx, case, state)
    o = ctx.default_opts().vel
    out = []
    for c, timed in ((ctx, False), (ctx, True), (groups, False)):
        c.set_timing(timed)
        x = u.clone()
        assert c.solve_velocity(sys, x, o)["status"] == 0
        c.set_timing(False)
        out.append(x)
    small, timed, grouped = out
    assert not torch.equal(small, timed) and torch.equal(timed, grouped)
    assert rel(host(small), host(timed)) < 1e-5


@pytest.mark.parametrize("precond", [0, 2])
@pytest.mark.parametrize("prec", ["f64", "f32", "mixed"])
@pytest.mark.parametrize("dims,periodic", [((20, 20), (0, 1)), ((64, 64), (0, 1)), ((12, 8, 32), (0, 1, 2))])
def test_residual_without_a_part_along_its_start(dims, periodic, prec, precond):
    """Couplings one way along x and a right-hand side in one cell: the first iteration leaves a
    residual orthogonal to the start's to the last bit (rho = 0).  The solve goes on from it, in
    one work-group and launched, with C and C^T, Jacobi and ILU(0): x = 0.25^k along the row."""
    api = _api()
    ctx = api.Context(_case(dims, periodic).domain, prec)
    sys = ctx.new_system()
    sys["A"].fill_(1.0)
    sys["C"][1, 0].fill_(-0.25)   # the cell above along x depends on this one
    sys["b"][:, 0] = 1.0
    o = ctx.default_opts().vel
    o.precond, o.rtol = precond, 1e-6 if prec == "f32" else 1e-10
    row = 0.25 ** np.arange(dims[0]) / (1.0 - 0.25 ** dims[0])
    tol = 1e-5 if prec == "f32" else 1e-9
    for transposed in (False, True):
        for timed in (False, True):
            ctx.set_timing(timed)
            if transposed:
                g = ctx.new_system_grad()
                zero = torch.zeros_like(sys["b"])
                info = ctx.solve_velocity_backward(sys, zero, sys["b"], g, o)
                x, want = g["db"], np.roll(row[::-1], 1)
            else:
                x = torch.zeros_like(sys["b"])
                info = ctx.solve_velocity(sys, x, o)
                want = row
            ctx.set_timing(False)
            got = host(x)
            say(dims, prec, precond, transposed, timed, info["status"], info["iters"], rel(got[:, :dims[0]], want[None]))
            assert info["status"] == 0
            assert np.abs(got[:, :dims[0]] - want).max() < tol and np.abs(got[:, dims[0]:]).max() == 0


@pytest.mark.parametrize("prec", ["f64", "f32", "mixed"])
@pytest.mark.parametrize("dims,periodic", [((64, 60), ()), ((24, 20), ()), ((32, 30, 28), (0, 2))])
def test_rejected_operators(dims, periodic, prec, monkeypatch):
    """A viscosity that varies over two decades at nu dt / h^2 >> 1: turned down by the fast
    diagonalisation, the solve is the V-cycle's bit for bit, launched and on grids that otherwise
    solve in one work-group.  From the second such operator on, nothing but its judgement is
    launched ahead of the V-cycle; the next operator near a product is accepted."""
    api = _api()
    case = _case(dims, periodic)
    u, p, S, ub, nu = random_state(case, seed=73)
    wild = 10.0 ** np.random.default_rng(74).uniform(-2, 0, nu.shape)
    out = []
    for env in (None, "auto"):
        if env:
            monkeypatch.setenv("PISO_MG_LINE", env)
        ctx = api.Context(case.domain, prec)
        monkeypatch.delenv("PISO_MG_LINE", raising=False)
        o = ctx.default_opts().pres
        o.max_iter = 100
        res = []
        for k, (dt, v) in enumerate(((5.0, wild), (5.0, 1.5 * wild), (4.0, wild), (0.01, nu), (5.0, wild))):
            case.dt = dt
            sys, ud, pd, ubd = _system(ctx, case, (u, p, S, ub, v))
            ctx.set_timing(k == 2)
            x = pd.clone()
            info = ctx.solve_pressure(sys, ud, ubd, pd, x, o)
            count = {n: t[1] for n, t in ctx.get_timing().items()}
            ctx.set_timing(False)
            assert ctx.pressure_preconditioner == ("fast diagonalisation" if k == 3 and not env else "multigrid")
            res.append((info["iters"], x, count))
        out.append(res)
    say(dims, prec, [[r[0] for r in res] for res in out], [res[2][2] for res in out])
    for k in (0, 1, 2, 4):
        assert out[0][k][0] == out[1][k][0] and torch.equal(out[0][k][1], out[1][k][1])
    assert out[0][2][2] == out[1][2][2]
    assert out[0][3][0] < out[1][3][0]


def test_preconditioner_of_the_last_solve(monkeypatch):
    """What the context reports of its last pressure solve, by grid, option and request."""
    api = _api()
    fdm, mg = "fast diagonalisation", "multigrid"
    for dims, periodic, env, precond, want in [((24, 20), (), None, 1, fdm), ((24, 20), (), "auto", 1, mg),
                                               ((24, 20), (), None, 0, "jacobi"), ((70, 64), (0,), None, 1, fdm),
                                               ((513, 8), (0,), None, 1, mg), ((512, 8), (0,), None, 1, fdm),
                                               ((32, 32, 15), (0, 2), None, 1, mg), ((32, 32, 16), (0, 2), None, 1, fdm)]:
        case = _case(dims, periodic)
        if env:
            monkeypatch.setenv("PISO_MG_LINE", env)
        ctx = api.Context(case.domain, "f32")
        monkeypatch.delenv("PISO_MG_LINE", raising=False)
        assert ctx.pressure_preconditioner is None
        u, p, S, ub, nu = [dev(x, ctx.dtype) for x in random_state(case, seed=10)]
        o = ctx.default_opts()
        o.pres.precond = precond
        ctx.step(u, p, nu, S, ub, case.dt, o)
        assert ctx.pressure_preconditioner == want, (dims, env, precond)


@pytest.mark.parametrize("name", ["tgv", "channel", "box"])
def test_a_step_under_capture_is_refused(name):
    """A step reads its solves' states back, so it cannot be captured: the call says so (and does
    not wait for kernels that will not run), and the context goes on outside."""
    api = _api()
    case = {"tgv": lambda: cases.taylor_green(16), "channel": lambda: cases.channel(24, 24, 32),
            "box": lambda: _case((64, 60), ())}[name]()
    ctx = api.Context(case.domain, "f64")
    u, p, S, ub, nu = [dev(x, ctx.dtype) for x in random_state(case, seed=11)]
    u1, p1 = ctx.step(u, p, nu, S, ub, case.dt)
    torch.cuda.synchronize()
    s, g = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    with torch.cuda.stream(s):
        g.capture_begin()
        with pytest.raises(RuntimeError):
            ctx.step(u, p, nu, S, ub, case.dt)
        with pytest.raises(RuntimeError):
            g.capture_end()
    u2, p2 = ctx.step(u, p, nu, S, ub, case.dt)
    assert torch.equal(u1, u2) and torch.equal(p1, p2)
