"""Fast-diagonalisation preconditioner of the pressure PCG: the kernels at the edges of
their tiles against the oracle, the multigrid where an operator or a grid is turned down.

PISO_MG_LINE=0 keeps the multigrid with point smoothing, the other path of the same solve."""
import numpy as np
import pytest
import torch

import cases
from oracle.adjoint import step_vjp
from oracle.piso import Geometry, step as oracle_step
from tests.gpu_common import dev, host, random_state, rel, rel_p, say, tight_opts

pytestmark = pytest.mark.gpu


def _api():
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_2505_16992_amd import api
    return api


def _case(dims, periodic, beta=1.5):
    """Tensor-product block: the listed axes wrap (uniform), the others are stretched walls."""
    d = len(dims)
    v = [np.linspace(0.0, 2.0, n + 1) if a in periodic else cases.tanh_vertices(n, beta, 0.0, 1.0)
         for a, n in enumerate(dims)]
    T, J, _ = cases.tensor_metrics(v)
    sides = cases.periodic_sides(0, d, periodic)
    sides += [cases.Side(0, 2 * a + s, cases.DIRICHLET) for a in range(d) if a not in periodic for s in (0, 1)]
    dom = cases.Domain(d, [tuple(dims) + ((1,) if d == 2 else ())], sides, T, J)
    n = dom.n_cells
    return cases.Case("box", dom, np.zeros((d, n)), np.zeros(n), np.zeros((d, n)), 0.01, 0.01,
                      cases.boundary_values(dom, lambda si: np.zeros(d)), 1)


# dims, periodic axes.  Remainders of the 16-wide tiles in every axis, whole tiles, rows that
# are no quads, extents of one to three, lines along y and along z and no line axis, axes long
# enough for output rows split over work-groups (2D)
SHAPES = [((32, 32, 17), (0, 2)), ((33, 37, 15), (0,)), ((16, 48, 24), ()), ((18, 30, 31), (0, 1, 2)),
          ((49, 18, 20), (0, 1)), ((200, 91, 1), (0, 2)),
          ((18, 16), (0, 1)), ((40, 23), ()), ((129, 70), (0,)), ((64, 97), ()), ((3, 200), (0,)), ((90, 81), (0, 1)),
          ((70, 30), (1,))]


def _blocks():
    """Layouts that are a box cut into blocks: the cylinder's O-H grid (theta becomes the
    box's first axis, gathered through the map), and 3D channels cut in two along x (rows of
    two blocks) and along y."""
    out = {"cylinder": cases.cylinder_oh(32, 9, 7), "cylinder_q": cases.cylinder_oh(64, 24, 12)}
    for axis in (0, 1):
        whole = _case((28, 30, 23), (0, 2))
        dims = [28, 30, 23]
        cut = 11
        parts, blocks = [], []
        idx = np.arange(whole.domain.n_cells).reshape(23, 30, 28)
        for sl in (slice(0, cut), slice(cut, dims[axis])):
            pick = [slice(None)] * 3
            pick[2 - axis] = sl
            c = idx[tuple(pick)]
            parts.append(c.ravel())
            blocks.append(tuple(c.shape[::-1]))
        order = np.concatenate(parts)
        sides = []
        for b in range(2):
            for a in range(3):
                for s in (0, 1):
                    if a == axis and (axis == 0 or s == 1 - b):
                        sides.append(cases.Side(b, 2 * a + s, cases.CONNECT, other_block=1 - b))
                    elif a == 1:
                        sides.append(cases.Side(b, 2 * a + s, cases.DIRICHLET))
                    else:
                        sides.append(cases.Side(b, 2 * a + s, cases.CONNECT, other_block=b))
        dom = cases.Domain(3, blocks, sides, whole.domain.T[:, :, order], whole.domain.J[order])
        n = dom.n_cells
        out["cut%d" % axis] = cases.Case("cut", dom, np.zeros((3, n)), np.zeros(n), np.zeros((3, n)), 0.01, 0.01,
                                         cases.boundary_values(dom, lambda si: np.zeros(3)), 1)
    return out


def _run(ctx, case, state, opts):
    u, p, S, ub, nu = state
    t = ctx.dtype
    a = [dev(x, t) for x in (u, p, nu, S, ub)]
    tape = ctx.new_tape()
    u1, p1, info = ctx.step(*a, case.dt, opts, tape=tape, info=True)
    w = torch.sin(a[0])
    g = ctx.step_backward(tape, a[0], a[1], a[2], a[4], case.dt, w, None, opts)
    return host(u1), host(p1), [q["iters"] for q in info["pres"]], host(w), host(g["S"]), info


@pytest.mark.parametrize("prec", ["f64", "mixed", "f32"])
@pytest.mark.parametrize("dims,periodic", SHAPES + [(n, None) for n in ("cylinder", "cylinder_q", "cut0", "cut1")])
def test_step_and_adjoint(dims, periodic, prec, monkeypatch):
    """Against the oracle (F64 and MIXED at 1e-12, F32 at its defaults), with
    fewer iterations than the V-cycle needs on the same system."""
    api = _api()
    say(dims, periodic, prec)
    case = _blocks()[dims] if periodic is None else _case(dims, periodic)
    state = random_state(case, seed=71)
    geo = Geometry(case.domain)
    u, p, S, ub, nu = [x.astype(np.float32).astype(np.float64) for x in state] if prec == "f32" else state
    how = dict(mode="iterative", rtol=1e-13) if case.domain.dim == 3 else {}   # direct solves in 2D
    ref = oracle_step(geo, u, p, nu, S, case.dt, ub, **how)
    iters = []
    for env in (None, "0"):
        if env:
            monkeypatch.setenv("PISO_MG_LINE", env)
        ctx = api.Context(case.domain, prec)
        monkeypatch.delenv("PISO_MG_LINE", raising=False)
        o = ctx.default_opts() if prec == "f32" else tight_opts(ctx)
        u1, p1, it, w, gS, _ = _run(ctx, case, (u, p, S, ub, nu), o)
        gr = step_vjp(geo, ref, w, np.zeros(geo.N), **how)["S"]
        iters.append(sum(it))
        eu, ep, eg = rel(u1, ref.u2), rel_p(p1, ref.p2), rel(gS, gr)
        say("  env %s: iters %s, u %.2e p %.2e dS %.2e" % (env, it, eu, ep, eg))
        # bounds of the other parity tests of each form
        assert eu < (1e-5 if prec == "f32" else 1e-9) and ep < (1e-5 if prec == "f32" else 1e-8)
        assert eg < (1e-5 if prec == "f32" else 1e-8)
    assert iters[0] < iters[1]


@pytest.mark.parametrize("periodic", [(0, 2), (0, 1, 2)])
@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_long_axis(prec, periodic, monkeypatch):
    """Many columns along an axis of 400 cells, as lines and (periodic) as the fused product:
    two LDS tiles of 64 kB (F32) or 128 kB (F64), against the multigrid."""
    api = _api()
    case = _case((16, 400, 100), periodic)
    state = random_state(case, seed=72)
    out = []
    for env in (None, "0"):
        if env:
            monkeypatch.setenv("PISO_MG_LINE", env)
        ctx = api.Context(case.domain, prec)
        monkeypatch.delenv("PISO_MG_LINE", raising=False)
        o = ctx.default_opts() if prec == "f32" else tight_opts(ctx)
        out.append(_run(ctx, case, state, o))
    say("iters", out[0][2], out[1][2], "u %.2e p %.2e" % (rel(out[0][0], out[1][0]), rel_p(out[0][1], out[1][1])))
    assert sum(out[0][2]) < sum(out[1][2])
    assert rel(out[0][0], out[1][0]) < (1e-5 if prec == "f32" else 1e-9)
    assert rel(out[0][4], out[1][4]) < (1e-5 if prec == "f32" else 1e-9)


@pytest.mark.parametrize("prec", ["f64", "mixed"])
def test_rejected_operator_runs_multigrid(prec, monkeypatch):
    """A viscosity that varies over four decades at nu dt / h^2 >> 1 is no product over the
    axes: the operator is turned down on the device and the solve is the multigrid one, bit
    for bit, in both correctors and in the adjoint; the next operator is judged anew."""
    api = _api()
    case = _case((24, 20), ())
    u, p, S, ub, nu = random_state(case, seed=73)
    rng = np.random.default_rng(74)
    case.dt = 5.0
    wild = 10.0 ** rng.uniform(-4, 0, nu.shape)
    res = []
    for env in (None, "0"):
        if env:
            monkeypatch.setenv("PISO_MG_LINE", env)
        ctx = api.Context(case.domain, prec)
        monkeypatch.delenv("PISO_MG_LINE", raising=False)
        o = tight_opts(ctx)
        first = _run(ctx, case, (u, p, S, ub, wild), o)
        case.dt = 0.01
        second = _run(ctx, case, (u, p, S, ub, nu), o)
        case.dt = 5.0
        res.append((first, second))
    (f0, s0), (f1, s1) = res
    say("rejected: iters", f0[2], f1[2], "accepted:", s0[2], s1[2])
    assert f0[2] == f1[2] and np.array_equal(f0[0], f1[0]) and np.array_equal(f0[1], f1[1])
    assert np.array_equal(f0[4], f1[4])
    assert sum(s0[2]) < sum(s1[2]) and rel(s0[0], s1[0]) < 1e-9


def test_replay_matches_eager(monkeypatch):
    """Replays of the recorded iteration pair, with eager work between them, against eager
    launches: bit for bit."""
    api = _api()
    case = _case((32, 20, 28), (0, 2))
    u, p, S, ub, nu = random_state(case, seed=75)
    seqs = []
    for env in ("1", None):
        if env:
            monkeypatch.setenv("PISO_NO_GRAPH", env)
        ctx = api.Context(case.domain, "f32")
        monkeypatch.delenv("PISO_NO_GRAPH", raising=False)
        t = ctx.dtype
        uu, pp, seq = dev(u, t), dev(p, t), []
        for _ in range(4):
            uu, pp = ctx.step(uu, pp, dev(nu, t), dev(S, t), dev(ub, t), case.dt)
            torch.cuda.synchronize()
            seq.append((uu.clone(), pp.clone()))
        seqs.append(seq)
    for (ue, pe), (ug, pg) in zip(*seqs):
        assert torch.equal(ue, ug) and torch.equal(pe, pg)
