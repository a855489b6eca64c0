"""Arbitrary-order plane moments, their gradient, field gradients and the turbulent
budget terms of Sec. 2.5 (library kernels) against the oracle (oracle/moments.py)."""
import numpy as np
import pytest
import torch

import cases
from oracle import moments as om
from oracle.piso import Geometry
from tests.gpu_common import dev, host, max_elem, rel, say, small_cases, tight_opts

pytestmark = pytest.mark.gpu


def _api():
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_2505_16992_amd import api
    return api


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("name,m,order,axis", [("channel", 3, 4, 1), ("channel", 6, 2, 1), ("channel", 4, 3, 2),
                                               ("cavity12", 2, 4, 0), ("tgv16", 2, 3, 1)])
def test_moments_and_gradient_vs_oracle(prec, name, m, order, axis):
    api = _api()
    case = small_cases()[name]
    dims = case.domain.blocks[0]
    ctx = api.Context(case.domain, prec)
    t = ctx.dtype
    rng = np.random.default_rng(50 + m + order)
    xs = [np.asarray(1.5 + rng.standard_normal((m, ctx.N)) * (1 + 0.5 * q), dtype=np.float32 if prec == "f32"
                     else np.float64).astype(np.float64) for q in range(3)]
    state = ctx.moments_state(m, order, axis)
    ost = om.empty_state(dims[axis], m, order)
    for x in xs:
        ctx.moments_accumulate(dev(x, t), state, order, axis)
        ost = om.accumulate(ost, x, dims, axis)
    mean, mom = ctx.moments_finalize(state, m, order, axis)
    mref, oref = om.finalize(ost)
    em, eo = rel(host(mean), mref), max_elem(host(mom), oref)
    mbar = rng.standard_normal(mref.shape)
    obar = rng.standard_normal(oref.shape)
    gx = ctx.moments_backward(dev(xs[1], t), state, dev(mbar, torch.float64), dev(obar, torch.float64), order, axis)
    gref = om.moments_vjp(ost, xs[1], dims, axis, mbar, obar)
    eg = rel(host(gx), gref)
    say("%s %s m=%d order=%d: mean %.2e moments %.2e gradient %.2e" % (name, prec, m, order, em, eo, eg))
    assert em < 1e-13 and eo < 1e-11
    assert eg < (1e-12 if prec == "f64" else 1e-6)


@pytest.mark.parametrize("m,order,grid", [(2, 2, (33, 4, 31)), (2, 3, (32, 4, 32)), (2, 4, (41, 4, 25)),
                                          (3, 2, (64, 4, 32)), (3, 3, (683, 4, 3)), (3, 4, (64, 4, 64)),
                                          (4, 2, (17, 4, 241)), (4, 3, (2, 4, 2)), (6, 2, (7, 4, 16))])
def test_moment_orders_and_plane_sizes(m, order, grid):
    """Every pair of variables and order, planes of one sample short of, at and beyond a
    work-group's threads and its batch of loads.  An FP64 sum of n <= 4100 terms is within
    n eps ~ 1e-12 of exact relative to the sum of magnitudes: 1e-11 as elsewhere."""
    api = _api()
    case = cases.channel(*grid)
    dims = case.domain.blocks[0]
    ctx = api.Context(case.domain, "f64")
    rng = np.random.default_rng(53 + 10 * m + order)
    state = ctx.moments_state(m, order, 1)
    ost = om.empty_state(dims[1], m, order)
    for q in range(2):
        x = 0.7 + (1 + q) * rng.standard_normal((m, ctx.N))
        ctx.moments_accumulate(dev(x, ctx.dtype), state, order, 1)
        ost = om.accumulate(ost, x, dims, 1)
    mean, mom = ctx.moments_finalize(state, m, order, 1)
    mref, oref = om.finalize(ost)
    em, eo = rel(host(mean), mref), max_elem(host(mom), oref)
    say("m=%d order=%d %s: mean %.2e moments %.2e" % (m, order, grid, em, eo))
    assert em < 1e-13 and eo < 1e-11


@pytest.mark.parametrize("name", ["channel", "sheared", "cylinder", "cavity12"])
def test_field_gradient_vs_oracle(name):
    api = _api()
    case = small_cases()[name]
    geo = Geometry(case.domain)
    ctx = api.Context(case.domain, "f64")
    t = ctx.dtype
    rng = np.random.default_rng(51)
    u = rng.standard_normal((geo.d, geo.N))
    ub = rng.standard_normal((geo.d, geo.nb))
    p = rng.standard_normal((1, geo.N))
    gu = ctx.field_gradient(dev(u, t), dev(ub, t) if geo.nb else None)
    gp = ctx.field_gradient(dev(p, t), None)
    eu = rel(host(gu), om.field_gradient(geo, u, ub if geo.nb else None))
    ep = rel(host(gp), om.field_gradient(geo, p, None))
    say("%s: velocity gradient %.2e, pressure gradient %.2e" % (name, eu, ep))
    assert eu < 1e-13 and ep < 1e-13


@pytest.mark.parametrize("prec", ["f64", "mixed"])
def test_budget_terms_vs_oracle(prec):
    """Budget terms from a few PISO steps of a small stretched channel (the library's
    steps, statistics and budget kernel) against the oracle's from the same fields."""
    api = _api()
    case = cases.channel(8, 12, 6)
    geo = Geometry(case.domain)
    dims = case.domain.blocks[0]
    ctx = api.Context(case.domain, prec)
    t = ctx.dtype
    rng = np.random.default_rng(52)
    u = case.u0 + 0.3 * rng.standard_normal(case.u0.shape)
    ud, pd = dev(u, t), dev(case.p0, t)
    nu, S, ub = dev([case.nu], t), dev(case.S, t), dev(case.u_b, t)
    tb = api.TurbulenceBudget(ctx, axis=1, order=4)
    su, sg, sup = om.empty_state(dims[1], 3, 4), [om.empty_state(dims[1], 3, 2) for _ in range(3)], \
        om.empty_state(dims[1], 6, 2)
    o = tight_opts(ctx)
    for _ in range(4):
        ud, pd = ctx.step(ud, pd, nu, S, ub, case.dt, o)
        tb.accumulate(ud, pd, ub)
        uh, ph = host(ud), host(pd)
        g = om.field_gradient(geo, uh, case.u_b)
        gp = om.field_gradient(geo, ph[None], None)[:, 0]
        su = om.accumulate(su, uh, dims, 1)
        for k in range(3):
            sg[k] = om.accumulate(sg[k], g[k], dims, 1)
        sup = om.accumulate(sup, np.concatenate([uh, gp]), dims, 1)
    wall = (np.zeros(3), np.zeros(3))
    out = tb.terms(wall)
    ref = om.budget(geo, dims, 1, om.finalize(su), [om.finalize(s)[1] for s in sg], om.finalize(sup)[1], wall)
    mean, mom = tb.moments()
    assert max_elem(host(mom), om.finalize(su)[1]) < 1e-11
    for k in ("P", "eps", "T", "D", "Pi"):
        e = max_elem(host(out[k]), ref[k])
        say("  %s %s: max elem %.2e (|ref| max %.3e)" % (prec, k, e, np.abs(ref[k]).max()))
        assert e < 1e-10, k
