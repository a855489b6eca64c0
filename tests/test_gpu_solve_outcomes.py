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
