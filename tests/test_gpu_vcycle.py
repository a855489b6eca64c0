"""The multigrid V-cycle on grids where the fast diagonalisation otherwise takes its place: the
checks of tests/test_gpu_mg.py and tests/test_gpu_line.py with contexts that keep the V-cycle
(PISO_MG_LINE=auto: its own choice of the smoother), and a look at what ran in each."""
import pytest

from tests import test_gpu_fdm as fdm
from tests import test_gpu_line as line
from tests import test_gpu_mg as mg
from tests.gpu_common import small_cases

pytestmark = pytest.mark.gpu


@pytest.fixture
def vcycle(monkeypatch):
    """Contexts keep the V-cycle; afterwards each one's last pressure solve is asked for."""
    api = mg._api()
    made = []

    class Context(api.Context):
        def __init__(self, *a, **k):
            super().__init__(*a, **k)
            made.append(self)

    monkeypatch.setattr(api, "Context", Context)
    monkeypatch.setenv("PISO_MG_LINE", "auto")
    yield monkeypatch
    ran = [c.pressure_preconditioner for c in made]
    assert ran and "multigrid" in ran and set(ran) <= {"multigrid", "jacobi", None}, ran


@pytest.mark.parametrize("name", list(small_cases()))
def test_step_f64(name, vcycle):
    mg.test_step_both_preconditioners_f64(name, mg.MG)


@pytest.mark.parametrize("prec", ["f32", "mixed"])
def test_step_single_precision(prec, vcycle):
    mg.test_step_mg_single_precision(prec)


def test_iteration_counts(vcycle):
    mg.test_mg_iteration_counts()


def test_adjoint(vcycle):
    mg.test_mg_adjoint_matches_jacobi_adjoint()


@pytest.mark.parametrize("prec", ["f64", "mixed"])
def test_graph_replay(prec, vcycle):
    mg.test_graph_replay_matches_eager(prec, vcycle)


@pytest.mark.parametrize("name", ["channel_q", "channel", "tgv16", "cavity12"])
def test_position_indexed_levels(name, vcycle):
    mg.test_position_indexed_levels_match_tables(name, vcycle)


@pytest.mark.parametrize("name", list(line.line_cases()))
def test_line_step_f64(name, vcycle):
    line.test_line_step_f64(name, vcycle)


@pytest.mark.parametrize("prec", ["f32", "mixed"])
def test_line_step_single_precision(prec, vcycle):
    line.test_line_step_single_precision(prec)


@pytest.mark.parametrize("prec", ["f64", "mixed", "f32"])
@pytest.mark.parametrize("dims", [(24, 40, 36), (19, 37, 27)])
def test_fast_diagonalisation_with_walls_along_x_alone(dims, prec, monkeypatch):
    """3D boxes periodic in y and z: x and y change places in the transforms' box (rows of quads
    and not)."""
    fdm.test_step_and_adjoint(dims, (1, 2), prec, monkeypatch)
