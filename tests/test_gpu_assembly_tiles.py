"""Assembly at the edges of its tiles (32 x 8 or 64 x 4 columns) and marches
(up to 16 planes): grids a column short of, on and past them, one plane, one
column of each colour, more planes than a march, for every fluid model (black
oil with a third of the cells undersaturated).  Against the oracle to 1e-13
of the largest entry (a few dozen FP64 operations per entry on both sides),
and the residual written in place of the state (which goes through
colour-split copies) bit for bit against the one written beside it."""
import numpy as np
import pytest

from oracle import model
from paper_1606_00548_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SHAPES = [(2, 1, 1), (30, 7, 3), (32, 8, 2), (34, 9, 5), (64, 4, 3), (66, 5, 1), (128, 4, 40), (2, 3, 70)]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("name", ["single", "oil-water", "black-oil"])
def test_jacobian_and_residual(name, shape):
    from paper_1606_00548_amd import cprmi
    nx, ny, nz = shape
    wells = [synth.well(0, 0, nz, "inj", 300.0)]
    if name == "single":
        case = synth.single_phase_uniform(nx, ny, nz)
    else:
        case = (synth.black_oil_layered if name == "black-oil" else synth.oil_water_lognormal)(nx, ny, nz)
        wells += [synth.well(nx - 1, ny - 1, nz, "prod", 150.0)]
    case["wells"] = wells
    x = synth.random_state_perturbation(case, 31)
    if name == "black-oil":
        x = synth.undersaturated_cells(case, x, 32, frac=0.33)
    R, J = model.assemble(case["grid"], case["fluid"], case["perm"], case["poro"], wells, case["x_old"], x, case["dt"])
    s = cprmi.Solver.from_case(case)
    xo, xg = (torch.as_tensor(np.ascontiguousarray(a)).cuda() for a in (case["x_old"], x))
    rhs = s.assemble(xo, xg, case["dt"])
    Jg = s.export_jacobian().cpu().numpy()
    assert np.abs(Jg - J).max() <= 1e-13 * np.abs(J).max()
    assert np.abs(rhs.cpu().numpy() + R).max() <= 1e-13 * max(np.abs(R).max(), np.abs(J).max())
    inplace = xg.clone()
    s.assemble(xo, inplace, case["dt"], inplace)
    assert torch.equal(inplace, rhs)
    assert np.array_equal(s.export_jacobian().cpu().numpy(), Jg)
