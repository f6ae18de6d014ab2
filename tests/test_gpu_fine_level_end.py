"""The end of the fine pressure level inside the first kernel of stage 2 (its
last red half-sweep) and the restriction by runs of 64 coarse cells, where
they can go wrong: a coarse level of fewer than 64 cells, of 64, of 65, odd
fine rows and planes, an odd coarse width, one plane.  Every decoupling and
composition, and the cycles V(1,1) and V(2,2), against the oracle: one
application to 1e-9 in FP64 and 1e-5 with the FP32 preconditioner (tolerances
as in the other parity tests)."""
import numpy as np
import pytest

from oracle import cpr, model
from paper_1606_00548_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SHAPES = [(6, 4, 3), (8, 8, 8), (10, 26, 1), (14, 7, 13), (34, 6, 5)]


@pytest.mark.parametrize("decoupling,composition", [("qimpes", "two-stage"), ("abf", "two-stage"), ("qimpes", "fpf"),
                                                    ("abf", "fpf")])
@pytest.mark.parametrize("shape", SHAPES)
def test_application_matches_oracle(shape, decoupling, composition):
    from paper_1606_00548_amd import cprmi
    gen = synth.black_oil_layered if shape[2] > 1 else synth.oil_water_lognormal
    case = gen(*shape)
    nx, ny, nz = shape
    case["wells"] = [synth.well(0, 0, nz, "inj", 300.0), synth.well(nx - 1, ny - 1, nz, "prod", 150.0)]
    x = synth.random_state_perturbation(case, 5)
    R, J = model.assemble(case["grid"], case["fluid"], case["perm"], case["poro"], case["wells"], case["x_old"], x,
                          case["dt"])
    s = cprmi.Solver.from_case(case)
    s.import_jacobian(J)
    v = -R / np.linalg.norm(R)
    t = torch.as_tensor(np.ascontiguousarray(v)).cuda()
    for pre, post in ((1, 1), (2, 2)):
        ref = cpr.cpr_apply(cpr.cpr_setup(J, 16, decoupling=decoupling, pre=pre, post=post), v, composition=composition)
        for precision, tol in (("fp64", 1e-9), ("mixed", 1e-5)):
            s.setup(precision=precision, mg_coarsest=16, mg_pre=pre, mg_post=post, decoupling=decoupling,
                    composition=composition)
            z = s.precond(t).cpu().numpy()
            assert np.linalg.norm(z - ref) <= tol * np.linalg.norm(ref)
