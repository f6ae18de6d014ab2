"""A coarsest multigrid level of a single cell (mg_coarsest 1, or below the
eight cells of the level above it): there is no black cell to eliminate and
the inverse is 1 / A.  One application against the oracle, to 1e-9 in FP64 and
1e-5 with the FP32 preconditioner (tolerances as in the other parity tests),
and a solve to its tolerance."""
import numpy as np
import pytest

from oracle import cpr, model
from paper_1606_00548_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("coarsest", [1, 2, 7])
@pytest.mark.parametrize("shape", [(8, 8, 8), (2, 2, 2), (6, 5, 3), (14, 9, 1), (32, 32, 8)])
def test_application_and_solve(shape, coarsest):
    from paper_1606_00548_amd import cprmi
    case = synth.oil_water_lognormal(*shape)
    x = synth.random_state_perturbation(case, 5)
    R, J = model.assemble(case["grid"], case["fluid"], case["perm"], case["poro"], case["wells"], case["x_old"], x,
                          case["dt"])
    s = cprmi.Solver.from_case(case)
    s.import_jacobian(J)
    v = -R / np.linalg.norm(R)
    t = torch.as_tensor(np.ascontiguousarray(v)).cuda()
    ref = cpr.cpr_apply(cpr.cpr_setup(J, coarsest), v)
    for precision, tol in (("fp64", 1e-9), ("mixed", 1e-5)):
        s.setup(precision=precision, mg_coarsest=coarsest, rtol=1e-6)
        z = s.precond(t).cpu().numpy()
        assert np.linalg.norm(z - ref) <= tol * np.linalg.norm(ref)
        _, st = s.solve(t)
        assert st["status"] == 0 and st["true_rel"] <= 1e-6
