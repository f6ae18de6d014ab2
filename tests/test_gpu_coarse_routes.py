"""The routes of the small multigrid levels: all of them in the
single-workgroup kernel's LDS, some or all of them as multi-block kernels
with the coarsest solve as a kernel of its own.  Cells of the levels below
4,096: 2,380 over 315 (odd nx, natural coarsest), 1,600 over 200, 1,872 over
234 (odd ny), 1,920 over 240 and 1,944 over 243 leave the kernel; 864 alone
is a coarsest level of its own (mg_coarsest 1000).  The levels that stay in
it are the other parity tests'.  Each against the
oracle: one application of each cycle to 1e-9 in FP64 and 1e-5 with the FP32
preconditioner (tolerances as in the other parity tests)."""
import numpy as np
import pytest

from oracle import cpr, model
from paper_1606_00548_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

CASES = {(20, 28, 34): 512, (40, 40, 8): 512, (48, 26, 12): 512, (40, 32, 12): 512, (36, 36, 12): 512,
         (24, 24, 12): 1000}


def _gpu(a):
    return torch.as_tensor(np.ascontiguousarray(a, dtype=np.float64)).cuda()


@pytest.mark.parametrize("shape", list(CASES))
def test_application_matches_oracle(shape):
    from paper_1606_00548_amd import cprmi
    case = synth.oil_water_lognormal(*shape)
    x = synth.random_state_perturbation(case, 5)
    R, J = model.assemble(case["grid"], case["fluid"], case["perm"], case["poro"], case["wells"], case["x_old"], x,
                          case["dt"])
    s = cprmi.Solver.from_case(case)
    s.import_jacobian(J)
    v = -R / np.linalg.norm(R)
    for pre, post, alpha in ((1, 1, 1.0), (2, 2, 1.25)):
        ref = cpr.cpr_apply(cpr.cpr_setup(J, CASES[shape], pre=pre, post=post), v, alpha=alpha)
        for precision, tol in (("fp64", 1e-9), ("mixed", 1e-5)):
            s.setup(precision=precision, mg_coarsest=CASES[shape], mg_pre=pre, mg_post=post, mg_alpha=alpha)
            z = s.precond(_gpu(v)).cpu().numpy()
            assert np.linalg.norm(z - ref) <= tol * np.linalg.norm(ref)
