"""Well indices of many perforations, gathered by one kernel: as many as one
workgroup of it has threads, one less and one more, in one well and in two,
against the oracle's residual and Jacobian to 1e-13 of the largest entry, as
in the other assembly tests."""
import numpy as np
import pytest

from oracle import model
from paper_1606_00548_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nz,split", [(255, 255), (256, 256), (257, 257), (140, 139), (1, 1)])
def test_assembly_with_many_perforations_matches_oracle(nz, split):
    from paper_1606_00548_amd import cprmi
    case = synth.oil_water_lognormal(4, 2, nz)
    wells = [synth.well(1, 1, split, "inj", 300.0)]
    if split < nz:
        wells.append(synth.well(2, 0, nz, "prod", 150.0))
    case["wells"] = wells
    x = synth.random_state_perturbation(case, 5)
    R, J = model.assemble(case["grid"], case["fluid"], case["perm"], case["poro"], wells, case["x_old"], x, case["dt"])
    s = cprmi.Solver.from_case(case)
    t = lambda a: torch.as_tensor(np.ascontiguousarray(a)).cuda()   # noqa: E731
    rhs = s.assemble(t(case["x_old"]), t(x), case["dt"]).cpu().numpy()
    assert np.abs(s.export_jacobian().cpu().numpy() - J).max() <= 1e-13 * np.abs(J).max()
    assert np.abs(rhs + R).max() <= 1e-13 * max(np.abs(R).max(), np.abs(J).max())
