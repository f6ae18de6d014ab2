"""The vector behind the last basis vector of an FGMRES cycle: what is left of
A M^-1 v after its projection, in one piece whichever way the cycle stores its
vectors (black halves, or whole ones with tiles as colours).  The projection is
formed here from the exported basis with the library's products, to the
1e-11 of the Arnoldi relation's tests."""
import pytest

from paper_1606_00548_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ilu_order", ["red-black", "tiles"])
@pytest.mark.parametrize("model,shape", [("oil-water", (10, 7, 5)), ("black-oil", (12, 9, 7)), ("black-oil", (16, 16, 8))])
def test_vector_behind_the_basis(model, shape, ilu_order):
    from paper_1606_00548_amd import cprmi
    nx, ny, nz = shape
    case = (synth.black_oil_layered if model == "black-oil" else synth.oil_water_lognormal)(nx, ny, nz)
    case["wells"] = [synth.well(0, 0, nz, "inj", 300.0), synth.well(nx - 1, ny - 1, nz, "prod", 150.0)]
    s = cprmi.Solver.from_case(case)
    t = lambda a: torch.as_tensor(a).cuda().contiguous()   # noqa: E731
    rhs = s.assemble(t(case["x_old"]), t(synth.random_state_perturbation(case, 3)), case["dt"])
    k = 4
    s.setup(rtol=0.0, max_iter=k, ilu_order=ilu_order, mg_coarsest=16)
    s.solve(torch.randn_like(rhs))      # other vectors in the slots before
    _, st = s.solve(rhs)
    assert st["iterations"] == k and st["cycles"] == 1
    V = torch.stack([s.export_krylov(j).flatten() for j in range(k)])
    u = s.export_krylov(k).flatten()
    w = s.spmv(s.precond(V[-1].reshape(rhs.shape))).flatten()
    left = w - V.T @ (V @ w)
    assert float((u - left).norm()) <= 1e-11 * float(w.norm())
