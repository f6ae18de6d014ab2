"""Black-row FGMRES cycles and products on the GPU.

The red-black block ILU(0) solves the red rows of the decoupled system
exactly, so (A M^-1 v)_red = v_red; FGMRES then keeps the red half of its
basis as one multiple per vector, and BiCGSTAB and the CGS2 path copy the red
half of each product.  Checked on grids whose colour half is no multiple of
the 64-cell tile (and one that is), for every decoupling and composition:
the identity itself, the orthonormality of the exported basis, and the
Arnoldi relation, with whole products of the library's SpMV.

Tolerances: both sides of the identity carry eps |A| |z| (eps = 1.1e-16),
which for these systems is at most 1e-13 |v| (|A| |z| / |v| <= 1e3); the
basis is orthonormal to a few eps times its length, as whole vectors are.
1e-11 and 1e-12 leave two orders for the sums.
"""
import numpy as np
import pytest

from paper_1606_00548_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

CASES = [("oil-water", (2, 5, 3)), ("oil-water", (10, 7, 5)), ("black-oil", (6, 5, 1)), ("black-oil", (12, 9, 7)),
         ("black-oil", (16, 16, 8)), ("single", (18, 3, 5))]


def _solver(model, shape):
    from paper_1606_00548_amd import cprmi
    nx, ny, nz = shape
    if model == "single":
        case = synth.single_phase_uniform(nx, ny, nz, wells=[synth.well(0, 0, nz, "inj", 300.0)])
    else:
        gen = synth.black_oil_layered if model == "black-oil" else synth.oil_water_lognormal
        case = gen(nx, ny, nz)
        case["wells"] = [synth.well(0, 0, nz, "inj", 300.0), synth.well(nx - 1, ny - 1, nz, "prod", 150.0)]
    s = cprmi.Solver.from_case(case)
    t = lambda a: torch.as_tensor(a).cuda().contiguous()   # noqa: E731
    rhs = s.assemble(t(case["x_old"]), t(synth.random_state_perturbation(case, 3)), case["dt"])
    return s, rhs


def _red(shape):
    nx, ny, nz = shape
    k, j, i = np.meshgrid(range(nz), range(ny), range(nx), indexing="ij")
    return torch.as_tensor((i + j + k) % 2 == 0).cuda()


@pytest.mark.parametrize("decoupling,composition", [("qimpes", "two-stage"), ("abf", "two-stage"), ("qimpes", "fpf"),
                                                    ("abf", "fpf")])
@pytest.mark.parametrize("model,shape", CASES)
def test_red_rows_and_arnoldi_relation(model, shape, decoupling, composition):
    s, rhs = _solver(model, shape)
    red = _red(shape)
    k = 4
    opts = dict(rtol=0.0, max_iter=k, decoupling=decoupling, composition=composition)
    s.setup(**opts)
    v = torch.randn_like(rhs)
    y = s.spmv(s.precond(v))
    assert float((y - v)[:, red].abs().max()) <= 1e-11 * float(v.norm())
    _, st = s.solve(rhs)
    # vectors of the last cycle: all steps, unless an exact preconditioner (a
    # single pressure level) broke the first cycle off
    n = st["iterations"] if st["cycles"] == 1 else 1
    V = torch.stack([s.export_krylov(j).flatten() for j in range(n)])
    eye = torch.eye(n, dtype=V.dtype, device=V.device)
    assert float((V @ V.T - eye).abs().max()) <= 1e-12
    for j in range(n - 1):
        w = s.spmv(s.precond(V[j].reshape(rhs.shape))).flatten()
        basis = V[:j + 2]
        left = w - basis.T @ (basis @ w)
        assert float(left.norm()) <= 1e-11 * float(w.norm())


@pytest.mark.parametrize("model,shape", CASES)
def test_methods_with_copied_red_rows_agree(model, shape):
    # DCGS2 (black halves), CGS2 and BiCGSTAB (copied red rows) solve to the
    # same solution: each stops at 1e-10 of a residual computed whole
    s, rhs = _solver(model, shape)
    sol = {}
    for orth in ("dcgs2", "cgs2"):
        s.setup(rtol=1e-10, orth=orth)
        sol[orth], st = s.solve(rhs)
        assert st["status"] == 0 and st["true_rel"] <= 1e-10
    sol["bicgstab"], st = s.bicgstab(rhs)
    assert st["status"] == 0 and st["true_rel"] <= 1e-10
    for q in sol.values():
        r = rhs - s.spmv(q)
        assert float(r.norm()) <= 2e-10 * float(rhs.norm())
