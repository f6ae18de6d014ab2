"""cpr_spmv in natural order (vectors apart) against its route through
colour-split copies (a product in place, y = x): the sums run in the same
order, so the products must agree bit for bit, for every block size, on grids
whose rows are no multiple of a wave, down to one cell per colour, and on both
sides of the 1 M-cell launch limit of 3x3 systems."""
import pytest

from paper_1606_00548_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("b,shape", [(1, (2, 1, 1)), (1, (18, 7, 5)), (2, (2, 3, 9)), (2, (60, 22, 17)), (3, (6, 5, 1)),
                                     (3, (70, 9, 11)), (3, (128, 96, 86))])
def test_natural_product_equals_the_permuted_one(b, shape):
    from paper_1606_00548_amd import cprmi
    nx, ny, nz = shape
    fluid = {1: synth.SINGLE_PHASE, 2: synth.OIL_WATER, 3: synth.BLACK_OIL}[b]
    one = torch.ones((3, nz, ny, nx), dtype=torch.float64, device="cuda")
    s = cprmi.Solver(synth.grid_of(nx, ny, nz), fluid, one, one[0].contiguous(), [])
    gen = torch.Generator(device="cuda").manual_seed(b)
    rnd = lambda *d: torch.randn(*d, generator=gen, dtype=torch.float64, device="cuda")   # noqa: E731
    J = rnd(7, b, b, nz, ny, nx)
    for d, (axis, edge) in enumerate(((2, 0), (2, -1), (1, 0), (1, -1), (0, 0), (0, -1)), start=1):
        J[d].select(2 + axis, edge).zero_()      # blocks towards cells outside the grid
    s.import_jacobian(J)
    x = rnd(b, nz, ny, nx)
    y = s.spmv(x)
    z = x.clone()
    s.spmv(z, z)
    assert torch.equal(y, z)
    # and against the stencil itself: 7 b products a sum, eps of each
    ref = torch.einsum("rczyx,czyx->rzyx", J[0], x)
    for d, (axis, step) in enumerate(((2, 1), (2, -1), (1, 1), (1, -1), (0, 1), (0, -1)), start=1):
        ref += torch.einsum("rczyx,czyx->rzyx", J[d], torch.roll(x, step, dims=1 + axis))
    assert float((y - ref).abs().max()) <= 1e-13 * 7 * b * float(J.abs().max() * x.abs().max())
