"""The mixed-precision solve, pinned to the bit.

Its FP32 preconditioner rounds every Krylov vector, so a last bit of a norm or
of a Gram-Schmidt coefficient becomes another FP32 value in some of millions of
entries, and the solution of the stopped iteration moves by up to 1e-8 where
the matrix has an outlying mode.  The whole-vector route therefore keeps its
order of summation: norms over whole vectors, |a|^2 and a.c one term after the
other.  The values are those of the kernels that formed each of these sums in
a launch of its own.

Inputs are exact in binary (no wells, rock of a few values), so that only GPU
arithmetic enters; both ILU orders, both orthogonalisations, and time steps
whose forcing terms read the residual norms.
"""
import hashlib

import numpy as np
import pytest

from paper_1606_00548_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# model, grid, ILU order, orthogonalisation, dt: iterations, ||b||, true
# relative residual and dx of a Newton step; x of a time step with EW1, EW2
CASES = [
    ("black-oil", (20, 46, 9), "red-black", "dcgs2", 1.0,
     (12, "0x1.cd376bd74e4b9p+5", "0x1.9afb2c57c98ecp-21", "5da45b9481a7378d"), "2a50e5d3070de709", "d75364eb79b67559"),
    ("black-oil", (40, 95, 3), "red-black", "dcgs2", 0.05,
     (7, "0x1.dc1ece51569c2p+2", "0x1.58180e91a72b4p-22", "a6579b904d73aba3"), "e0409ae855d4be37", "d9cbc51084e63198"),
    ("black-oil", (68, 30, 5), "red-black", "dcgs2", 0.05,
     (7, "0x1.ca3b4a94f3e64p+2", "0x1.9e25e38b8be16p-22", "5cb3a69a7fd20db0"), "3c9a8b971071936b", "1494d2372149191b"),
    ("oil-water", (96, 64, 24), "red-black", "dcgs2", 0.05,
     (8, "0x1.7dbb47e09474ep+4", "0x1.ced6f0c1e6a75p-21", "71f074495e8c5c47"), "a317de405b9e6d65", "b18ab4b6f8cd9aad"),
    ("black-oil", (26, 56, 14), "tiles", "dcgs2", 1.0,
     (12, "0x1.6c504d35ffce5p+6", "0x1.c2ef316600a96p-22", "3562e07602b2ba9d"), "ace97b18a0b6aa94", "ace97b18a0b6aa94"),
    ("black-oil", (26, 56, 14), "red-black", "cgs2", 1.0,
     (13, "0x1.6c504d35ffce5p+6", "0x1.3561d8a0ab314p-21", "0b80a55031540c2c"), "062a3828dd58b3eb", "c24ce6fcde92427b"),
    ("black-oil", (96, 96, 24), "red-black", "dcgs2", 0.05,
     (7, "0x1.0c980e3b3b869p+5", "0x1.fcd2b7cd0c0e9p-22", "dac5564adde2b11c"), "a334653f2865f7f7", "5774917a2eebe7e9"),
]


def _hash(t):
    return hashlib.sha256(t.cpu().numpy().tobytes()).hexdigest()[:16]


@pytest.mark.parametrize("model,shape,ilu,orth,dt,step,ew1,ew2", CASES)
def test_newton_and_time_steps_keep_their_bits(model, shape, ilu, orth, dt, step, ew1, ew2):
    from paper_1606_00548_amd import cprmi
    nx, ny, nz = shape
    rng = np.random.default_rng(nx)
    cells = (nz, ny, nx)
    fluid = synth.BLACK_OIL if model == "black-oil" else synth.OIL_WATER
    grid = synth.grid_of(nx, ny, nz)
    k = np.array([2.0, 16.0, 128.0, 512.0])[rng.integers(0, 4, cells)]
    poro = np.array([0.125, 0.1875, 0.25])[rng.integers(0, 3, cells)]
    x_old = synth.initial_state(grid, fluid)
    x = x_old.copy()
    x[0] += 0.25 * rng.integers(-20, 21, cells)
    x[1] += rng.integers(-4, 5, cells) / 64.0
    s = cprmi.Solver(grid, fluid, np.stack([k, k, 0.125 * k]), poro, [])
    t = lambda a: torch.as_tensor(a).cuda().contiguous()   # noqa: E731
    options = dict(precision="mixed", ilu_order=ilu, orth=orth)
    dx, st = cprmi.newton_step(s, t(x_old), t(x), dt, **options)
    assert (st["iterations"], st["bnorm"].hex(), st["true_rel"].hex(), _hash(dx)) == step
    for forcing, want in (("ew1", ew1), ("ew2", ew2)):
        xn, _ = s.time_step(t(x), dt, cprmi.default_options(**options), dict(forcing=forcing))
        assert _hash(xn) == want
