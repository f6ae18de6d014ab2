"""Mixed solves that fall back to FP64, pinned to the bit.

A solve falls back where the FP32 preconditioner stalls, and such systems have
modes that amplify last bits: with a coarsest inverse that differed by rounding
alone, dx of 256x256x64 cells moved by 4e-5 in 75 iterations (one iteration
fewer).  So the fallback keeps one elimination of the coarsest level and one
order of every sum for good.  The values are those of the elimination in one
workgroup's LDS (up to 128 cells) or in one launch a column, and of one
workgroup's dense product.

Inputs are exact in binary (no wells, rock of a few values); every first cycle
of five steps is declared stalled.  Coarsest levels of 8 (below 64), 180, 240,
288, 432, 512, 864 and 1,150 cells; both ILU orders and orthogonalisations;
ABF."""
import hashlib

import numpy as np
import pytest

from paper_1606_00548_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# model, grid, options: iterations, true relative residual, dx
CASES = [
    ("black-oil", (20, 46, 9), dict(), 14, "0x1.343fcbcb1441cp-21", "e3e3fc0fe4500e7c"),
    ("black-oil", (20, 46, 9), dict(ilu_order="tiles"), 13, "0x1.35712fb687920p-21", "1e437c9c06eb3254"),
    ("black-oil", (20, 46, 9), dict(orth="cgs2"), 14, "0x1.343fcbcb16ae4p-21", "360a61c5de65237a"),
    ("black-oil", (20, 46, 9), dict(decoupling="abf"), 14, "0x1.89451dbe3d0b7p-21", "6dd2deb875b3b17e"),
    ("black-oil", (20, 46, 9), dict(mg_coarsest=64), 14, "0x1.3eabf7b89b117p-21", "0ba282365debbc73"),
    ("oil-water", (96, 64, 24), dict(), 14, "0x1.f16c552283933p-21", "0aa198f1c5f32ba7"),
    ("oil-water", (96, 64, 24), dict(ilu_order="tiles"), 14, "0x1.29e55631a25fep-21", "097df12ae30a9974"),
    ("oil-water", (96, 64, 24), dict(orth="cgs2"), 14, "0x1.f16c5522861e1p-21", "27d2ca33a201a06d"),
    ("oil-water", (96, 64, 24), dict(decoupling="abf"), 17, "0x1.aed3515c6badfp-21", "dd1c83dd6b04a7b6"),
    ("oil-water", (96, 64, 24), dict(mg_coarsest=64), 15, "0x1.48c79bf256ac6p-21", "91dc33817651571a"),
    ("black-oil", (32, 32, 32), dict(), 15, "0x1.ffbc96bc73314p-22", "334a29d167c39509"),
    ("black-oil", (96, 96, 24), dict(), 16, "0x1.82e2e313f71b9p-21", "55067d1d646a9e7b"),
    ("black-oil", (8, 6, 5), dict(), 6, "0x1.fed11251a467dp-23", "11fa94fe987daa84"),
    ("black-oil", (20, 46, 9), dict(mg_coarsest=1200), 13, "0x1.a3e9c95003e38p-22", "67e1d3f318b2b043"),
    ("black-oil", (70, 46, 15), dict(), 15, "0x1.f5b52b689b235p-21", "87636c957bb631e6"),
    ("black-oil", (24, 24, 12), dict(mg_coarsest=1000), 12, "0x1.a4d73eccb55e8p-21", "4eb7acb6c287eaa8"),
]


@pytest.mark.parametrize("model,shape,options,iterations,true_rel,dx", CASES)
def test_fallback_keeps_its_bits(model, shape, options, iterations, true_rel, dx):
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
    for _ in range(2):     # a second solve forms the fallback's inverse anew
        d, st = cprmi.newton_step(s, t(x_old), t(x), 1.0, precision="mixed", restart=5, stall_ratio=1e-300, **options)
        assert st["fp64_fallback"] == 1
        assert (st["iterations"], st["true_rel"].hex()) == (iterations, true_rel)
        assert hashlib.sha256(d.cpu().numpy().tobytes()).hexdigest()[:16] == dx
