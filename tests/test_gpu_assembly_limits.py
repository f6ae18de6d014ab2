"""Residuals at the limits of the fluid data that cpr_create takes, where
quotients are infinite: end points of the relative permeabilities that meet
(s_wc + s_or = 1, sg_den = 0), so that a normalised saturation is plus or minus
infinity and clips to 1 or 0.  Against the oracle, whose NumPy divisions do the
same, to 1e-13 of the largest entry as in the other assembly tests.  (Their
derivatives are 0 / 0 on both sides.)"""
import numpy as np
import pytest

from oracle import model
from paper_1606_00548_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,limits", [("oil-water", dict(s_wc=0.25, s_or=0.75)), ("black-oil", dict(sg_den=0.0)),
                                         ("black-oil", dict(s_wc=0.25, s_or=0.75)),
                                         ("black-oil", dict(s_wc=0.25, s_or=0.75, sg_den=0.0))])
def test_residual_is_finite(name, limits):
    from paper_1606_00548_amd import cprmi
    case = (synth.black_oil_layered if name == "black-oil" else synth.oil_water_lognormal)(12, 7, 5)
    case["fluid"] = dict(case["fluid"], **limits)
    rng = np.random.default_rng(4)
    x = case["x_old"].copy()
    x[0] += 5.0 * rng.standard_normal(x[0].shape)
    x[1] = np.where(rng.random(x[0].shape) < 0.5, 0.125, 0.375)
    if name == "black-oil":
        x[2] = rng.uniform(0.05, 0.2, x[0].shape)
    with np.errstate(all="ignore"):
        R, _ = model.assemble(case["grid"], case["fluid"], case["perm"], case["poro"], [], case["x_old"], x, case["dt"])
    assert np.isfinite(R).all()
    t = lambda a: torch.as_tensor(np.ascontiguousarray(a)).cuda()   # noqa: E731
    s = cprmi.Solver(case["grid"], case["fluid"], case["perm"], case["poro"], [])
    rhs = s.assemble(t(case["x_old"]), t(x), case["dt"]).cpu().numpy()
    assert np.abs(rhs + R).max() <= 1e-13 * np.abs(R).max()
