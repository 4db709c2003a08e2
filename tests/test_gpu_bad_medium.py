"""A porosity or permeability below zero or not a number at one node: the run is reported as diverged
(the square roots of Eq. (5) have no value there), in every precision, layout and form of the step."""
import pytest
import torch

from paper_1308_2071_amd import LBM_DIV_NONFINITE, Cavity, lbm_run_noalloc, make_params, workloads
from paper_1308_2071_amd._abi import LBM_E_DIVERGED

pytestmark = pytest.mark.gpu
BAD = [("K", -1.0), ("K", -1e-30), ("K", float("nan")), ("phi", -0.4), ("phi", float("nan"))]


def medium(nx, ny, dtype, which, value, at):
    tdt = torch.float64 if dtype == "fp64" else torch.float32
    m = dict(phi=torch.full((ny, nx), 0.5, dtype=tdt), K=torch.full((ny, nx), 10.0, dtype=tdt))
    m[which][at] = value
    return m


@pytest.mark.parametrize("dtype", ["fp32", "fp64", "fp32_f64"])
@pytest.mark.parametrize("which,value", BAD)
@pytest.mark.parametrize("at", [(9, 17), (1, 1), (19, 30)])
def test_flagged_in_every_form(dtype, which, value, at):
    p = workloads.cavity(40, 33, Ra=1e4, Pr=0.71, dtype=dtype)
    m = medium(40, 33, dtype, which, value, at)
    forms = [dict(steps_per_launch=k) for k in ((1, 2, 4, 8, 3) if dtype == "fp32" else (1, 2, 4, 8))]
    for form in forms + [dict(layout="aa")]:
        c = Cavity(dict(p, **form), **m)
        for n in (0, 8):
            o = c.step(n).observables()
            assert o["diverged"] and o["why"] & LBM_DIV_NONFINITE, (form, n, o["why"])
        c.close()
    g = {k: v.cuda() for k, v in m.items()}
    s, o = lbm_run_noalloc(make_params(**p), g["phi"], g["K"], 1.0, 5)
    assert s == LBM_E_DIVERGED and o.why & LBM_DIV_NONFINITE
