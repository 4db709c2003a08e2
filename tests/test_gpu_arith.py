"""The macroscopics' roots and quotients at operands where a Newton step can go wrong: no drag
(den = 1 exactly), drag over twelve decades, phi near its ends, speeds from the smallest normal to
the largest the scheme carries, each against the FP64 oracle after one step from a sheared state."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

from oracle import ref
from paper_1308_2071_amd import Cavity


@pytest.mark.parametrize("dtype", ["fp32", "fp64", "fp32_f64"])
@pytest.mark.parametrize("accel", [1e-30, 1e-12, 1e-4, 3e-2])
def test_velocity_over_the_range_of_drag_and_speed(dtype, accel):
    ny, nx = 24, 40
    rng = np.random.default_rng(5)
    phi = np.clip(rng.uniform(-0.1, 1.1, (ny, nx)), 1e-3, 1.0)
    K = 10.0 ** rng.uniform(-6, 6, (ny, nx))
    f32 = dtype != "fp64"
    if f32:
        phi, K = phi.astype(np.float32).astype(float), K.astype(np.float32).astype(float)
    params = dict(nx=nx, ny=ny, Ra=1e4, Pr=0.71, bc=(2, 2, 2, 2), ext_accel=(accel, -0.5 * accel),
                  tau_v=0.8, tau_T=0.9, gbeta=0.0, T_init=0.5)
    tdt = torch.float32 if f32 else torch.float64
    cav = Cavity(dict(params, dtype=dtype), phi=torch.tensor(phi, dtype=tdt),
                 K=torch.tensor(K, dtype=tdt))
    lat = ref.RefLattice(phi=phi, K=K, **params)
    # FP32: v is exact to a few roundings, |v| and |u| to 1 ulp each; 24 roundings cover one
    # step's chain.  FP64: the oracle carries populations with their rest part, so its velocity
    # moves by the rounding of 1 over the smallest denominator.
    for n in (1, 2):
        cav.step(1)
        lat.step(1)
        o, r = cav.observables(), lat.observables(dynamic_pressure=True)
        for k in ("ux", "uy"):
            g, e = o[k].double().cpu().numpy(), r[k]
            eps = 2.0 ** -24 if dtype == "fp32" else 2.0 ** -24 if f32 else 2.0 ** -53
            tol = 24 * eps * n * np.abs(e).max() + 16 * 2.0 ** -53
            assert np.isfinite(g).all()
            assert np.abs(g - e).max() <= tol, (dtype, accel, k, n)
    cav.close()
    lat.close()
