"""The observables and the stream function against the fields of the same state, at the sizes where
their launches change shape: one node per work-item or several, 16 columns per work-group of the
stream function and 256 rows at a time."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

from paper_1308_2071_amd import (LBM_PERIODIC, LBM_WALL_ADIABATIC, LBM_WALL_ISOTHERMAL, Batch,
                                 Cavity)

CAV = (LBM_WALL_ISOTHERMAL, LBM_WALL_ISOTHERMAL, LBM_WALL_ADIABATIC, LBM_WALL_ADIABATIC)
BOX = (LBM_PERIODIC,) * 4


def params(nx, ny, dtype, **kw):
    d = dict(nx=nx, ny=ny, bc=CAV, Ra=1e4, Pr=0.71, Da=1e-2, T_init=0.4, dtype=dtype)
    d.update(kw)
    return d


def check_obs(o, f, nx, ny, dtype):
    """Extremes are those of the stored fields; sums agree to the rounding of the fields they are
    formed from again here (u and T in the storage type, Nu's stencil times L)."""
    eps = 2.0 ** -52 if dtype == "fp64" else 2.0 ** -23
    T, ux, uy = (f[k].double().cpu().numpy() for k in ("T", "ux", "uy"))
    assert abs(o["T_min"] - T.min()) <= eps * abs(T.min())
    assert abs(o["T_max"] - T.max()) <= eps * abs(T.max())
    sp = np.hypot(ux, uy).max()
    assert abs(o["max_speed"] - sp) <= 4 * eps * sp
    c = np.array([-25.0, 48.0, -36.0, 16.0, -3.0]) / 12.0
    w = np.ones(ny)
    w[0] = w[-1] = 0.5
    L = nx - 1.0
    hot = -L / (ny - 1) * (w * (T[:, :5] @ c)).sum()
    cold = L / (ny - 1) * (w * (T[:, ::-1][:, :5] @ c)).sum()
    tol = 2 * eps * L * np.abs(c).sum() * 1.5    # each T within 1 ulp of up to 1.5
    assert abs(o["nu_hot"] - hot) <= tol and abs(o["nu_cold"] - cold) <= tol


@pytest.mark.parametrize("dtype", ["fp32", "fp64", "fp32_f64"])
@pytest.mark.parametrize("nx,ny", [(5, 5), (64, 64), (362, 362), (363, 363), (41, 1025),
                                   (1023, 300)])
def test_observables_match_the_fields(nx, ny, dtype):
    cav = Cavity(params(nx, ny, dtype), phi_uniform=0.5)
    o = cav.step(9).observables()
    check_obs(o, o, nx, ny, dtype)
    assert o["step"] == 9 and not o["diverged"]
    cav.close()


def test_batch_observables_match_the_fields(tmp_path):
    sizes = [(5, 7), (64, 64), (110, 112), (111, 111), (130, 128)]
    for dtype in ("fp32", "fp64"):
        b = Batch([params(nx, ny, dtype) for nx, ny in sizes], [0.5] * len(sizes))
        _, obs = b.step(7).observables()
        for i, (nx, ny) in enumerate(sizes):
            check_obs(obs[i], b.fields(i), nx, ny, dtype)
            ref = Cavity(params(nx, ny, dtype), phi_uniform=0.5)
            r = ref.step(7).observables(fields=False)
            assert all(r[k] == obs[i][k] for k in ("nu_hot", "nu_cold", "max_speed", "T_min",
                                                   "T_max", "phip_dev"))
            ref.close()
        b.close()


@pytest.mark.parametrize("dtype", ["fp32", "fp64", "fp32_f64"])
@pytest.mark.parametrize("layout", ["pull", "aa"])
@pytest.mark.parametrize("nx,ny,bc", [(5, 5, CAV), (16, 255, CAV), (17, 256, CAV), (15, 257, CAV),
                                      (33, 513, CAV), (300, 61, CAV), (2, 2, BOX),
                                      (18, 260, BOX)])
def test_stream_function_integrates_u(nx, ny, bc, layout, dtype):
    cav = Cavity(params(nx, ny, dtype, bc=bc, layout=layout, tau_v=0.8, tau_T=0.9, gbeta=1e-3,
                        ext_accel=(1e-4, 2e-5)), phi_uniform=0.6)
    o = cav.step(5).observables()
    psi = cav.stream_function().double().cpu().numpy()
    u = o["ux"].double().cpu().numpy()
    ref = np.zeros((ny, nx))
    ref[1:] = np.cumsum(0.5 * (u[1:] + u[:-1]), axis=0)
    # u is rounded to the storage type in `ref` but not in psi, whose own rounding comes on top
    eps = 2.0 ** -52 if dtype == "fp64" else 2.0 ** -23
    tol = eps * (np.cumsum(np.abs(u), axis=0) + np.abs(ref)) * (ny if dtype == "fp64" else 1)
    assert (np.abs(psi - ref) <= tol + 1e-300).all()
    cav.close()
