"""The stream function of wide grids, whose work-groups take 64 columns and 32 rows at a time instead
of 16 and 256: around the limits of that rule and its rows, against the integral of the stored u, and
the time of a wide grid of five rows, of which the other form leaves most work-items without a row."""
import numpy as np
import pytest
import torch

from paper_1308_2071_amd import Cavity

pytestmark = pytest.mark.gpu


def cavity(nx, ny, dtype, **kw):
    return Cavity(dict(nx=nx, ny=ny, bc=(2, 2, 0, 1) if ny >= 5 else (2, 2, 2, 2), dtype=dtype,
                       T_wall=(0.0, 0.0, 1.0, 0.0), tau_v=0.8, tau_T=0.9, gbeta=1e-3, T_init=0.4,
                       ext_accel=(1e-4, 2e-5), **kw), phi_uniform=0.6)


@pytest.mark.parametrize("dtype", ["fp32", "fp64", "fp32_f64"])
@pytest.mark.parametrize("layout", ["pull", "aa"])
@pytest.mark.parametrize("nx,ny", [(8191, 5), (8192, 2), (8193, 31), (8255, 33), (8192, 256),
                                   (8192, 257), (32769, 300)])
def test_stream_function_of_wide_grids(nx, ny, layout, dtype):
    cav = cavity(nx, ny, dtype, layout=layout)
    u = cav.step(5).observables()["ux"].double().cpu().numpy()
    psi = cav.stream_function().double().cpu().numpy()
    ref = np.zeros((ny, nx))
    ref[1:] = np.cumsum(0.5 * (u[1:] + u[:-1]), axis=0)
    # u is rounded to the storage type in `ref` but not in psi, whose own rounding comes on top
    eps = 2.0 ** -52 if dtype == "fp64" else 2.0 ** -23
    tol = eps * (np.cumsum(np.abs(u), axis=0) + np.abs(ref)) * (ny if dtype == "fp64" else 1)
    assert np.abs(psi).max() > 0 and (np.abs(psi - ref) <= tol + 1e-300).all()
    cav.close()


def test_a_wide_grid_of_few_rows_takes_a_fraction_of_a_higher_one():
    """88 of 163 us before the rule, 20 of 84 with it."""
    def best(c):
        e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        times = []
        for _ in range(20):
            e[0].record()
            c.stream_function()
            e[1].record()
            e[1].synchronize()
            times.append(e[0].elapsed_time(e[1]))
        return min(times)
    low, high = cavity(100000, 5, "fp32"), cavity(100000, 60, "fp32")
    assert best(low) < 0.4 * best(high)
    low.close()
    high.close()
