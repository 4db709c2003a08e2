"""Two and three steps per launch on tiles in LDS against one step per launch, bitwise, where the
tiles and their regions end: one node more or less than a tile (30 x 14 and 62 x 14 for two steps,
28 x 12 and 28 x 28 for three), tiles one node thick at a wall, periodic axes shorter than a
region, and grids on both sides of the size from which the larger tiles are taken; the default
form of FP64 grids, which may take three steps, included."""
import pytest
import torch

from paper_1308_2071_amd import Cavity, lbm_step_shape, workloads

pytestmark = pytest.mark.gpu

CAV = dict(bc=(0, 0, 1, 1), T_wall=(1.0, 0.0, 0.0, 0.0))
MIX = dict(bc=(1, 0, 0, 0), T_wall=(0.0, 0.2, 1.0, 0.6))
CHX = dict(bc=(2, 2, 0, 1), T_wall=(0.0, 0.0, 1.0, 0.0), ext_accel=(1e-5, 0.0))
BOX = dict(bc=(2, 2, 2, 2), ext_accel=(3e-5, -1e-5), T_init=0.4)


def compare(params, dtype, spl, steps, medium=True):
    nx, ny = params["nx"], params["ny"]
    tdt = torch.float64 if dtype == "fp64" else torch.float32
    kw = dict(phi_uniform=0.55)
    if medium:
        phi, K = workloads.random_medium(ny, nx, seed=nx + 3 * ny)
        kw = dict(phi=torch.tensor(phi, dtype=tdt), K=torch.tensor(K, dtype=tdt))
    base = dict(params, dtype=dtype, tau_v=0.7, tau_T=0.8, gbeta=1e-3)
    a = Cavity(dict(base, steps_per_launch=1), **kw)
    b = Cavity(dict(base, steps_per_launch=spl), **kw)
    for n in steps:
        a.step(n)
        b.step(n)
        oa, ob = a.observables(), b.observables()
        for k in ("ux", "uy", "p", "T"):
            assert torch.equal(oa[k], ob[k]), (params, dtype, spl, n, k)
    shape = lbm_step_shape(b.ctx)
    a.close()
    b.close()
    return shape


@pytest.mark.parametrize("dtype", ["fp32", "fp64", "fp32_f64"])
@pytest.mark.parametrize("bc", [CAV, MIX, CHX, BOX], ids=["cav", "mix", "chx", "box"])
@pytest.mark.parametrize("shape", [(5, 5), (29, 13), (30, 14), (31, 15), (61, 29), (91, 43),
                                   (2, 7), (40, 2)])
def test_two_steps(shape, bc, dtype):
    nx, ny = shape
    if (nx < 5 and bc["bc"][0] != 2) or (ny < 5 and bc["bc"][2] != 2):
        pytest.skip("a walled axis needs five nodes")
    s = compare(dict(bc, nx=nx, ny=ny), dtype, 2, (2, 7))
    assert s[0] == 2 and s[2] == 14


@pytest.mark.parametrize("bc", [CAV, MIX, CHX, BOX], ids=["cav", "mix", "chx", "box"])
@pytest.mark.parametrize("shape", [(5, 5), (27, 11), (28, 12), (29, 13), (57, 25), (85, 37),
                                   (2, 9), (40, 3)])
def test_three_steps(shape, bc):
    nx, ny = shape
    if (nx < 5 and bc["bc"][0] != 2) or (ny < 5 and bc["bc"][2] != 2):
        pytest.skip("a walled axis needs five nodes")
    s = compare(dict(bc, nx=nx, ny=ny), "fp32", 3, (3, 8))
    assert s[0] == 3 and s[2] == 12


@pytest.mark.parametrize("dtype,spl,rows", [("fp32", 2, 14), ("fp64", 2, 14), ("fp32", 3, 28),
                                            ("fp64", 0, 12), ("fp32_f64", 0, 14)])
@pytest.mark.parametrize("shape", [(1551, 1541), (1541, 1569)])
def test_larger_tiles_on_larger_grids(shape, dtype, spl, rows):
    """1551 is one more than a multiple of 62, 1541 and 1569 than one of 28 (and 14): the last tiles
    are one node thick."""
    nx, ny = shape
    s = compare(dict(CAV, nx=nx, ny=ny), dtype, spl, (7,))
    assert s[2] == rows


@pytest.mark.parametrize("shape", [(400, 381), (513, 300)])
def test_fp64_default_takes_three_steps(shape):
    s = compare(dict(MIX, nx=shape[0], ny=shape[1]), "fp64", 0, (3, 100), medium=False)
    assert s[0] == 3
