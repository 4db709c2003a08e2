"""The adjoint on tiles in LDS (three backward steps per launch, states recomputed several steps
per launch) against the same gradient with checkpoints every other step, whose segments are too
short for either: bitwise equal.  Grids end one node before, at and after a tile of 16 nodes, on
walled and periodic axes; the larger grids take each form of the recompute."""
import pytest
import torch

from paper_1308_2071_amd import Cavity, workloads

pytestmark = pytest.mark.gpu

CAV = dict(bc=(0, 0, 1, 1), T_wall=(1.0, 0.0, 0.0, 0.0))
MIX = dict(bc=(0, 1, 1, 0), T_wall=(1.0, 0.0, 0.0, 0.3))
ISO = dict(bc=(0, 0, 0, 0), T_wall=(1.0, 0.0, 0.6, 0.2))
CHY = dict(bc=(0, 0, 2, 2), T_wall=(1.0, 0.0, 0.0, 0.0), ext_accel=(0.0, 2e-5))


def gradient(params, dtype, every, steps, medium):
    nx, ny = params["nx"], params["ny"]
    tdt = torch.float64 if dtype == "fp64" else torch.float32
    kw = dict(phi_uniform=0.55)
    if medium:
        phi, K = workloads.random_medium(ny, nx, seed=nx + 3 * ny)
        kw = dict(phi=torch.tensor(phi, dtype=tdt), K=torch.tensor(K, dtype=tdt))
    p = dict(params, dtype=dtype, tau_v=0.7, tau_T=0.8, gbeta=1e-3, checkpoint_every=every)
    c = Cavity(p, nsteps_max=steps, **kw)
    c.step(steps)
    out = [g.clone() for g in c.grad()]
    c.close()
    return out


def compare(params, dtype, every, steps, medium=True):
    want = gradient(params, dtype, 2, steps, medium)
    got = gradient(params, dtype, every, steps, medium)
    for a, b, k in zip(want, got, ("phi", "K")):
        assert torch.isfinite(a).all() and a.abs().max() > 0, k
        assert torch.equal(a, b), (params, dtype, every, k)


@pytest.mark.parametrize("dtype", ["fp32", "fp64"])
@pytest.mark.parametrize("bc", [CAV, MIX, ISO, CHY], ids=["cav", "mix", "iso", "chy"])
@pytest.mark.parametrize("shape", [(5, 5), (15, 16), (16, 17), (17, 18), (18, 33), (31, 32),
                                   (33, 34), (35, 15), (49, 31), (6, 2), (33, 3)])
def test_tile_edges(shape, bc, dtype):
    nx, ny = shape
    if ny < 5 and bc["bc"][2] != 2:
        pytest.skip("a walled axis needs five nodes")
    compare(dict(bc, nx=nx, ny=ny), dtype, 8, 21)      # sweeps of 8 and 5: tiles and single steps


def test_uniform_medium():
    compare(dict(CAV, nx=47, ny=35), "fp32", 7, 20, medium=False)


@pytest.mark.parametrize("dtype", ["fp32", "fp64", "fp32_f64"])
@pytest.mark.parametrize("shape", [(330, 333), (331, 334), (400, 310), (450, 340), (1540, 1537)])
def test_recompute_forms(shape, dtype):
    """Both sides of 110,000 nodes (the last grid of three backward steps per launch and of four
    recomputed), of 150,000 and of the larger tiles."""
    nx, ny = shape
    compare(dict(CAV, nx=nx, ny=ny), dtype, 9, 13)
