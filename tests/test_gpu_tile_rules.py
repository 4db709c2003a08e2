"""Which tile two steps per launch take by grid and types, seen in the work-groups per launch, and the
62 x 14 tiles in FP64 and the 30 x 14 ones with FP64 arithmetic on large grids bitwise against one step
per launch, with tiles one node wide and high at the walls."""
import pytest
import torch

from paper_1308_2071_amd import Cavity, lbm_step_shape, workloads

pytestmark = pytest.mark.gpu


def groups(nx, ny, cols, rows):
    return -(-nx // cols) * -(-ny // rows)


@pytest.mark.parametrize("nx,ny,dtype,cols", [
    (1540, 1530, "fp32", 30), (1541, 1535, "fp32", 62),
    (1541, 1569, "fp64", 30), (2500, 2499, "fp64", 30), (2500, 2500, "fp64", 62),
    (1541, 1569, "fp32_f64", 30), (2600, 2600, "fp32_f64", 30)])
def test_tile_of_two_steps(nx, ny, dtype, cols):
    c = Cavity(dict(workloads.cavity(nx, ny, Ra=1e5, Pr=0.71, dtype=dtype), steps_per_launch=2),
               phi_uniform=0.5)
    assert lbm_step_shape(c.ctx) == (2, 0, 14, groups(nx, ny, cols, 14))
    c.close()


@pytest.mark.parametrize("dtype", ["fp64", "fp32_f64"])
@pytest.mark.parametrize("medium", [False, True])
def test_large_grids_equal_single_steps(dtype, medium):
    nx, ny = 2543, 2521        # one more than a multiple of 62, and of 14
    tdt = torch.float64 if dtype == "fp64" else torch.float32
    kw = dict(phi_uniform=0.55)
    if medium:
        phi, K = workloads.random_medium(ny, nx, seed=3)
        kw = dict(phi=torch.tensor(phi, dtype=tdt), K=torch.tensor(K, dtype=tdt))
    fields = []
    for spl in (1, 2):
        c = Cavity(dict(workloads.cavity(nx, ny, Ra=1e5, Pr=0.71, dtype=dtype, tau_v=0.7, tau_T=0.8,
                                         gbeta=1e-3), steps_per_launch=spl), **kw)
        o = c.step(7).observables()
        fields.append([o[k] for k in ("ux", "uy", "p", "T")])
        c.close()
    for a, b in zip(*fields):
        assert torch.equal(a, b)
