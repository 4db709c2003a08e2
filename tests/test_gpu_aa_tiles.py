"""The AA layout against the pull layout, bitwise, where its tiles (128 x 2 nodes) end: last tiles
one node wide or high at a wall (which move so that wall nodes stay with their inward neighbours),
periodic axes of two nodes, and a state beyond the size that runs in tiles."""
import pytest
import torch

from paper_1308_2071_amd import Cavity, workloads

pytestmark = pytest.mark.gpu

BCS = {"cav": (0, 0, 1, 1), "iso": (0, 0, 0, 0), "chx": (2, 2, 0, 1), "chy": (0, 0, 2, 2),
       "box": (2, 2, 2, 2)}


def compare(nx, ny, bc, dtype, steps):
    phi, K = workloads.random_medium(ny, nx, seed=nx + ny)
    tdt = torch.float64 if dtype == "fp64" else torch.float32
    kw = dict(phi=torch.tensor(phi, dtype=tdt), K=torch.tensor(K, dtype=tdt))
    p = dict(nx=nx, ny=ny, bc=bc, T_wall=(1.0, 0.0, 0.3, 0.6), Ra=1e5, Pr=0.71, tau_v=0.7,
             tau_T=0.8, gbeta=1e-3, ext_accel=(1e-5, 2e-5), T_init=0.4, dtype=dtype)
    a = Cavity(dict(p, steps_per_launch=1), **kw)
    b = Cavity(dict(p, layout="aa"), **kw)
    for n in steps:
        oa, ob = a.step(n).observables(), b.step(n).observables()
        for k in ("ux", "uy", "p", "T"):
            assert torch.equal(oa[k], ob[k]), (nx, ny, bc, dtype, n, k)
    a.close()
    b.close()


@pytest.mark.parametrize("dtype", ["fp32", "fp64", "fp32_f64"])
@pytest.mark.parametrize("bc", list(BCS))
@pytest.mark.parametrize("shape", [(5, 5), (128, 6), (129, 7), (130, 9), (257, 5), (2, 8), (9, 2)])
def test_tiles(shape, bc, dtype):
    nx, ny = shape
    if (nx < 5 and BCS[bc][0] != 2) or (ny < 5 and BCS[bc][2] != 2):
        pytest.skip("a walled axis needs five nodes")
    compare(nx, ny, BCS[bc], dtype, (1, 2, 99))


@pytest.mark.parametrize("n", [2176, 2200])
def test_either_side_of_the_cache_size(n):
    """A state of 253 MiB (FP32, with its row pitch) runs in tiles, one of 263 MiB does not."""
    compare(n, n, BCS["cav"], "fp32", (1, 4))
