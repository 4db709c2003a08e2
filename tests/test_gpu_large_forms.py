"""Forms of the step and of the adjoint's recompute and sweep that the default takes, each against one
step per launch or against checkpoints every other step (segments too short for any other form),
bitwise: three steps per launch on states of 2 GiB and more, eight, four and two steps recomputed per
launch, and the backward tiles with a uniform medium beyond 256 tiles and on an axis periodic along
x."""
import pytest
import torch

from paper_1308_2071_amd import Cavity, lbm_step_shape, workloads

pytestmark = pytest.mark.gpu

CAV = dict(bc=(0, 0, 1, 1), T_wall=(1.0, 0.0, 0.0, 0.0))
CHX = dict(bc=(2, 2, 0, 1), T_wall=(0.0, 0.0, 1.0, 0.0), ext_accel=(2e-5, 0.0))
GROUPS = dict(tau_v=0.7, tau_T=0.8, gbeta=1e-3)


@pytest.mark.parametrize("n,dtype", [(8192, "fp32"), (9000, "fp64")])
def test_three_steps_on_states_beyond_2_gib(n, dtype):
    """3.8 GB, and 9.1 GB, whose halves are beyond 2 GiB too; five steps: three, then two."""
    fields = []
    for spl in (1, 0):
        c = Cavity(dict(CAV, **GROUPS, nx=n, ny=n, dtype=dtype, steps_per_launch=spl),
                   phi_uniform=0.55)
        assert lbm_step_shape(c.ctx)[0] == (1 if spl else 3)
        o = c.step(5).observables()
        fields.append([o[k].cpu() for k in ("ux", "uy", "p", "T")])
        c.close()
        del c, o
    for a, b in zip(*fields):
        assert torch.equal(a, b)


def gradient(params, dtype, every, steps, medium):
    nx, ny = params["nx"], params["ny"]
    tdt = torch.float64 if dtype == "fp64" else torch.float32
    kw = dict(phi_uniform=0.55)
    if medium:
        phi, K = workloads.random_medium(ny, nx, seed=nx + 3 * ny)
        kw = dict(phi=torch.tensor(phi, dtype=tdt), K=torch.tensor(K, dtype=tdt))
    c = Cavity(dict(params, **GROUPS, dtype=dtype, checkpoint_every=every), nsteps_max=steps, **kw)
    out = c.step(steps).grad()
    c.close()
    return out


def compare(params, dtype, every, steps, medium):
    want = gradient(params, dtype, 2, steps, medium)
    got = gradient(params, dtype, every, steps, medium)
    for a, b, k in zip(want, got, ("phi", "K")):
        assert torch.isfinite(a).all() and a.abs().max() > 0, k
        assert torch.equal(a, b), (params, dtype, every, k)


@pytest.mark.parametrize("dtype", ["fp32", "fp64", "fp32_f64"])
@pytest.mark.parametrize("medium", [False, True])
@pytest.mark.parametrize("shape", [(128, 128), (61, 47), (9, 130)])
@pytest.mark.parametrize("every", [9, 11, 18])
def test_eight_steps_recomputed(every, shape, medium, dtype):
    compare(dict(CAV, nx=shape[0], ny=shape[1]), dtype, every, 2 * every + 3, medium)


@pytest.mark.parametrize("dtype,shape", [("fp32", (300, 257)), ("fp64", (257, 250)),
                                         ("fp32_f64", (300, 257))])
@pytest.mark.parametrize("medium", [False, True])
@pytest.mark.parametrize("every", [9, 40, 41, 43])
def test_four_or_two_steps_recomputed(every, medium, dtype, shape):
    """With FP64 arithmetic segments of up to 40 steps go in pairs, longer ones in fours."""
    compare(dict(CAV, nx=shape[0], ny=shape[1]), dtype, every, every + 7, medium)


@pytest.mark.parametrize("dtype,shape", [("fp32", (330, 329)), ("fp64", (255, 250))])
def test_backward_tiles_with_a_uniform_medium(dtype, shape):
    compare(dict(CAV, nx=shape[0], ny=shape[1]), dtype, 7, 17, False)


@pytest.mark.parametrize("dtype", ["fp32", "fp64"])
@pytest.mark.parametrize("shape", [(5, 6), (16, 17), (17, 33), (31, 15), (50, 5), (330, 300)])
def test_backward_tiles_periodic_along_x(shape, dtype):
    compare(dict(CHX, nx=shape[0], ny=shape[1]), dtype, 8, 21, True)
