"""Three and four steps per launch of a batch (tiles of 28 x 12, 28 x 28 and 16 x 16 nodes), which
the tuner tries on batches of half a million nodes and more, and the untuned default there: every
cavity bitwise its own run one step per launch, through a graph replay and a remainder of single
steps; and a cache line whose tile the library does not have is tuned again."""
import pytest
import torch

from paper_1308_2071_amd import Batch, Cavity, workloads

pytestmark = pytest.mark.gpu

FIELDS = ("ux", "uy", "p", "T")
SIZES = [(29, 57), (28, 12), (85, 17), (5, 6), (700, 721)]   # the last makes it a large batch


def batch(dtype):
    ps = [workloads.cavity(nx, ny, Ra=3e4 + 10 * nx, Pr=0.71, Da=1e-2, dtype=dtype, tau_v=0.8,
                           tau_T=0.9, gbeta=1e-4) for nx, ny in SIZES]
    return ps, [0.4 + 0.1 * i for i in range(len(ps))]


def check(b, params, phis, steps, what):
    b.step(steps)
    for i, (p, phi) in enumerate(zip(params, phis)):
        c = Cavity(dict(p, steps_per_launch=1), phi_uniform=phi)
        o = c.step(steps).observables()
        f = b.fields(i)
        for k in FIELDS:
            assert torch.equal(f[k], o[k]), (what, i, k)
        c.close()


@pytest.mark.parametrize("dtype", ["fp32", "fp64", "fp32_f64"])
def test_three_and_four_steps_equal_standalone_runs(dtype, tmp_path):
    params, phis = batch(dtype)
    path = tmp_path / "tune.txt"
    Batch(params, phis, tune_cache_path=str(path)).close()
    line = path.read_text().split()
    for rows, steps in ((12, 3), (28, 3), (16, 4)):
        path.write_text(" ".join(line[:4] + [str(rows), "3"]) + "\n")
        b = Batch(params, phis, tune_cache_path=str(path))
        assert b.shape()[4] == steps and b.shape()[5] == rows
        check(b, params, phis, 59, (dtype, rows))
        b.close()
    path.write_text(" ".join(line[:4] + ["7", "1"]) + "\n")   # no such tile
    b = Batch(params, phis, tune_cache_path=str(path))
    assert len(path.read_text().splitlines()) == 2
    check(b, params, phis, 5, dtype)
    b.close()


@pytest.mark.parametrize("dtype", ["fp32", "fp64"])
def test_untuned_large_batch(dtype):
    params, phis = batch(dtype)
    b = Batch(params, phis)
    assert b.shape()[4] == 3 and b.shape()[5] == 12
    check(b, params, phis, 53, dtype)
    b.close()
    small = Batch(params[:4], phis[:4])
    assert small.shape()[4] == 2
    check(small, params[:4], phis[:4], 51, dtype)
    small.close()
