"""What three and four steps per launch of a batch leave goes in a launch of two steps on the same
tiles: every cavity bitwise its own run one step per launch, for each of the three tiles, and
lbm_batch_step(2) no slower than in a batch that takes two steps per launch throughout (two single
steps took 1.6 times as long in FP64)."""
import pytest
import torch

from paper_1308_2071_amd import Batch, Cavity, workloads

pytestmark = pytest.mark.gpu

SIZES = [(29, 57), (28, 12), (85, 17), (5, 6), (33, 29), (700, 721)]


def batch(dtype, **kw):
    ps = [workloads.cavity(nx, ny, Ra=3e4 + 10 * nx, Pr=0.71, Da=1e-2, dtype=dtype, tau_v=0.8,
                           tau_T=0.9, gbeta=1e-4, **kw) for nx, ny in SIZES]
    return ps, [0.4 + 0.1 * i for i in range(len(ps))]


@pytest.mark.parametrize("dtype", ["fp32", "fp64", "fp32_f64"])
def test_remainders_equal_standalone_runs(dtype, tmp_path):
    params, phis = batch(dtype)
    path = tmp_path / "tune.txt"
    Batch(params, phis, tune_cache_path=str(path)).close()
    line = path.read_text().split()
    calls = (2, 5, 7, 50)
    want = []
    for p, phi in zip(params, phis):
        c = Cavity(dict(p, steps_per_launch=1), phi_uniform=phi)
        want.append([c.step(n).observables() for n in calls])
        c.close()
    for rows, steps in ((12, 3), (28, 3), (16, 4)):
        path.write_text(" ".join(line[:4] + [str(rows), "3"]) + "\n")
        b = Batch(params, phis, tune_cache_path=str(path))
        assert b.shape()[4] == steps and b.shape()[5] == rows
        for j, n in enumerate(calls):
            b.step(n)
            for i, w in enumerate(want):
                f = b.fields(i)
                for k in ("ux", "uy", "p", "T"):
                    assert torch.equal(f[k], w[j][k]), (dtype, rows, n, i, k)
        b.close()


def test_two_steps_take_one_launch():
    def best(b):
        e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        times = []
        for _ in range(8):
            e[0].record()
            for _ in range(40):
                b.step(2)
            e[1].record()
            e[1].synchronize()
            times.append(e[0].elapsed_time(e[1]))
        return min(times[2:])
    ps = [workloads.cavity(n, n - 90, Ra=1e5, Pr=0.71, Da=1e-2, dtype="fp64") for n in (900, 1100)]
    a = Batch(ps, [0.5, 0.6])
    b = Batch([dict(p, steps_per_launch=2) for p in ps], [0.5, 0.6])
    assert a.shape()[4] == 3 and b.shape()[4] == 2
    assert best(a) < 1.25 * best(b)
    a.close()
    b.close()
