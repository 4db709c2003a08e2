"""lbm_step_shape's work-groups per launch of the one-step forms: rows of 256 nodes, and in the AA
layout tiles of 128 x 2 up to a state of 256 MiB."""
import pytest

from paper_1308_2071_amd import Cavity, lbm_step_shape, workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,dtype,groups", [(300, 200, "fp32", 3 * 100), (257, 33, "fp64", 3 * 17),
                                                (1500, 1300, "fp64", 12 * 650),
                                                (2500, 2500, "fp32", 10 * 2500),
                                                (2000, 1500, "fp64", 8 * 1500)])
def test_aa_layout(nx, ny, dtype, groups):
    c = Cavity(dict(workloads.cavity(nx, ny, Ra=1e5, Pr=0.71, dtype=dtype), layout="aa"),
               phi_uniform=0.5)
    assert lbm_step_shape(c.ctx) == (1, 1, 0, groups)
    c.close()


def test_pull_layout():
    c = Cavity(dict(workloads.cavity(300, 200, Ra=1e5, Pr=0.71), steps_per_launch=1),
               phi_uniform=0.5)
    assert lbm_step_shape(c.ctx) == (1, 0, 0, 2 * 200)
    c.close()
