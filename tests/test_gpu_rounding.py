"""recip, quotient and root of lbm_device.hpp, which Eqs. (21) and (5) and the adjoint use in place of
the compiler's division and square root: correctly rounded over the whole FP32 range the step can reach
and at random FP64 operands (tests/native/arith.hip counts the differences), and the velocity of Eq.
(21) at every node of a state at rest against extended precision, without an absolute floor."""
import ctypes
import os

import numpy as np
import pytest
import torch

from paper_1308_2071_amd import Cavity, lbm_derived, make_params
from paper_1308_2071_amd.build import compile_shared

pytestmark = pytest.mark.gpu
NATIVE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "native")
ERGUN = np.longdouble(7) / 4 / np.sqrt(np.longdouble(150))


def test_rounding_of_reciprocals_quotients_and_roots():
    path = os.path.join(NATIVE, "libarith.so")
    if not os.path.exists(path):
        compile_shared([os.path.join(NATIVE, "arith.hip")], path)
    torch.cuda.init()
    counts = (ctypes.c_ulonglong * 10)()
    assert ctypes.CDLL(path).arith_check(counts, 256) == 0      # 2^26 random operands
    names = ("recip f32", "root f32", "reciprocal f32", "quotient f32", "quotient f64", "root f64",
             "reciprocal f64", "root f64 below 2^-970", "special f32", "special f64")
    assert {n: c for n, c in zip(names, counts) if c} == {}


@pytest.mark.parametrize("dtype", ["fp32", "fp64", "fp32_f64"])
@pytest.mark.parametrize("accel", [1e-29, 1e-12, 1e-4, 3e-2])
@pytest.mark.parametrize("forchheimer", [0, 1])
def test_velocity_at_rest_node_by_node(accel, dtype, forchheimer):
    """A state at rest has j = 0, so v of Eq. (22) is phi G / 2 and u of Eq. (21) follows from phi, K
    and G alone.  In units e of one rounding (2^-24, FP64 2^-53), with the hardware's square roots at
    2 e: G 1 and v 2; 1/sqrt(K) 2, c_lin 8, l0 9; c_nl 7, |v| 5, l1 |v| 13; the root's argument 19,
    the root 10.5, the denominator 11.5; u 14.5.  FP32 storage of an FP64 result adds one rounding."""
    ny, nx = 24, 40
    rng = np.random.default_rng(5)
    f32 = dtype != "fp64"
    phi = rng.uniform(0.01, 1.0, (ny, nx))
    K = 10.0 ** rng.uniform(-5, 6, (ny, nx))
    if f32:
        phi, K = phi.astype(np.float32).astype(float), K.astype(np.float32).astype(float)
    p = make_params(nx=nx, ny=ny, bc=(2, 2, 2, 2), dtype=dtype, tau_v=0.8, tau_T=0.9, gbeta=0.0,
                    ext_accel=(accel, -0.5 * accel), T_init=0.5, forchheimer=forchheimer)
    tdt = torch.float32 if f32 else torch.float64
    c = Cavity(p, phi=torch.tensor(phi, dtype=tdt), K=torch.tensor(K, dtype=tdt))
    o = c.observables()
    e = 2.0 ** -24 if dtype == "fp32" else 2.0 ** -53
    tol = 16 * e + (2.0 ** -24 if f32 else 0.0)
    phi, K = phi.astype(np.longdouble), K.astype(np.longdouble)
    nu = np.longdouble(lbm_derived(p)["nu"])
    vx, vy = phi * accel / 2, -phi * accel / 4
    l0 = 0.5 + phi * nu / K / 4
    l1 = ERGUN / np.sqrt(phi * K) / 2 * forchheimer
    den = l0 + np.sqrt(l0 * l0 + l1 * np.sqrt(vx * vx + vy * vy))
    for k, v in (("ux", vx), ("uy", vy)):
        want = v / den
        assert np.abs(want).min() > 2.0 ** -120       # normal in FP32
        got = o[k].double().cpu().numpy()
        assert (np.abs(got - want) <= tol * np.abs(want)).all(), (k, np.abs(got / want - 1).max())
    c.close()
