"""The observables of a batch of more cavities than a launch grid's y index takes: every cavity's own
temperature, speed and step come back, on both sides of each launch's last cavity."""
import numpy as np
import pytest

from paper_1308_2071_amd import Batch, Cavity, make_params, params_dict
from paper_1308_2071_amd._abi import LbmParams

pytestmark = pytest.mark.gpu


def test_observables_of_seventy_thousand_cavities():
    n = 70000
    base = make_params(nx=2, ny=2, bc=(2, 2, 2, 2), dtype="fp32", tau_v=0.8, tau_T=0.9,
                       gbeta=0.0, ext_accel=(1e-4, 0.0))
    params = []
    for i in range(n):
        p = LbmParams.from_buffer_copy(base)
        p.T_init = 0.25 + i * 2.0 ** -18     # exact in FP32
        params.append(p)
    b = Batch(params, [0.5] * n)
    s, obs = b.step(1).observables()
    assert s == 0 and len(obs) == n
    T = np.array([(o["T_min"], o["T_max"]) for o in obs])
    want = 0.25 + np.arange(n) * 2.0 ** -18
    # a uniform temperature: five weighted parts summed, a few roundings of it
    assert np.abs(T - want[:, None]).max() <= 8 * 2.0 ** -24
    assert len({o["step"] for o in obs}) == 1
    for i in (0, 32767, 32768, 65535, 65536, n - 1):
        c = Cavity(dict(params_dict(params[i])), phi_uniform=0.5)
        r = c.step(1).observables(fields=False)
        assert r["max_speed"] > 0
        for k in ("max_speed", "T_min", "T_max", "phip_dev", "step"):
            assert obs[i][k] == r[k], (i, k)
        c.close()
    b.close()
