"""A step without any error (an oscillator at rest) grows by alpha_max under every
controller: the Newton root at the edge of its range, and the PI form where the
previous norm's power vanishes, on single lanes, groups and tangent lanes."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from gpu_util import gpu_solve, oracle_solve, to_np  # noqa: E402
from paper_2609_28458_amd import api  # noqa: E402

NU = {"dopri5": 5, "tsit5": 5, "verner7": 7}
CTL = {"pi": dict(beta1=0.1, beta2=0.08),
       "vanishing": dict(beta1=0.1, beta2=100.0),
       "no beta1": dict(beta1=1e-320, beta2=0.1)}


def _edge(tab):  # the largest bound for which the kernels take the Newton root
    return dict(safety=0.9, alpha_max=0.9 * 10.0 ** (15.0 / NU[tab]))


@pytest.mark.parametrize("kind", ["pi", "vanishing", "no beta1", "edge"])
@pytest.mark.parametrize("tab", ["dopri5", "tsit5", "verner7"])
def test_step_without_error_grows_by_the_upper_bound(orc, tab, kind):
    n = 5
    ctl = {"h0": 1e-3, **(_edge(tab) if kind == "edge" else CTL[kind])}
    # The span ends where so many steps, each alpha_max times the one before,
    # reach to the last bit: a factor one bit smaller takes a step more.
    steps, t1, h = 4, 0.0, ctl["h0"]
    for _ in range(steps):
        t1, h = t1 + h, h * ctl.get("alpha_max", 5.0)
    w = dict(rhs="harmonic", tableau=tab, t0=0.0, t1=t1, rtol=1e-6, atol=1e-9, t_out=None,
             y0=np.zeros((2, n)), theta=np.linspace(0.5, 2.0, n)[None, :])
    o = oracle_solve(orc, w, **ctl)
    assert np.all(o["status"] == 0) and np.all(o["n_accepted"] == steps)
    prob = api.make_problem(w["rhs"], tab, w["y0"], w["theta"], 0.0, t1, 1e-6, 1e-9)
    got = {"one lane": gpu_solve(w, api.Launch(schedule="static", **ctl)),
           "groups": gpu_solve(w, api.Launch(wide=n, **ctl)),
           "tangent lanes": api.solve_sens(prob, [0, 2], api.Launch(**ctl))[0]}
    torch.cuda.synchronize()
    for name, sol in got.items():
        g = to_np(sol)
        for k in ("status", "n_accepted", "n_rejected"):
            np.testing.assert_array_equal(g[k], o[k], err_msg=f"{name} {k}")
        assert np.all(g["y_final"] == 0.0)
