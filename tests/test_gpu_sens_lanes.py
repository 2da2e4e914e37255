"""The two mappings of a sensitivity solve agree bit for bit: dual numbers in
one lane (large ensembles) and tangent lanes, one vector per lane (small
ensembles, the head of the order with `wide`, and pairs whose dual numbers do
not fit the registers).  Both compute every value and tangent with the same
operations in the same order, so no tolerance is involved."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2609_28458_amd import api, inputs  # noqa: E402

# beyond the rule's line for up to 9 columns (12 lanes each, 5 launches of 1.5
# wavefronts on each of 1,024 SIMDs: 40,960)
LARGE, SMALL = 41_001, 157


def _workload(rhs, n):
    if rhs == "quint":
        return inputs.quintessence(n, seed=41)
    rng = np.random.default_rng(41)
    w = inputs.orbits_forward(n, seed=41)
    if rhs == "harmonic":
        w.update(rhs=rhs, y0=rng.normal(size=(2, n)), theta=rng.uniform(0.5, 2.0, (1, n)))
    elif rhs == "kepler":
        w.update(rhs=rhs, y0=np.stack([rng.uniform(0.8, 1.2, n), np.zeros(n), np.zeros(n),
                                       rng.uniform(0.7, 1.1, n)]), theta=np.array([1.0]))
    w.update(rtol=1e-6, atol=1e-8, t1=3.0, t_out=np.array([0.0, 0.4, 0.41, 1.7, 3.0]))
    return w


def _solve(w, n, cols, launch):
    th = w["theta"] if np.ndim(w["theta"]) == 1 else w["theta"][:, :n]
    p = api.make_problem(w["rhs"], w["tableau"], w["y0"][:, :n], th, w["t0"], w["t1"], w["rtol"],
                         w["atol"], w["t_out"])
    sol, Sf, So = api.solve_sens(p, cols, launch)
    torch.cuda.synchronize()
    y_out = sol.y_out
    if y_out is not None and launch.out_layout == "knd":
        y_out = y_out.permute(2, 0, 1)
    out = [sol.y_final, sol.n_accepted, sol.n_rejected, sol.status, Sf] + (
        [] if So is None else [y_out, So])
    return [t[..., :SMALL].cpu().numpy() for t in out]


@pytest.mark.parametrize("M", [1, 2, 3, 9])
@pytest.mark.parametrize("nodes", [False, True])
@pytest.mark.parametrize("rhs,tab", [("harmonic", "dopri5"), ("kepler", "verner7"),
                                     ("loghalo", "tsit5"), ("loghalo", "verner7"),
                                     ("quint", "dopri5")])
def test_mappings_agree_bitwise(rhs, tab, nodes, M):
    api.lib()
    w = {**_workload(rhs, LARGE), "tableau": tab}
    if not nodes:
        w["t_out"] = None
    ncol = api.DIM[api.RHS[rhs]] + api.NPARAM[api.RHS[rhs]]
    cols = [(3 * m + 1) % ncol for m in range(M)]
    layout = "knd" if M == 2 else "dkn"
    few = _solve(w, SMALL, cols, api.Launch(out_layout=layout))
    assert np.all(few[3] == 0)
    for wide in (0, 70):  # one lane each; the head of the order on tangent lanes
        many = _solve(w, LARGE, cols, api.Launch(out_layout=layout, wide=wide))
        for a, b in zip(many, few):
            np.testing.assert_array_equal(a, b)
