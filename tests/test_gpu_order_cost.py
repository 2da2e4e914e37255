"""The queue order the library builds by itself may not cost a short solve as much as
the solve: a tape with room for 256 steps around solves of five.  And the order at
the sizes where its kernels go round: keys beyond one round of the key kernel (131,072),
all in one bucket, none finite."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2609_28458_amd import api, inputs  # noqa: E402


def _order(n, cost):
    w = inputs.orbits_forward(1, seed=111)
    prob = api.make_problem("loghalo", "dopri5", np.repeat(w["y0"], n, axis=1), w["theta"], 0.0,
                            1.0, 1e-6, 1e-6)
    return api.Solution(prob, api.Launch()).queue_order(cost=torch.as_tensor(cost, device="cuda"))


@pytest.mark.parametrize("n", [1, 63, 64, 257, 131_071, 131_072, 131_073, 400_003])
@pytest.mark.parametrize("keys", ["spread", "equal", "few", "not finite"])
def test_order_is_a_permutation_longest_first(n, keys):
    rng = np.random.default_rng(n)
    cost = {"spread": rng.normal(size=n), "equal": np.full(n, 3.0),
            "few": rng.integers(0, 5, n).astype(float), "not finite": np.full(n, np.inf)}[keys]
    if keys == "spread" and n > 64:
        cost[[1, n - 1]] = [np.nan, -np.inf]
    o = _order(n, cost).cpu().numpy()
    assert np.array_equal(np.sort(o), np.arange(n))
    fin = np.isfinite(cost)
    assert np.all(fin[o[:fin.sum()]])  # the others come last
    k = cost[o[:fin.sum()]]
    if k.size:
        width = (k.max() - k.min()) / 65534
        assert np.all(np.diff(k) <= width * (1 + 1e-9))


def test_own_order_of_a_short_solve():
    n = 262_144
    w = inputs.orbits_forward(n, seed=112)
    prob = api.make_problem("loghalo", "dopri5", w["y0"], w["theta"], 0.0, 0.1, 1e-8, 1e-10)
    sols = [api.Solution(prob, api.Launch(ckpt_every=1, ckpt_capacity=258)) for _ in range(2)]
    sols[1].set_order(np.arange(n))
    ms = [[], []]
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    for rep in range(12):
        for s, t in zip(sols, ms):
            ev[0].record()
            for _ in range(5):
                s.run()
            ev[1].record()
            torch.cuda.synchronize()
            t.append(ev[0].elapsed_time(ev[1]) / 5)
    assert int(sols[0].n_accepted.max()) < 10
    # 2.5 times as long with one pair of atomics per wavefront on the key range
    assert min(ms[0]) < 2.0 * min(ms[1]), (min(ms[0]), min(ms[1]))
