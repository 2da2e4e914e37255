"""Fits beyond one launch of the Gauss-Newton kernel (2^24), and beyond the count
at which eight lanes to a fit pass the 2^32 lanes of any launch (2^29): every fit
of a small ensemble, repeated, gets the bits it gets in the small ensemble."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2609_28458_amd import api  # noqa: E402

OUT = ("omega_m", "h", "a0", "chi2", "chi2_prev", "decrement", "dist", "status")


@pytest.mark.parametrize("n,iters", [(2 ** 24 + 9, 1), (2 ** 29 + 9, 0)])
def test_many_fits(n, iters):
    api.lib()
    if torch.cuda.mem_get_info()[1] < (16 << 30) + 350 * n:
        pytest.skip("the arrays do not fit this device")
    torch.cuda.empty_cache()
    m = 8  # different fits
    lam = np.linspace(0.2, 0.9, m)
    om = np.linspace(0.28, 0.32, m)
    data = np.stack([np.linspace(0.25, 0.3, m), np.linspace(0.8, 0.9, m)])[:, None, :]

    def run(size):
        rep = -(-size // m)

        def cut(x):
            return torch.as_tensor(x, device="cuda").repeat(*[1] * (x.ndim - 1), rep)[..., :size]

        return api.de_profile(cut(lam), cut(om), cut(np.full(m, 1.0)), cut(1.0 - om), 9e-5,
                              np.array([-0.3]), cut(data), np.array([[0.003], [0.009]]),
                              iters=iters, newton=0, rtol=1e-2, atol=1e-4)

    small, many = run(m), run(n)
    torch.cuda.synchronize()
    assert bool((small["status"] == 0).all())
    for k in OUT[:4] + OUT[6:] if iters == 0 else OUT:
        rows_s, rows_m = small[k].reshape(-1, m), many[k].reshape(-1, n)
        for s, r in zip(rows_s, rows_m):
            assert torch.equal(r[:n - n % m].view(-1, m), s.expand(n // m, m)), k
            assert torch.equal(r[n - n % m:], s[:n % m]), k
