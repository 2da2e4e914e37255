"""The Gauss-Newton kernel of gs_de_profile holds a fit on eight lanes: fits at
the ends of wavefronts and workgroups (8 fits to a wavefront, 32 to a workgroup),
and node and data counts that leave lanes without one, against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2609_28458_amd import api  # noqa: E402
from test_gpu_de import _oracle, _run_gpu, _setup  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    api.lib()


@pytest.mark.parametrize("n,nodes,data_points", [
    (1, 1, 0), (7, 9, 0), (8, 4, 8), (9, 5, 9), (31, 7, 3), (32, 16, 7), (33, 17, 16), (65, 8, 1)])
def test_fits_at_the_edges(orc, n, nodes, data_points):
    from oracle import de_profile as de
    w, s, lam, om, h, a0, _, _ = _setup(de, 1, n)
    w["nodes"] = np.linspace(-1.2, -0.1, nodes)
    w["N_data"] = np.linspace(-1.15, -0.15, data_points) if data_points else None
    w["iters"] = 2
    f, orad = w["fid"], w["omega_r"]
    lam1, om1 = np.array([f["lam"]]), np.array([f["om"]])
    a0f = de.flat_amplitude(1.0 - om1 - orad, lam1, om1, orad, s, 4)
    Dfid = de.at_data(de.model(a0f, lam1, om1, np.array([f["h"]]), orad, w["nodes"], s)[0],
                      w["nodes"], w["N_data"])[:, :, 0]
    eps = np.random.default_rng(n).normal(size=Dfid.shape + (n,))
    data = Dfid[:, :, None] * (1.0 + w["rel_noise"] * eps)
    sigma = w["rel_noise"] * Dfid
    g = _run_gpu(w, lam, om, h, a0, data, sigma)
    o = _oracle(de, w, s, lam, om, h, a0, data, sigma)
    assert np.all(g["status"] == 0)
    for k, ko in (("omega_m", "om"), ("h", "h"), ("a0", "a0"), ("dist", "dist")):
        np.testing.assert_allclose(g[k], o[ko], rtol=1e-9, err_msg=k)
    np.testing.assert_allclose(g["chi2"], o["chi2"], rtol=1e-7, atol=1e-9)
    # A fit does not depend on its neighbours.
    one = _run_gpu(w, lam[-1:], om[-1:], h[-1:], a0[-1:], data[:, :, -1:], sigma)
    for k in ("omega_m", "h", "a0", "chi2", "chi2_prev", "decrement"):
        np.testing.assert_array_equal(one[k][0], g[k][-1], err_msg=k)
