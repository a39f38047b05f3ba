"""The small exponential exp(T - theta I) e1 where its kernel can go wrong (orders around the eight steps of a
rescaling and the 64 lanes, widths from none to 1e6), against the eigendecomposition; and the single-kernel solve
around its row and vector groups, with the basis in LDS and not, against the schedule of one launch per phase."""
import numpy as np
import pytest
import scipy.linalg as sla

from tests import graphs_small as gs
from tests.test_gpu_parity import DenseBatch
from tests.test_gpu_single import api, assert_same, outputs, torch_mod, weighted

pytestmark = pytest.mark.gpu
EPS = 2.0 ** -52


@pytest.mark.parametrize("shift", [True, False])
@pytest.mark.parametrize("width", [1e-13, 1e-6, 0.3, 4.0, 60.0, 1e3, 1e6])
@pytest.mark.parametrize("k", [1, 2, 8, 9, 10, 16, 17, 63, 64, 65, 66, 128])
def test_expv(gpu_lib, k, width, shift):
    torch = torch_mod()
    if not shift and width > 60.0:
        pytest.skip("exp of the largest eigenvalue overflows the comparison")
    rng = np.random.default_rng(k)
    a = rng.uniform(-0.25, 0.25, size=(3, k)) * width
    b = rng.uniform(0.01, 0.25, size=(3, k)) * width
    b[1, k // 2:] *= 1e-9  # nearly decoupled
    a[2] = 0.1 * width      # constant diagonal, nearly equal couplings
    b[2] = 0.2 * width
    y, th = api().tridiag_expv(torch.tensor(a, device="cuda"), torch.tensor(b, device="cuda"), shift)
    y, th = y.cpu().numpy(), th.cpu().numpy()
    for i in range(3):
        lam, Q = sla.eigh(np.diag(a[i]) + np.diag(b[i][:k - 1], 1) + np.diag(b[i][:k - 1], -1))
        theta = lam[-1] if shift else 0.0
        # both sides: eigenvalues to a few units of the norm (at most the width) per order, exp to as much
        # absolutely, and the rounding of sqrt(84 d) + 12 terms
        assert abs(th[i] - theta) <= 4 * (8 + k) * EPS * width
        want = Q @ (np.exp(lam - theta) * Q[0])
        tol = EPS * (8 * (8 + k) * width + 16 * (np.sqrt(84 * width) + 12)) * (1.0 if shift else np.exp(max(lam[-1], 0)))
        assert np.abs(y[i] - want).max() <= tol


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("n", [2, 255, 256, 257, 1023, 1025, 2047, 2048])
def test_single_solve_row_groups(gpu_lib, n, dtype):
    hb = weighted(DenseBatch([[gs.random_graph(n, min(1.0, 6.0 / n), 1), gs.random_graph(n, min(1.0, 12.0 / n), 2)]],
                             dtype), 3)
    b = api().Batch.from_host(hb)
    for kw in (dict(m=9), dict(m=17), dict(m=33), dict(m=0, tol=1e-7, m_max=40)):
        assert_same(outputs(b, schedule="single", **kw), outputs(b, schedule="batched", hipgraph=False, **kw))
