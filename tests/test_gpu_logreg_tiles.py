"""The gradient product's feature tiles (32, 16 and 4 features) at the edges of the
half-widths they are chosen by: ell and grad ell against binary64 within the fp32
bound, which covers every order of the sums, and a run of equal particles, whose
gradients must not depend on the lane that holds them."""
import numpy as np
import pytest
import torch

from paper_2408_12057_amd import workloads as wl
from test_gpu_logreg import _bounds

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [1, 8, 9, 16, 17, 24, 25, 31, 32, 33, 40, 41, 49, 50, 51, 64])
def test_gradient_tiles_at_their_edges(d):
    import paper_2408_12057_amd as oa
    n, N = 290, 131  # chunks and tiles with a remainder
    X, y, th_star = wl.logreg_data(n, d, 31 * d)
    theta = (th_star[None, :] + 0.3 * np.random.default_rng(d).normal(size=(N, d))).astype(np.float32)
    theta[64:128] = theta[70]
    ell, grad = oa.logreg_eval(oa.Problem.logreg(X, y), torch.tensor(theta, device="cuda"))
    ell, grad = ell.cpu().numpy(), grad.cpu().numpy()
    e_ref, g_ref, b_ell, b_g = _bounds(X, y, theta)
    assert np.all(np.abs(ell - e_ref) <= b_ell)
    assert np.all(np.abs(grad.astype(np.float64) - g_ref) <= b_g)
    assert np.array_equal(grad[64:128], np.broadcast_to(grad[70], (64, d)))
    assert np.all(ell[64:128] == ell[70])
