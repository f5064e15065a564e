"""The merges of the slots' moments at the edges of their workgroup (64 slots a wave, 8
waves): any number of slots gives the moments of one slot, for a plain pass and for
segments between fixed resampling times.

The sums have N positive terms in binary64 in another order: N u = 1.5e-11 relative,
so that much in their logarithms; the particles themselves do not depend on the slots."""
import numpy as np
import pytest
import torch

from parity_util import gpu_problem
from paper_2408_12057_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("slots", [2, 63, 64, 65, 511, 512, 513, 1025, 2048])
@pytest.mark.parametrize("segments", [False, True])
def test_slots_do_not_change_the_moments(slots, segments):
    import paper_2408_12057_amd as oa
    N, T = 2048 * 64, 4
    p = gpu_problem(oa, "gauss", wl.random_gauss(np.random.default_rng(1), 2), 1.0)
    beta = np.linspace(0, 1, T + 1) ** 2
    kw = dict(resample_=True, trigger="fixed", resample_at=[0, 1, 0, 0]) if segments else {}
    a, b = (oa.asmc(p, N, beta, 0.3, 5, move="rwmh", slots=s, **kw) for s in (1, slots))
    np.testing.assert_allclose(b["log_g"], a["log_g"], rtol=0, atol=2e-11)
    assert np.array_equal(b["accept"], a["accept"])
    assert abs(b["logZ"] - a["logZ"]) < 4e-11
    assert torch.equal(b["x"], a["x"])
