"""HMC on a mixture whose squared distances pass the largest binary32 number while the
components' weights stay comparable: every component with weight enters ell and its
gradient (the oracle's decisions, states bit for bit, and weights)."""
import numpy as np
import pytest
import torch

import oracle as orc
from parity_util import ORC_MOVE, compare_round, gpu_problem, oracle_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [30, 60, 100, 200])
def test_distances_beyond_binary32(d):
    import paper_2408_12057_amd as oa
    assert torch.cuda.is_available()
    N, T, K = 67, 4, 6
    # two components at 3.2e38 (finite in binary32), four at 3.6e38 (not), 1 / (2 v) =
    # 1.25e-37: exponents -40 and -45, far from where exp gives zero
    r2 = np.array([3.2e38] * 2 + [3.6e38] * 4)
    signs = np.where(np.random.default_rng(d).random((K, d)) < 0.5, -1.0, 1.0)
    params = dict(means=(signs * np.sqrt(r2 / d)[:, None]).astype(np.float32),
                  log_scales=np.full(K, 0.5 * np.log(4e36), np.float32))
    ref = 1e30
    beta = np.linspace(0, 1, T + 1) ** 2
    eps = np.full(T, 0.3e15 * d ** -0.25)
    g = oa.asmc(gpu_problem(oa, "gmm", params, ref), N, beta, eps, 9, move="hmc", leapfrog=3, accept_bits=True)
    o = orc.asmc(oracle_problem("gmm", d, params, ref),
                 orc.Opts(move=ORC_MOVE["hmc"], leapfrog=3, state_f32=1), N, beta, eps, 9, traces=True)
    compare_round(g, o, T, N)
