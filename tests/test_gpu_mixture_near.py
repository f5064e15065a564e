"""HMC on mixtures over 2 to 16 lanes a particle with components far apart (one
matters at a time), close together (all matter) and in between, up to the most
components, ragged particle counts and dimensions that do and do not fill their
quads: the oracle's decisions, states bit for bit, and weights."""
import numpy as np
import pytest
import torch

import oracle as orc
from parity_util import ORC_MOVE, compare_round, gpu_problem, oracle_problem

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def oa():
    import paper_2408_12057_amd as m
    assert torch.cuda.is_available()
    return m


@pytest.mark.parametrize("d", [9, 30, 33, 60, 100, 129, 200])
@pytest.mark.parametrize("K", [1, 2, 5, 16])
@pytest.mark.parametrize("spread,resample", [(4.0, False), (0.7, True), (0.05, False)])
def test_hmc_matches_oracle(oa, d, K, spread, resample):
    N, T = 67, 5
    rng = np.random.default_rng(d * 100 + K)
    params = dict(means=(spread * rng.standard_normal((K, d))).astype(np.float32),
                  log_scales=rng.uniform(-1.2, -0.9, K).astype(np.float32))
    beta = np.linspace(0, 1, T + 1) ** 2
    eps = 0.3 / np.sqrt(1 + 10 * beta[1:]) * d ** -0.25
    g = oa.asmc(gpu_problem(oa, "gmm", params, 4.0), N, beta, eps, 9, move="hmc", leapfrog=4, accept_bits=True,
                resample_=resample, trigger="sir" if resample else "ess")
    o = orc.asmc(oracle_problem("gmm", d, params, 4.0),
                 orc.Opts(move=ORC_MOVE["hmc"], leapfrog=4, resample=int(resample), trigger=2, nu=0.5, state_f32=1),
                 N, beta, eps, 9, traces=True)
    compare_round(g, o, T, N)
