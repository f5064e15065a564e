"""HMC on mixtures in the layouts of 2 lanes of 16 and 4 lanes of 8 coordinates, which
many particles of 9 to 32 coordinates take: components far apart, in between and close
together, the last tile ragged.  The oracle's decisions, states bit for bit, and
weights."""
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
    m.autotune(-1)  # the rule's shapes
    return m


@pytest.mark.parametrize("d,N,layout", [(25, 65536 + 33, (2, 16)), (32, 65536 + 1, (2, 16)),
                                        (9, 8193, (4, 8)), (30, 8200, (4, 8))])
@pytest.mark.parametrize("K", [2, 5, 16])
@pytest.mark.parametrize("spread", [4.0, 0.7, 0.05])
def test_layout_matches_oracle(oa, d, N, layout, K, spread):
    T, L = 2, 2
    rng = np.random.default_rng(d * 100 + K)
    params = dict(means=(spread * rng.standard_normal((K, d))).astype(np.float32),
                  log_scales=rng.uniform(-1.2, -0.9, K).astype(np.float32))
    p = gpu_problem(oa, "gmm", params, 4.0)
    assert oa.shape(p, N, move="hmc", leapfrog=L) == layout
    beta = np.linspace(0, 1, T + 1) ** 2
    eps = 0.3 / np.sqrt(1 + 10 * beta[1:]) * d ** -0.25
    g = oa.asmc(p, N, beta, eps, 9, move="hmc", leapfrog=L, accept_bits=True)
    o = orc.asmc(oracle_problem("gmm", d, params, 4.0),
                 orc.Opts(move=ORC_MOVE["hmc"], leapfrog=L, state_f32=1), N, beta, eps, 9, traces=True)
    compare_round(g, o, T, N)
