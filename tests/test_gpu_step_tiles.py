"""The per-step path with more tiles than one grid of resident blocks holds, gradient
moves: blocks that walk over several tiles, accepted and rejected proposals, states from
the gathered copies after an event at every step and in place, a ragged last tile,
against the oracle."""
import numpy as np
import pytest
import torch

import oracle as orc
from parity_util import ORC_MOVE, compare_round, gpu_problem, oracle_problem
from paper_2408_12057_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("family,d,move,N", [("gmm", 100, "hmc", 20011), ("gmm", 100, "mala", 20011),
                                             ("gmm", 60, "hmc", 70001), ("gauss", 10, "mala", 300007)])
@pytest.mark.parametrize("trigger", ["sir", "ess"])
def test_more_tiles_than_blocks(family, d, move, N, trigger):
    import paper_2408_12057_amd as oa
    assert torch.cuda.is_available()
    T = 3
    rng = np.random.default_rng(d)
    params = wl.random_gauss(rng, d) if family == "gauss" else wl.random_gmm(rng, d, 2)
    beta = np.linspace(0, 1, T + 1) ** 2
    eps = np.full(T, 3.2 * d ** -0.25)  # proposals are rejected too
    g = oa.asmc(gpu_problem(oa, family, params, 1.5), N, beta, eps, 9, move=move, leapfrog=2, accept_bits=True,
                resample_=True, trigger=trigger)
    o = orc.asmc(oracle_problem(family, d, params, 1.5),
                 orc.Opts(move=ORC_MOVE[move], leapfrog=2, resample=1, trigger={"ess": 0, "sir": 2}[trigger],
                          nu=0.5, state_f32=1), N, beta, eps, 9, traces=True)
    assert 0.02 < o["acc"].min() and o["acc"][0] < 0.7
    compare_round(g, o, T, N)
