"""HMC on mixtures over lanes whose components lie together in one half and apart in the
other: tiles that find few near components, tiles that look in vain and wait, and
trajectories that pass from one to the other, over enough steps for every length of the
wait.  The oracle's decisions, states bit for bit, and weights."""
import numpy as np
import pytest
import torch

import oracle as orc
from parity_util import ORC_MOVE, compare_round, gpu_problem, oracle_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [30, 60, 100, 200])
@pytest.mark.parametrize("K", [5, 16])
@pytest.mark.parametrize("resample", [None, "sir", "fixed"])
def test_look_and_wait_match_oracle(d, K, resample):
    import paper_2408_12057_amd as oa
    assert torch.cuda.is_available()
    N, T, L = 67, 36, 3
    rng = np.random.default_rng(d * 100 + K)
    together = K - K // 3
    means = np.concatenate([0.02 * rng.standard_normal((together, d)),
                            2.0 * rng.standard_normal((K - together, d))])
    params = dict(means=means.astype(np.float32), log_scales=np.full(K, -1.2, np.float32))
    beta = np.linspace(0, 1, T + 1) ** 2
    eps = 0.3 / np.sqrt(1 + 10 * beta[1:]) * d ** -0.25
    flags = np.array([t % 5 == 0 for t in range(1, T + 1)], dtype=np.int32)
    kw = dict(resample_at=flags) if resample == "fixed" else {}
    trigger = {None: 0, "sir": 2, "fixed": 3}[resample]
    g = oa.asmc(gpu_problem(oa, "gmm", params, 4.0), N, beta, eps, 9, move="hmc", leapfrog=L, accept_bits=True,
                resample_=resample is not None, trigger=trigger, **kw)
    o = orc.asmc(oracle_problem("gmm", d, params, 4.0),
                 orc.Opts(move=ORC_MOVE["hmc"], leapfrog=L, resample=int(resample is not None), trigger=trigger,
                          nu=0.5, state_f32=1, **kw), N, beta, eps, 9, traces=True)
    compare_round(g, o, T, N)
