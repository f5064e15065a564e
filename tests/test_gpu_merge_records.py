"""The per-step merge's two levels at the edges of its grid (a block takes 256 tiles, at
most 64 blocks): the records of all blocks reach the moments, the counts, the event and
the weights of the next step, every step, against the oracle."""
import numpy as np
import pytest
import torch

import oracle as orc
from parity_util import ORC_MOVE, compare_round, gpu_problem, oracle_problem
from paper_2408_12057_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [1021, 1024, 1025, 33 * 1024 + 3, 64 * 1024, 65600])
@pytest.mark.parametrize("trigger", ["ess", "sir"])
def test_merge_records_match_oracle(N, trigger):
    import paper_2408_12057_amd as oa
    assert torch.cuda.is_available()
    d, T = 100, 6  # 4 particles a tile
    params = wl.random_gauss(np.random.default_rng(N), d)
    beta = np.linspace(0, 1, T + 1) ** 2
    eps = np.full(T, 0.1)
    g = oa.asmc(gpu_problem(oa, "gauss", params, 1.5), N, beta, eps, 7, move="rwmh", resample_=True,
                trigger=trigger, accept_bits=True)
    o = orc.asmc(oracle_problem("gauss", d, params, 1.5),
                 orc.Opts(move=ORC_MOVE["rwmh"], resample=1, trigger={"ess": 0, "sir": 2}[trigger], nu=0.5,
                          state_f32=1), N, beta, eps, 7, traces=True)
    assert g["n_resample"] == o["n_resample"] > 0
    np.testing.assert_array_equal(g["resampled"], o["resampled"])
    np.testing.assert_allclose(g["ess"], o["ess"], rtol=1e-10)
    compare_round(g, o, T, N)
