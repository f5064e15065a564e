"""The kernels at their largest LDS (16 components at d = 256: 69 KB of parameters for
HMC, 52 KB otherwise): sweeps, segments, the per-step path, tempering, against the oracle."""
import numpy as np
import pytest
import torch

import oracle as orc
from parity_util import ORC_MOVE, compare_round, gpu_problem, oracle_problem

pytestmark = pytest.mark.gpu
D, K = 256, 16


@pytest.fixture(scope="module")
def params():
    rng = np.random.default_rng(4)
    return dict(means=(0.3 * rng.standard_normal((K, D))).astype(np.float32),
                log_scales=rng.uniform(-0.7, -0.5, K).astype(np.float32))


@pytest.mark.parametrize("move", ["rwmh", "mala", "hmc"])
@pytest.mark.parametrize("resample", [None, "sir", "fixed"])
def test_passes(params, move, resample):
    import paper_2408_12057_amd as oa
    assert torch.cuda.is_available()
    N, T = 131, 4
    beta = np.linspace(0, 1, T + 1) ** 2
    eps = np.full(T, {"rwmh": 0.02, "mala": 0.1, "hmc": 0.05}[move])
    kw = dict(resample_at=np.array([0, 1, 0, 0], dtype=np.int32)) if resample == "fixed" else {}
    trigger = {None: 0, "sir": 2, "fixed": 3}[resample]
    g = oa.asmc(gpu_problem(oa, "gmm", params, 2.0), N, beta, eps, 5, move=move, leapfrog=3, accept_bits=True,
                resample_=resample is not None, trigger=trigger, **kw)
    o = orc.asmc(oracle_problem("gmm", D, params, 2.0),
                 orc.Opts(move=ORC_MOVE[move], leapfrog=3, resample=int(resample is not None), trigger=trigger,
                          nu=0.5, state_f32=1, **kw), N, beta, eps, 5, traces=True)
    compare_round(g, o, T, N)


def test_tempering(params):
    import paper_2408_12057_amd as oa
    Np, Tp, copies = 31, 4, 3  # the most chains a copy holds at this d
    beta = np.linspace(0, 1, Np + 1) ** 2
    eps = np.full(Np + 1, 0.05)
    g = oa.pt(gpu_problem(oa, "gmm", params, 2.0), copies, beta, eps, Tp, 11, move="hmc", leapfrog=3)
    o = orc.pt(oracle_problem("gmm", D, params, 2.0), orc.Opts(move=orc.MOVE_HMC, leapfrog=3, state_f32=1),
               copies, beta, eps, Tp, 11)
    np.testing.assert_allclose(g["ss"], o["ss"], rtol=1e-11, atol=1e-11)
    assert g["trips"] == o["trips"]
    np.testing.assert_allclose(g["tmean"], o["tmean"], rtol=1e-12, atol=1e-13)
