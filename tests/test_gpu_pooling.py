"""The sums over many copies or tiles at the edges of the workgroups that form them:
parallel tempering's pooled outputs over more copies than a workgroup has threads,
against the oracle, and rejuvenation's averages over more tiles than a workgroup has
threads, against the states themselves after one step."""
import numpy as np
import pytest
import torch

import oracle as orc
from parity_util import gpu_problem, oracle_problem
from paper_2408_12057_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def oa():
    import paper_2408_12057_amd as m
    assert torch.cuda.is_available()
    return m


@pytest.mark.parametrize("family,d,K,Np,Tp", [("gauss", 3, 1, 1, 2), ("gauss", 3, 255, 2, 3),
                                              ("gauss", 10, 257, 5, 4), ("gmm", 40, 300, 40, 2)])
def test_pt_pooled_over_copies(oa, family, d, K, Np, Tp):
    rng = np.random.default_rng(K)
    params = wl.random_gauss(rng, d) if family == "gauss" else wl.random_gmm(rng, d, 3)
    beta = np.linspace(0, 1, Np + 1) ** 2
    eps = np.full(Np + 1, 0.2)
    g = oa.pt(gpu_problem(oa, family, params, 1.5), K, beta, eps, Tp, 11, move="rwmh")
    o = orc.pt(oracle_problem(family, d, params, 1.5), orc.Opts(move=orc.MOVE_RWMH, state_f32=1),
               K, beta, eps, Tp, 11)
    # K T' (40 terms a temperature at most 1200) summed in binary64 in another order
    np.testing.assert_allclose(g["ss"], o["ss"], rtol=1e-11, atol=1e-11)
    np.testing.assert_allclose(g["rej"], o["rej"], rtol=1e-12, atol=1e-13)
    assert g["trips"] == o["trips"]
    np.testing.assert_allclose(g["tmean"], o["tmean"], rtol=1e-12, atol=1e-13)
    np.testing.assert_allclose(g["tsecond"], o["tsecond"], rtol=1e-12, atol=1e-13)


@pytest.mark.parametrize("N,d", [(1, 2), (64 * 1024, 3), (64 * 1025 + 7, 5), (3 * 4096 + 1, 100)])
def test_rejuvenation_averages(oa, N, d):
    rng = np.random.default_rng(N)
    x = torch.tensor(rng.standard_normal((N, d)).astype(np.float32), device="cuda")
    lw = torch.tensor(rng.standard_normal(N), device="cuda")
    p = gpu_problem(oa, "gauss", wl.random_gauss(rng, d), 1.0)
    r = oa.rejuvenate(p, lw, x, 1, 0.1, 3, move="rwmh", return_states=True)
    xs = r["x"].cpu().numpy().astype(np.float64)
    # N terms of size 1 in binary64: N u of sum |x|, N <= 2^17
    np.testing.assert_allclose(r["mean"], xs.mean(0), rtol=0, atol=2e-11)
    np.testing.assert_allclose(r["second"], (xs ** 2).mean(0), rtol=2e-11, atol=0)
