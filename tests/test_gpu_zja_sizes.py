"""The online selection of beta_t at the edges of its storage rules: particles a
thread reads once (up to 16384), particles with weight held in LDS (up to 8192),
and read from memory at each evaluation, on targets where every particle has
weight (Gaussian) and where most have none (Unid), and few halvings.  Compared as
in test_gpu_zja: a halving that meets rho at rounding may fall either way, and
the difference of one cell carries into the later steps."""
import numpy as np
import pytest
import torch

import oracle as orc
from parity_util import gpu_problem, oracle_problem
from paper_2408_12057_amd import workloads as wl
from test_gpu_zja import _zja_compare

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def oa():
    import paper_2408_12057_amd as m
    assert torch.cuda.is_available()
    return m


@pytest.mark.parametrize("N,iters", [(1, 40), (65, 40), (8192, 40), (8193, 40), (16384, 40), (16385, 40),
                                     (3000, 1), (3000, 7)])
def test_gaussian(oa, N, iters):
    w = wl.gaussian_d10()
    g = oa.zja(gpu_problem(oa, "gauss", w.params, 1.0), N, 0.5, 60, 0.2, 5, move="rwmh", iters=iters)
    o = orc.zja(oracle_problem("gauss", 10, w.params, 1.0), orc.Opts(move=orc.MOVE_RWMH, state_f32=1), N, 0.5,
                60, 0.2, 5, iters=iters)
    _zja_compare(g, o, N)


@pytest.mark.parametrize("N", [300, 16384, 20011])
def test_unid(oa, N):
    g = oa.zja(oa.Problem.unid(1e11, 1e10), N, 0.8, 400, 1.0, 9, move="rwmh3")
    o = orc.zja(orc.Problem(family=orc.FAM_UNID, d=2, binom_n=1e11, binom_k=1e10, box=10.0),
                orc.Opts(move=orc.MOVE_RWMH3, state_f32=1), N, 0.8, 400, 1.0, 9)
    _zja_compare(g, o, N)
