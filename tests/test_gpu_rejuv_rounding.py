"""Rejuvenation's averages are sums of many terms: after one step they are compared with
sums of the returned states in 64-bit mantissas.  A pairwise sum over the tiles leaves
3.1e-16 of the largest average on these draws (mean over them of the largest error);
sixteen partial sums added one after the other leave 3.6e-16."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.skipif(np.finfo(np.longdouble).nmant < 63, reason="no 64-bit mantissas here")
def test_rounding_of_the_averages():
    import paper_2408_12057_amd as oa
    assert torch.cuda.is_available()
    err = []
    for seed in range(60):
        rng = np.random.default_rng(seed)
        N, d = int(np.exp(rng.uniform(np.log(1000), np.log(1 << 19)))), int(rng.integers(2, 40))
        x = torch.tensor(rng.standard_normal((N, d)).astype(np.float32), device="cuda")
        lw = torch.tensor(rng.standard_normal(N), device="cuda")
        p = oa.Problem.gauss((2 + 0.1 * rng.standard_normal(d)).astype(np.float32), 0.25, 1.0)
        r = oa.rejuvenate(p, lw, x, 1, 0.1, seed, move="rwmh", return_states=True)
        want = (r["x"].cpu().numpy().astype(np.longdouble) ** 2).mean(0)
        err.append(float(np.abs(r["second"] - want).max() / want.max()))
    assert np.mean(err) < 3.3e-16, np.mean(err)
