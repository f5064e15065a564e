"""A pass that fails after its schedule is on the way (its workspace is larger than the
GPU) leaves the handle as it was: the next passes, on the same and on another stream and
with a longer schedule, give what they gave before."""
import numpy as np
import pytest
import torch

from parity_util import gpu_problem
from paper_2408_12057_amd import workloads as wl

pytestmark = pytest.mark.gpu


def test_next_calls_after_a_failed_one():
    import paper_2408_12057_amd as oa
    assert torch.cuda.is_available()
    p = gpu_problem(oa, "gauss", wl.random_gauss(np.random.default_rng(0), 256), 1.0)

    def run(T, N=300, **kw):
        return oa.asmc(p, N, np.linspace(0, 1, T + 1) ** 2, 0.05, 7, resample_=True, trigger="ess", **kw)

    want = {T: run(T) for T in (5, 9, 4000)}
    other = torch.cuda.Stream()
    for T in (5, 9, 4000):
        with pytest.raises(oa.OasmcError):
            run(T, N=1 << 30, return_state=False)  # states of 1 TiB
        with torch.cuda.stream(other):
            got = run(T)
        torch.cuda.synchronize()
        again = run(T)
        for r in (got, again):
            assert r["logZ"] == want[T]["logZ"] and r["n_resample"] == want[T]["n_resample"]
            np.testing.assert_array_equal(r["log_g"], want[T]["log_g"])
            np.testing.assert_array_equal(r["ess"], want[T]["ess"])
            assert torch.equal(r["x"], want[T]["x"]) and torch.equal(r["lw"], want[T]["lw"])
