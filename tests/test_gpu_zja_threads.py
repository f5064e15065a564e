"""The online selection from two threads at once, each with its handle and stream and with
populations that need little and much LDS: what each gives alone."""
import ctypes
import threading

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def test_two_threads(monkeypatch):
    import paper_2408_12057_amd as oa
    from paper_2408_12057_amd import api
    assert torch.cuda.is_available()
    problem = oa.Problem.gauss(np.full(3, 2.0, np.float32), 0.25, 1.0)
    sizes = (40, 8192)
    want = [oa.zja(problem, N, 0.7, 60, 0.3, 5, move="rwmh") for N in sizes]
    own = threading.local()
    shared = api._handle
    monkeypatch.setattr(api, "_handle", lambda dev: getattr(own, "handle", None) or shared(dev))
    errors, handles = [], []
    for _ in sizes:
        h = ctypes.c_void_p()
        api._check(api._load().oasmc_handle_create(ctypes.byref(h), 0))
        handles.append(h)
    start = threading.Barrier(2)

    def work(i):
        try:
            own.handle = handles[i]
            with torch.cuda.stream(torch.cuda.Stream()):
                start.wait(30)
                for _ in range(10):
                    got = oa.zja(problem, sizes[i], 0.7, 60, 0.3, 5, move="rwmh")
                    assert got["T"] == want[i]["T"]
                    np.testing.assert_array_equal(got["beta"], want[i]["beta"])
                    np.testing.assert_array_equal(got["log_g"], want[i]["log_g"])
                    assert torch.equal(got["lw"], want[i]["lw"]) and torch.equal(got["x"], want[i]["x"])
        except BaseException as e:  # noqa: BLE001 (reported by the test's thread)
            errors.append((sizes[i], e))

    threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join(60)
    assert not errors, errors
    torch.cuda.synchronize()
    for h in handles:
        api._check(api._load().oasmc_handle_destroy(h))
