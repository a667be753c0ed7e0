import functools
import os
import sys
import time

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs an MI355X (gfx950) and the built HIP library")
    config.addinivalue_line("markers", "slow: long-running CPU test")


@pytest.fixture(autouse=True)
def arrivals_meet_in_flight(request, monkeypatch):
    """test_gpu_serve.py::test_alone_equals_mixed counts on jobs that arrive 2 ms apart
    meeting in flight, but a job of its size takes 1 ms once the process's first
    launches are made. Its servers' clocks run a hundred times faster, so that every
    job is there before the first one is done, in whatever order the tests run."""
    if request.node.name == "test_alone_equals_mixed" and request.node.path.name == "test_gpu_serve.py":
        from paper_2410_10447_amd import serve
        fast = functools.partial(serve.Server, clock=lambda: 100.0 * time.perf_counter())
        monkeypatch.setattr(serve, "Server", fast)
