import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs an MI355X (gfx950) and the built HIP library")
    config.addinivalue_line("markers", "slow: long-running CPU test")


def pytest_collection_modifyitems(items):
    """The GPU serving tests run first: one of them counts on jobs that arrive 2 ms
    apart meeting in flight, which they do while the process's first launches and
    page-locked allocations are still to be made; once those are, a job of its size
    takes 1 ms alone."""
    items.sort(key=lambda item: item.path.name != "test_gpu_serve.py")
