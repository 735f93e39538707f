import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu)")


@pytest.fixture(scope="session")
def oracle():
    import oracle as _oracle
    _oracle.build()
    return _oracle


@pytest.fixture(scope="session")
def kernels_of():
    """The names of the kernels that a call launches, in order, as the profiler reports them (template arguments included)."""
    import torch
    from torch.profiler import ProfilerActivity, profile

    def names(call):
        call()  # (once outside, so that nothing is set up inside)
        torch.cuda.synchronize()
        with profile(activities=[ProfilerActivity.CUDA]) as p:
            call()
            torch.cuda.synchronize()
        found = [e.name for e in p.events() if "mip::" in e.name]
        assert found, [e.name for e in p.events()]
        return found
    return names
