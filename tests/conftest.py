import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu)")


@pytest.fixture(scope="session")
def orc():
    import oracle
    oracle.lib()
    return oracle


@pytest.fixture(scope="module", autouse=True)
def _no_garbage_of_earlier_modules():
    """Tensors that a failed expectation or an autograd graph left in a reference cycle go before the next module
    starts: a test that watches the allocator's counters must not see the collector free them in between."""
    import gc
    gc.collect()
