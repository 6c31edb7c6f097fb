import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu on the GPU box)")


@pytest.fixture(scope="session")
def oracle():
    import oracle as _oracle
    _oracle.build()
    return _oracle


@pytest.fixture(params=[0, 32768], ids=["", "two kernels"])
def bound(request):
    """max_seq_len of the calls where it is more than the longest sequence.  At 0 a short context runs as one launch; from 32768 on
    every call runs as scan and select kernels, whatever its lengths (test_one_launch.py)."""
    return request.param
