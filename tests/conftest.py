import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu)")


@pytest.fixture(params=[0, 1, 2], ids=["chosen", "int8", "general"])
def kernels(request):
    """The test runs with the kernels the library chooses, with its int8 kernels only, and with its general kernel only."""
    import paper_2111_00153_amd as m
    m.rmsmp_debug_set_wave_split(0, 0, request.param, 0)
    yield request.param
    m.rmsmp_debug_set_wave_split(0, 0, 0, 0)


@pytest.fixture(scope="session")
def oracle():
    import oracle as _oracle
    _oracle.build()
    return _oracle
