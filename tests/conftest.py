import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu on the GPU box)")


@pytest.fixture(params=["short", "long"])
def attention_route(request):
    """Both sets of attention kernels, whichever the shape alone would take."""
    from paper_2511_12201_amd import binding as ob
    ob.debug_attention_route({"short": 1, "long": 2}[request.param])
    yield request.param
    ob.debug_attention_route(0)


@pytest.fixture(scope="session")
def repo_root():
    return ROOT
