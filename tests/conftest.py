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


@pytest.fixture(params=[None, 0], ids=["form by size", "main kernel"])
def attn_few(request):
    """Small bf16 batches in the attention form that their size gives them, and in the main kernel's."""
    from helpers import env_setting
    with env_setting("RESPEC_ATTN_FEW", request.param):
        yield request.param
