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
    from oracle import easyspec_oracle as eso
    eso.lib()
    return eso


@pytest.fixture(params=["one launch", "launches"])
def route(request, monkeypatch):
    """Passes of small models as the library runs them (one launch where that is faster), and all as separate launches."""
    if request.param == "launches":
        monkeypatch.setenv("EASYSPEC_RESIDENT", "0")
    return request.param
