import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu)")
    config.addinivalue_line("markers", "slow: full-size case (seconds on the GPU, minutes of oracle work where it is not precomputed)")


@pytest.fixture(params=[0, 2], ids=["as_it_comes", "ordered"])
def form(request, engine):
    """The test's batches in the form that their sizes choose, and in the ordered forms whatever their sizes."""
    engine.sja_set_resolve_mode(request.param)
    yield request.param
    engine.sja_set_resolve_mode(0)


@pytest.fixture(scope="session")
def oracle():
    import oracle as O
    O.build()
    return O
