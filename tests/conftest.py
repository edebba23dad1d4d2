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
    import oracle as o

    o.build()
    return o


@pytest.fixture(params=["own", "teams"])
def route(request):
    """The route the library chooses, and that of the large calls for calls it sends another way because they are
    small: a test of either kernel with inputs that are small enough to be checked against the oracle."""
    import paper_2502_20704_amd as fsd

    if request.param == "own":
        yield request.param
        return
    prev = fsd.debug_set_small_calls(False)
    try:
        yield request.param
        assert fsd.debug_last_route() == 0
    finally:
        fsd.debug_set_small_calls(prev)


@pytest.fixture
def small_and_large(route):
    """As `route`, for a test whose last call is one that the library does take the small route for."""
    import paper_2502_20704_amd as fsd

    yield route
    if route == "own":
        assert fsd.debug_last_route() != 0
