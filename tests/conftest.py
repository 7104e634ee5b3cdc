import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs an MI355X (gfx950) GPU and the built HIP library")
    config.addinivalue_line("markers", "slow: full-size workload; minutes of work")


@pytest.fixture
def launch_shape(request):
    """The launch shape of the test's decode calls (``launch_shape.pinned``)."""
    from launch_shape import pinned
    with pinned(request.param):
        yield request.param
