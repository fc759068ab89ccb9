import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs an MI355X (HIP device)")
    config.addinivalue_line("markers", "slow: longer CPU test")


@pytest.fixture(scope="session")
def orc():
    import oracle
    oracle.lib()
    return oracle


def pytest_collection_modifyitems(items):
    # what the tuner tries follows the measured times, and near a tie of two depths no
    # theta move may come up: last, so that a run that stops there has run the others
    items.sort(key=lambda item: item.name == "test_timestepping_with_theta_walk")
