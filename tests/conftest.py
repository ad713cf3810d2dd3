import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu)")


@pytest.fixture
def always_halves():
    """Chains on two streams work on the halves of a batch side by side even where the layers are short."""
    from paper_2202_05239_amd import binding as f8
    f8.f8_tuning_set("halves", 2)
    yield
    f8.f8_tuning_set("halves", 1)


@pytest.fixture(scope="session")
def oracle():
    from oracle import build, ref
    build.build(force=False)
    return ref
