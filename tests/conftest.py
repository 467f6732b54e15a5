import gc
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu)")


def pytest_runtest_setup(item):
    # tensors that an earlier test left in reference cycles (pytest.raises keeps a frame) go now, not in the middle of a test
    # that looks at what the allocator has handed out
    if item.get_closest_marker("gpu"):
        gc.collect()
