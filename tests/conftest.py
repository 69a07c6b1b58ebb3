import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs an MI355X (gfx950) GPU and the HIP library")
    config.addinivalue_line("markers", "slow: long-running CPU test")


@pytest.fixture(scope="session")
def gpu_available():
    import torch
    return torch.cuda.is_available()


# tests that link the library's objects by hand: they get objects of the
# present sources, not whatever an earlier build left
LINK_OBJECTS = ("test_sanitize_cpu.py", "test_pass_forms_cpu.py")


def pytest_runtest_setup(item):
    if item.path.name in LINK_OBJECTS:
        from paper_2602_01888_amd import build
        if os.path.exists(build.HIPCC) and build.stale_objects():
            build.build()
