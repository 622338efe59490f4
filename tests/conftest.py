import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs an MI355X (runs the HIP library)")
    config.addinivalue_line("markers", "slow: long-running CPU test")


@pytest.fixture(scope="session")
def gpu_device():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


@pytest.fixture(params=["default", "general"])
def in_core_path(request, monkeypatch):
    """Runs a test of graphs that one workgroup can hold on the path they take
    by themselves and on the general path."""
    if request.param == "general":
        monkeypatch.setenv("WL_SMALL", "0")
    return request.param
