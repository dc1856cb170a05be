import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu on the GPU box)")


@pytest.fixture(scope="session")
def golden_dir():
    return os.path.join(ROOT, "tests", "golden")


@pytest.fixture(scope="session")
def few_cus():
    """A stream of eight of the device's CUs (no more than 64 workgroups of four waves at a time)."""
    import ctypes

    import torch

    hip, handle = ctypes.CDLL("libamdhip64.so"), ctypes.c_void_p()
    torch.cuda.synchronize()
    assert hip.hipExtStreamCreateWithCUMask(ctypes.byref(handle), 8, (ctypes.c_uint32 * 8)(255)) == 0
    return torch.cuda.ExternalStream(handle.value)


LEAVE = 1 << 20


@pytest.fixture
def looks(few_cus):
    """with looks(limit): compress calls whose workgroups look so often for one another's counts (0: as built; INTERNAL_NO_SHORT: two
    launches); LEAVE: on few CUs and once, so that in launches of more workgroups than these hold most leave their tiles."""
    import contextlib

    import torch

    import paper_2605_01708_amd as sz

    @contextlib.contextmanager
    def way(limit):
        sz.internal_test_short(1 if limit == LEAVE else limit, limit == LEAVE)
        torch.cuda.synchronize()
        try:
            with torch.cuda.stream(few_cus) if limit == LEAVE else contextlib.nullcontext():
                yield
            torch.cuda.synchronize()
        finally:
            sz.internal_test_short()

    yield way
