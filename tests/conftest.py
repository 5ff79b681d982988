import os
import sys
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu)")


def pytest_collection_modifyitems(config, items):
    """GPU tests are skipped, not failed, where no device is visible."""
    try:
        import torch
        have = torch.cuda.is_available()
    except Exception:
        have = False
    if have:
        return
    skip = pytest.mark.skip(reason="no GPU visible")
    for it in items:
        if "gpu" in it.keywords:
            it.add_marker(skip)


@pytest.fixture(params=[1, 2], ids=["default", "two_streams"])
def backward_streams(request):
    """The encoder's backward passes as a user gets them (one stream for models as small as the tests'), and with the second
    stream that large ones take."""
    import ctypes
    import paper_2310_05674_amd as pkg
    lib = pkg.load_library()
    lib.sama_dev_side_stream(ctypes.c_int32(request.param))
    yield request.param
    lib.sama_dev_side_stream(ctypes.c_int32(1))
