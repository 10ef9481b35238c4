import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu)")


@pytest.fixture(scope="session")
def lib():
    """The ctypes binding over the C-ABI library (built in-tree if absent)."""
    from paper_2410_18311_amd import build as _build
    if not os.path.exists(_build.LIB_PATH):
        _build.build_library()
    from paper_2410_18311_amd import coreinfer
    return coreinfer


@pytest.fixture(autouse=True)
def _development_settings_are_put_back(request):
    """A test that changes a development setting puts it back: the tests after it run what a user gets."""
    if "lib" not in request.fixturenames:
        yield
        return
    library = request.getfixturevalue("lib")
    before = library.dev_params()
    assert before == _SETTINGS.setdefault("defaults", before)
    yield
    after = library.dev_params()
    for name, value in before.items():
        library.dev_set_param(name, value)
    assert after == before, "development settings left changed"


_SETTINGS: dict = {}


def gpu_available() -> bool:
    import torch
    return torch.cuda.is_available()
