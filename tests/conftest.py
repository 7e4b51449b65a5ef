import ctypes
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs an MI355X (gfx950) GPU")
    config.addinivalue_line("markers", "slow: full-size workloads")


def pytest_collection_modifyitems(config, items):
    # Full-size oracle runs take minutes of host time; they run only on request.
    if os.environ.get("PEEK_SLOW") == "1":
        return
    skip = pytest.mark.skip(reason="full-size workload; set PEEK_SLOW=1 to run")
    for item in items:
        if "slow" in item.keywords:
            item.add_marker(skip)


@pytest.fixture
def forced_library(monkeypatch):
    """The package on a build of the library with sampled places known beforehand and waits
    between workgroups that give up at once."""
    import paper_2607_02525_amd as P
    import paper_2607_02525_amd.runner as R
    lib = ctypes.CDLL(os.path.join(os.path.dirname(P.LIB_PATH), "libpeek_forced.so"))
    for name, res, args in P.EXPORTS:
        fn = getattr(lib, name)
        fn.restype, fn.argtypes = res, args
    monkeypatch.setattr(P, "_lib", lib)
    monkeypatch.setattr(R, "_lib", lib)
    return lib
