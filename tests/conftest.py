import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs an MI355X (runs through the C-ABI library)")
    config.addinivalue_line("markers", "slow: oracle checks that take more than a few seconds")


GOLDEN = os.path.join(ROOT, "tests", "golden")


def read_golden(name):
    """Parse a `key = value` fixture (lines starting with # are comments)."""
    out = {}
    with open(os.path.join(GOLDEN, name)) as fh:
        for line in fh:
            line = line.split("#", 1)[0].strip()
            if not line:
                continue
            key, val = (s.strip() for s in line.split("=", 1))
            out[key] = val
    return out


@pytest.fixture(autouse=True)
def no_pinned_shape_outlives_its_test(monkeypatch):
    """Stencil shapes are pinned for the whole process: after a test that pinned
    one, the table is cleared, so that the next test runs what the tuner picks."""
    pinned = []

    def module():
        return sys.modules.get("paper_1106_4964_amd.ovl")

    if module():
        pin = module().stencil_set_shape

        def noted(*args):
            pinned.append(args)
            return pin(*args)

        monkeypatch.setattr(module(), "stencil_set_shape", noted)
    else:
        pinned.append("a test that loads the library is not watched")
    yield
    if pinned and module():
        module().ovl_stencil_tune(0 if os.environ.get("OVL_TUNE", "1").startswith("0") else 1)
