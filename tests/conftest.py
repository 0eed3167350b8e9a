import os
import re
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu)")


def _have_gpu() -> bool:
    try:
        import torch
        return torch.cuda.is_available()
    except Exception:
        return False


def pytest_collection_modifyitems(config, items):
    if _have_gpu():
        return
    skip = pytest.mark.skip(reason="no GPU in this process")
    for item in items:
        if "gpu" in item.keywords:
            item.add_marker(skip)


def nsk_switches():
    """The names that the library's header lists as its test switches."""
    text = open(os.path.join(ROOT, "include", "nsk.h")).read()
    listed = text[text.index("/* Test and A/B switches."):text.index("void nsk_test_hooks_reload")]
    return set(re.findall(r"NSK_[A-Z0-9_]+", listed))


@pytest.fixture
def nsk_env(monkeypatch):
    """Sets one of libnsk's NSK_* test switches for the duration of a test (None: not set).  The library reads its switches
    once, so every change (and the restoration afterwards) is followed by nsk_test_hooks_reload().  A name that the
    library does not read would force nothing: it is refused."""
    from paper_2409_11600_amd import binding
    known = nsk_switches()

    def set_switch(name, value):
        assert name in known, f"{name} is no switch of the library"
        if value is None:
            monkeypatch.delenv(name)
        else:
            monkeypatch.setenv(name, value)
        binding.lib().nsk_test_hooks_reload()

    yield set_switch
    monkeypatch.undo()
    binding.lib().nsk_test_hooks_reload()
