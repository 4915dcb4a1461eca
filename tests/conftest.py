import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu on the GPU box)")


def pytest_collection_modifyitems(config, items):
    """test_gpu_whole_planes runs other modules' tests once more with calls of few planes on other kernels.  Calls of fewer than four
    directions run the same kernel either way: not twice."""
    again = [i for i in items if i.module.__name__ == "test_gpu_whole_planes"
             and getattr(getattr(i, "callspec", None), "params", {}).get("mask", 15) not in (15, None)]
    if again:
        config.hook.pytest_deselected(items=again)
        items[:] = [i for i in items if i not in set(again)]


def _reload_library_env():
    """The library reads its GSPN_* testing aids once per process; tell it that they changed."""
    from paper_2512_07884_amd import binding
    if os.path.exists(binding.lib_path()):
        binding.gspn_reload_env()


@pytest.fixture
def monkeypatch(monkeypatch):
    """pytest's monkeypatch, with one addition: a change to a GSPN_* environment variable reaches the library."""
    setenv, delenv = monkeypatch.setenv, monkeypatch.delenv

    def setenv_and_reload(name, value, prepend=None):
        setenv(name, value, prepend)
        if name.startswith("GSPN_"):
            _reload_library_env()

    def delenv_and_reload(name, raising=True):
        delenv(name, raising)
        if name.startswith("GSPN_"):
            _reload_library_env()

    monkeypatch.setenv = setenv_and_reload
    monkeypatch.delenv = delenv_and_reload
    yield monkeypatch
    monkeypatch.undo()
    _reload_library_env()


@pytest.fixture
def family_kernels(monkeypatch):
    """For tests of the "plane", "tile" and "twopass" kernels: no any-size kernel in their place."""
    monkeypatch.setenv("GSPN_NO_ANY_SIZE", "1")
