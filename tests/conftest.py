import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs an MI355X (gfx950) GPU")


# the forms that small steps fall back to, at every size: built by
# __graft_entry__.build()
FALLBACKS = os.path.join(os.path.dirname(os.path.abspath(__file__)), "libsifar_fallbacks.so")


def _load_fallbacks(monkeypatch):
    import paper_2607_08973_amd as S

    monkeypatch.setattr(S, "_lib", None)
    S.load(FALLBACKS)


@pytest.fixture
def fallbacks(monkeypatch):
    """Handles of the fallback library: a per-epoch step is a graph of launches
    whatever its size (checked here on a step that one launch would serve)."""
    import paper_2607_08973_amd as S

    _load_fallbacks(monkeypatch)
    with S.Sifar(nranks=2, hidden=512, max_tokens=1, reduces_per_step=4) as s:
        assert s.step_plan(1) == (6, 1, 0)


@pytest.fixture(params=["padded", "unpadded"])
def grid(request, monkeypatch):
    """Persistent plain steps with the library's grid, whose idle rows put a
    chunk's consumer and producer on one XCD, or without those rows."""
    if request.param == "unpadded":
        _load_fallbacks(monkeypatch)
    return request.param
