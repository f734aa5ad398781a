"""Workspaces that the binding allocates by itself: with the optional part where there is room
for it, without it otherwise, and kept per key while they cover what is asked for.  The
allocator is torch's on the CPU, with a limit put in front of it."""
import pytest

torch = pytest.importorskip("torch")

from paper_1903_03056_amd import collision as C


@pytest.fixture
def room(monkeypatch):
    """A device with room for state["free"] bytes; state["made"] lists what was allocated."""
    state = {"free": 10 ** 6, "made": []}
    empty = torch.empty

    def limited(n, **kw):
        if n > state["free"]:
            raise torch.cuda.OutOfMemoryError("no room")
        state["made"].append(n)
        return empty(n, **kw)

    monkeypatch.setattr(torch, "empty", limited)
    return state


def test_optional_part_is_left_out_where_there_is_no_room(room):
    assert C._scratch(1000, 400, "cpu", None).numel() == 1000
    room["free"] = 999
    assert C._scratch(1000, 400, "cpu", None).numel() == 600
    with pytest.raises(torch.cuda.OutOfMemoryError):
        C._scratch(1000, 0, "cpu", None)
    with pytest.raises(torch.cuda.OutOfMemoryError):
        C._scratch(1400, 400, "cpu", None)


def test_kept_workspaces_cover_every_call(room):
    cache = C._ScratchCache()
    big = cache.get("a", 1000, lambda: 400, "cpu", None)
    assert cache.get("a", 900, lambda: 500, "cpu", None) is big
    assert cache.get("b", 900, lambda: 500, "cpu", None) is not big
    room["free"] = 1500
    lean = cache.get("a", 2000, lambda: 700, "cpu", None)
    assert lean.numel() == 1300
    # asked for again, and for less: kept; for less of which more is needed: not
    assert cache.get("a", 2000, lambda: 700, "cpu", None) is lean
    assert cache.get("a", 1500, lambda: 300, "cpu", None) is lean
    assert cache.get("a", 1450, lambda: 100, "cpu", None).numel() == 1450
    assert room["made"] == [1000, 900, 1300, 1450]
