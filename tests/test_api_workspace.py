"""The binding's growable workspace on a device without room for what a call asks for (no GPU: the allocator and the
library's size queries are stand-ins)."""
import pytest

torch = pytest.importorskip("torch")

from paper_2107_13797_amd import api  # noqa: E402

ASKED, LEAST = 5000, 1200


class Library:
    def haflo_workspace_bytes(self, handle, op, rows, cols):
        return ASKED * rows

    def haflo_workspace_bytes_least(self, handle, op, rows, cols):
        return LEAST * rows

    def haflo_encrypt(self, handle, plain, r, out, count, ws, nbytes, stream):
        Library.got = nbytes
        return 0

    def haflo_ctx_destroy(self, handle):
        return 0


class Device:
    """Memory of `room` bytes that only workspaces live in."""

    def __init__(self, monkeypatch, room):
        self.room, self.asked = room, []
        monkeypatch.setattr(api, "lib", Library)
        monkeypatch.setattr(api, "_ptr", lambda t: None)
        monkeypatch.setattr(api, "_stream", lambda: None)
        monkeypatch.setattr(api.torch, "empty", self.empty)
        monkeypatch.setattr(api.torch.cuda, "mem_get_info", lambda: (self.room, 1 << 40))
        monkeypatch.setattr(api.torch.cuda, "memory_reserved", lambda: 0)
        monkeypatch.setattr(api.torch.cuda, "memory_allocated", lambda: 0)
        monkeypatch.setattr(api.torch.cuda, "synchronize", lambda: None)

    def empty(self, nbytes, dtype=None, device=None):
        self.asked.append(nbytes)
        if nbytes > self.room:
            raise torch.cuda.OutOfMemoryError("out of memory")
        return torch.zeros(nbytes, dtype=dtype)


@pytest.fixture
def ctx():
    c = api.Context.__new__(api.Context)
    c.handle, c._ws, c._refused = 1, None, float("inf")
    yield c
    c.handle = None


def ask(ctx, rows):
    """The workspace that an encryption of `rows` elements is called with."""
    plain = torch.zeros((rows, 1))
    api.haflo_encrypt(ctx, plain, plain, out=plain)
    return Library.got


def test_room_for_what_is_asked(monkeypatch, ctx):
    d = Device(monkeypatch, 10 * ASKED)
    assert [ask(ctx, r) for r in (1, 3, 2)] == [ASKED, 3 * ASKED, 3 * ASKED]
    assert d.asked == [ASKED, 3 * ASKED]


def test_least_size_where_the_device_is_full(monkeypatch, ctx):
    d = Device(monkeypatch, 2 * ASKED)
    assert ask(ctx, 4) == 4 * LEAST
    assert d.asked == [4 * ASKED, 4 * LEAST]
    # the same call again finds its buffer and does not run into the wall once more
    assert ask(ctx, 4) == 4 * LEAST and len(d.asked) == 2
    # one that fits the device is asked for in full
    assert ask(ctx, 2) == 2 * ASKED
    # and so is the first one once there is room
    d.room = 4 * ASKED
    assert ask(ctx, 4) == 4 * ASKED


def test_no_room_at_all(monkeypatch, ctx):
    Device(monkeypatch, LEAST)
    with pytest.raises(torch.cuda.OutOfMemoryError):
        ask(ctx, 2)


def test_bad_query(monkeypatch, ctx):
    Device(monkeypatch, ASKED)
    with pytest.raises(api.HafloError):
        ctx.workspace(2 ** 64 - 1)
