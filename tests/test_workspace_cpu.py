"""rtx.Workspace: how large it gets, and for which calls."""
import pytest

from paper_1912_12786_amd import rtx


def test_get_is_exact():
    ws = rtx.Workspace("cpu")
    assert ws.get(0) == (None, 0)
    assert ws.get(100) == (ws.buf.data_ptr(), 100)
    assert ws.get(50)[1] == 100 and ws.get(5000)[1] == 5000


@pytest.mark.parametrize("shape,grows", [(None, True), ((64, 8, 64, 0), True), ((64, 16, 64, 1), True),
                                         ((256, 8, 64, 1), False), ((64, 8, 128, 1), False),
                                         ((64, 8, 32, 1), False)])
def test_room_for_spreading(shape, grows):
    """Only shapes that spread a small launch, up to SPREAD_BYTES, worked out
    once per depth and shape."""
    flags, asked = rtx.shape_flag(shape), []

    def size(n):
        asked.append(n)
        return n

    ws = rtx.Workspace("cpu")
    for _ in range(2):
        ws.make_room(20, flags | rtx.RT_FLAG_COUNT | rtx.tile_flag(64), lambda: size(3 << 20))
    assert ws.get(1000)[1] == (3 << 20 if grows else 1000) and len(asked) == grows
    ws.make_room(21, flags, lambda: size(1 << 20))
    assert ws.get(1000)[1] == (3 << 20 if grows else 1000)
    ws.make_room(90, flags, lambda: size(1 << 40))
    assert ws.get(1000)[1] == (rtx.SPREAD_BYTES if grows else 1000)
