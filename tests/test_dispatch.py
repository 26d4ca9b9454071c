"""The launch arithmetic on the CPU: tiles and pacing at the borders of their
rules."""
import pytest

import dispatch_rules as rules
import paper_2507_07114_amd as ll


def test_defaults_are_the_bindings():
    got, want = rules.defaults(), ll.ll_get_pacing()
    want["mode"] = rules.MODES[want["mode"]]
    assert got == want


@pytest.mark.parametrize("f32,n,d,L,step,flat", [
    # (fp32 rows, n, d, packet, of a step): flat tiles?
    (False, 64, 105_250_000, 4096, True, False),
    (False, 16, 16_777_259, 750, True, True),
    (False, 3, 70_001, 64, True, True),
    (False, 3, 70_001, 63, True, False),  # shorter than the shortest flat packet
    # full chunks off the 128-byte lines: by the number of rows in a step
    (False, 12, 6000 * 400, 6000, True, True),
    (False, 11, 6000 * 400, 6000, True, False),
    (False, 11, 6000 * 400, 6000, False, True),
    # a multiple of 8 in few tiles stays with chunks
    (False, 9, 256 * 1024, 256, True, False),
    (False, 9, 256 * 1025, 256, True, True),
    (True, 2, 72 * 4096, 72, True, False),
    (True, 2, 72 * 4097, 72, True, True),
])
def test_tiles(f32, n, d, L, step, flat):
    count, slots = rules.tiles(f32, n, d, L, step)
    T = 1024 if f32 else 2048
    P = -(-d // L)
    assert (slots > 0) == flat
    assert count == (-(-d // T) if flat else P * -(-L // T))
    # never more partials than the workspace holds, whatever the tiles
    assert count <= P * -(-L // 1024)
