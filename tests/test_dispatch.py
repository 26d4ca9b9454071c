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


@pytest.mark.parametrize("f32,flat,n,tiles,paced", [
    # two rounds (of 2048 bf16 or 1024 fp32 tiles) from 64 workers on
    (False, False, 64, 2048, False), (False, False, 64, 2049, True),
    (False, True, 63, 2049, False), (False, True, 64, 2049, True),
    # one round only with very many workers, and not a short one
    (False, False, 159, 2048, False), (False, False, 160, 2048, True),
    (False, False, 160, 1, False), (False, False, 1024, 16, False),
    (False, False, 160, 819, False), (False, False, 160, 820, True),
    (False, False, 1024, 159, False), (False, False, 1024, 160, True),
    (False, True, 160, 271, False), (False, True, 160, 272, True),
    (False, True, 1024, 100, False),
    # fewer workers: by workers x rounds, below 40 on chunk tiles 5.3 rounds
    (False, False, 24, 6 * 2048, False), (False, False, 24, 6 * 2048 + 1, True),
    (False, False, 28, 5 * 2048 + 1, False), (False, False, 32, 10854, False),
    (False, False, 32, 10855, True), (False, False, 39, 4 * 2048 + 1, False),
    (False, False, 40, 3 * 2048 + 1, True), (False, False, 40, 3 * 2048, False),
    (False, True, 28, 5 * 2048 + 1, True), (False, True, 28, 5 * 2048, False),
    (False, True, 32, 4 * 2048 + 1, True), (False, True, 23, 30 * 2048, False),
    # fp32 rows: eight rounds
    (True, False, 1024, 7 * 1024, False), (True, False, 64, 7 * 1024 + 1, True),
    (True, False, 56, 7 * 1024 + 1, False), (True, False, 16, 28 * 1024 + 1, True),
    (True, False, 15, 40 * 1024, False),
])
def test_broadcast_auto_pacing(f32, flat, n, tiles, paced):
    assert (rules.write_layout(f32, n, tiles, flat=flat) is not None) == paced
    assert rules.write_layout(f32, n, tiles, flat=flat, mode="always") is not None
