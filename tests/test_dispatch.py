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
    # other lengths: fp32 rows in very few tiles of short packets
    (True, 64, 36 * 1024, 375, True, False), (True, 64, 36 * 1024 + 1, 375, True, True),
    (True, 64, 33_001, 512 - 1, True, False), (True, 64, 33_001, 512 + 1, True, True),
    (True, 8, 64 * 1024, 100, False, False), (True, 8, 64 * 1024 + 1, 100, False, True),
    (True, 8, 60_000, 129, True, True), (True, 64, 33_001, 63, True, False),
    (False, 64, 33_001, 375, True, True),
])
def test_tiles(f32, n, d, L, step, flat):
    count, slots = rules.tiles(f32, n, d, L, step)
    T = 1024 if f32 else 2048
    P = -(-d // L)
    assert (slots > 0) == flat
    assert count == (-(-d // T) if flat else P * -(-L // T))
    # never more partials than the workspace holds, whatever the tiles
    assert count <= P * -(-L // 1024)


@pytest.mark.parametrize("f32,d,L,flat", [
    (False, 256 * 2560, 256, False), (False, 256 * 2561, 256, True),
    (False, 264 * 1024, 264, False), (False, 264 * 1025, 264, True),  # off the lines
    (False, 750 * 20, 750, True), (True, 256 * 4096, 256, False), (True, 256 * 4097, 256, True),
])
def test_tiles_of_stale_fill_without_drift(f32, d, L, flat):
    count, slots = rules.tiles(f32, 20, d, L, fill_only=True)
    assert (slots > 0) == flat
    assert flat or count == -(-d // L)  # one chunk a packet


@pytest.mark.parametrize("f32,n,d,L,flat", [
    (False, 23, 25_000_000, 512, False), (False, 24, 25_000_000, 512, True),
    (False, 12, 100_000_000, 448, True), (False, 12, 100_000_000, 520, True),
    (False, 12, 100_000_000, 1088, True),
    (False, 16, 3 << 23, 1024, True), (False, 16, (3 << 23) + 1, 1024, False),
    (False, 3, 200_000_000, 1024, True), (False, 4, 200_000_000, 1024, False),
    (True, 12, 100_000_000, 512, True),
])
def test_tiles_of_a_broadcast_of_few_long_rows(f32, n, d, L, flat):
    count, slots = rules.tiles(f32, n, d, L, False, write=True)
    assert (slots > 0) == flat
    assert flat or count == -(-d // L)


def test_rows_kept_by_the_caches():
    half = 128 << 20  # of the 256 MiB memory-side cache
    assert rules.keeps(1024, half) and not rules.keeps(1024, half + 1)
    assert not rules.keeps(1023, 1 << 20)
    assert rules.keeps(256, half, drift=True) and not rules.keeps(255, half, drift=True)
    assert not rules.keeps(256, half + 1, drift=True)
    assert rules.keeps(512, half * 2, fill=True) and not rules.keeps(511, half, fill=True)
    assert not rules.keeps(512, half * 2 + 1, fill=True)


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


# places of a round: 5 workgroups of bf16 rows with drift on each of 256
# compute units, 6 without, 1024 tiles of fp32 rows
@pytest.mark.parametrize("f32,n,tiles,kw,paced", [
    (False, 64, 2 * 1280, {}, False), (False, 64, 2 * 1280 + 1, {}, True),
    (False, 63, 3 * 1280, {}, False), (False, 48, 3 * 1280 + 1, {}, True),
    (False, 47, 4 * 1280, {}, False), (False, 32, 4 * 1280 + 1, {}, True),
    (False, 31, 80 * 1280, {}, False),
    (False, 64, 2 * 1536 + 1, dict(per_cu=6, drift=False), True),
    (True, 48, 7 * 1024, {}, False), (True, 48, 7 * 1024 + 1, {}, True),
    (True, 32, 15 * 1024 + 1, {}, True), (True, 32, 15 * 1024 + 1, dict(fill=True), False),
    (True, 12, 23 * 1024, {}, False), (True, 12, 23 * 1024 + 1, {}, True),
    (True, 11, 99 * 1024, {}, False),
    # stale fill: three rounds, long enough ones
    (False, 32, 2588, dict(fill=True), False), (False, 32, 3593, dict(fill=True), False),
    (False, 32, 3594, dict(fill=True), True), (False, 47, 2561, dict(fill=True), True),
    (False, 44, 2561, dict(fill=True), False), (False, 47, 2560, dict(fill=True), False),
    (False, 32, 3594, dict(fill=True, per_cu=6, drift=False), True),
    (False, 36, 3077, dict(fill=True, per_cu=6, drift=False), False),
    (False, 64, 2561, dict(fill=True), True), (False, 31, 9999, dict(fill=True), False),
    (False, 32, 2561, dict(fill=True, drift=False, flat=True), True),
    # flat tiles: never with drift
    (False, 64, 40_000, dict(flat=True, per_cu=4), False),
    (False, 300, 40_000, dict(flat=True, per_cu=4), False),
    (False, 64, 40_000, dict(flat=True, per_cu=4, fill=True), False),
    (True, 64, 40_000, dict(flat=True, per_cu=8), False),
    (False, 64, 40_000, dict(flat=True, per_cu=5, drift=False), True),
    (True, 16, 40_000, dict(flat=True, per_cu=8, drift=False), True),
])
def test_step_auto_pacing(f32, n, tiles, kw, paced):
    kw = {**(dict(per_cu=8) if f32 else {}), **kw}
    assert (rules.step_layout(f32, n, tiles, **kw) is not None) == paced
    assert rules.step_layout(f32, n, tiles, mode="always", **kw) is not None


def _bytes_us(tiles_bytes, k, rate):
    return tiles_bytes * k / rate * 1e6


@pytest.mark.parametrize("over,k,times", [
    (dict(), 2, (1.6, 0.8, 1.2)),                         # the defaults of fp32 rows
    (dict(headroom=0.9, bytes_per_s_f32=6.0e12), 2, (1.6, 0.8, 1.2)),
    # a layout that the caller sets is taken as it is
    (dict(tail_us=3.001), 1, (4.0, 2.0, 3.001)),
    (dict(lead_us=3.0), 1, (3.0, 2.0, 3.0)),
    (dict(gap_us=0.0), 1, (4.0, 0.0, 3.0)),
    (dict(resident=2), 1, (4.0, 2.0, 3.0)),
    (dict(overlap=2, resident=2), 2, (4.0, 2.0, 3.0)),
])
def test_layout_of_fp32_rows(over, k, times):
    n, tiles, q = 64, 49_152, 0.9
    st = {**rules.defaults(), **over}
    lead, gap, tail = times
    lay = rules.step_layout(True, n, tiles, per_cu=8, q=q, mode="always", **over)
    g, rate = lay["per_round"], st["bytes_per_s_f32"]
    assert g == (1024 if st["headroom"] == 1.0 else -(-tiles // -(-tiles // 921)))
    state = _bytes_us(g * 4096 * 3, k, rate)
    close = lambda a, b: abs(a - b) <= 0.01 + 1e-6 * b  # noqa: E731
    assert close(lay["off_g"], lead + state)
    assert close(lay["dg"], _bytes_us(g * 4096 * q, k, rate))
    assert close(lay["off_r"], lay["off_g"] + n * lay["dg"] + state + gap)
    length = lay["off_s"] + n * lay["ds"] + tail
    assert close(lay["round"], max((length - lead - gap - tail) / k,
                                   length / max(k, int(st["resident"]))))
    sweep = rules.write_layout(True, n, tiles, mode="always", **over)
    state = _bytes_us(sweep["per_round"] * 4096, k, 1.0625 * rate)
    assert close(sweep["off"], lead + state) and close(sweep["fixed"], lead + tail + state)
    assert close(sweep["slot"], _bytes_us(sweep["per_round"] * 4096, k, 1.0625 * rate))


def test_fp32_gradients_under_bf16_replicas_take_a_lower_rate():
    n, tiles = 64, 25_696
    like, unlike = (rules.step_layout(False, n, tiles, unlike=u) for u in (False, True))
    g = like["per_round"]
    assert unlike["per_round"] == g
    assert abs(like["dg"] - _bytes_us(g * 4096 * 0.9, 1, 6.7e12)) < 0.01
    assert abs(unlike["dg"] - _bytes_us(2 * g * 4096 * 0.9, 1, 0.9 * 6.7e12)) < 0.01
    assert abs(unlike["dr"] - like["dr"] / 0.9) < 0.01


def test_layout_of_bf16_and_persistent_rows_is_as_set():
    for over, k in ((dict(), 1), (dict(lead_us=3.0), 1), (dict(overlap=2, resident=2), 2)):
        st = {**rules.defaults(), **over}
        lay = rules.step_layout(False, 64, 25_696, mode="always", **over)
        rate = st["bytes_per_s"]
        assert abs(lay["off_g"] - st["lead_us"]
                   - _bytes_us(lay["per_round"] * 8192 * 3, k, rate)) < 0.01
    lean = rules.step_layout(True, 64, 49_152, per_cu=4, lean=True, mode="always", persistent=1)
    assert abs(lean["off_g"] - 4.0 - _bytes_us(lean["per_round"] * 4096 * 3, 1, 6.4e12)) < 0.01


@pytest.mark.parametrize("f32", [False, True])
@pytest.mark.parametrize("over", [dict(), dict(resident=2), dict(resident=4),
                                  dict(overlap=2, resident=2), dict(overlap=2, resident=4),
                                  dict(tail_us=0.0, lead_us=0.0)])
def test_broadcast_never_asks_for_more_than_its_rate(f32, over):
    # the bytes of a round, over the time between round starts, against the rate
    n, tiles = 64, 24_000
    lay = rules.write_layout(f32, n, tiles, mode="always", **over)
    rate = 1.0625 * 6.4e12 if f32 else 1.045 * 6.7e12
    row, vec = 4096, 4096 * (1 if f32 else 2)
    asked = lay["per_round"] * (n * row + vec) / (lay["round"] * 1e-6)
    assert asked <= rate * (1 + 1e-3)  # slots are whole 1/256 ticks
    assert lay["empty"] >= lay["per_round"] * vec / rate * 1e6 * (1 - 1e-3)
