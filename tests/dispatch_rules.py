"""The library's launch arithmetic (csrc/dispatch.h, plain C++) compiled by
itself: which tiles a kernel runs on, and whether and how it is paced."""
import ctypes
import functools
import os
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2507_07114_amd", "csrc")
CUS, TICK_HZ = 256, 1e8  # compute units and clock of the MI355X

SOURCE = r"""
#include "dispatch.h"
using namespace lossy;
static PaceSetting setting(const double* v) {
    return PaceSetting{(int)v[0], v[1], v[2], v[3], (int)v[4], (int)v[5], v[6], v[7], (int)v[8], v[9]};
}
extern "C" {
void defaults(double* v) {
    v[0] = kPaceAuto; v[1] = kDefaultPaceRate; v[2] = kDefaultPaceGapUs;
    v[3] = kDefaultPaceLeadUs; v[4] = kDefaultPaceOverlap; v[5] = kDefaultPaceResident;
    v[6] = kDefaultPaceHeadroom; v[7] = kDefaultPaceTailUs; v[8] = kDefaultPacePersistent;
    v[9] = kDefaultPaceRateF32;
}
void tiles(int f32, int n, int64_t d, int64_t L, int step, int call, int64_t* out) {
    const TileGrid t =
        tile_grid(f32, n, d, (d + L - 1) / L, L, 2, step ? kFewStepRows : 0, (TileCall)call);
    out[0] = t.tiles; out[1] = t.slots;
}
int keeps(int fill, int drift, int64_t tiles, double bytes) {
    return keep_rows(fill ? kKeepFill : drift ? kKeepDrift : kKeepStep, tiles, bytes);
}
int step_layout(const double* st, int f32, int lean, int flat, int per_cu, int n, int fill,
                int drift, int unlike, double grad, double rep, double stale, double in,
                int64_t tiles, int cus, double hz, double* out) {
    PaceTile w;
    w.n = n; w.fill = fill; w.flat = flat; w.drift = drift;
    w.unlike = unlike; w.grad = grad; w.rep = rep; w.stale = stale; w.in = w.out = in;
    PaceParams q;
    int64_t grid;
    uint64_t margin;
    if (!pace_layout(setting(st), f32, lean, per_cu, w, tiles, cus, hz, &q, &grid, &margin))
        return 0;
    const double v[] = {(double)q.per_round, (double)q.round, (double)q.off_g, (double)q.off_r,
                        (double)q.off_s, (double)q.dg, (double)q.dr, (double)q.ds};
    for (int i = 0; i < 8; ++i) out[i] = v[i];
    return 1;
}
int write_layout(const double* st, int f32, int flat, int per_cu, int n, double row, double in,
                 int64_t tiles, int cus, double hz, double* out) {
    SweepParams q;
    uint64_t margin;
    if (!sweep_layout(setting(st), f32, flat, per_cu, n, row, in, tiles, cus, hz, &q, &margin))
        return 0;
    const double v[] = {(double)q.per_round, (double)q.fixed, (double)q.off, (double)q.slot,
                        (double)sweep_spacing(q, q.slot), (double)sweep_spacing(q, 0)};
    for (int i = 0; i < 6; ++i) out[i] = v[i];
    return 1;
}
}
"""

FIELDS = ("mode", "bytes_per_s", "gap_us", "lead_us", "overlap", "resident", "headroom",
          "tail_us", "persistent", "bytes_per_s_f32")
MODES = dict(auto=0, always=1, never=2)


@functools.lru_cache(maxsize=None)
def _lib():
    with tempfile.TemporaryDirectory() as tmp:
        src, out = os.path.join(tmp, "rules.cpp"), os.path.join(tmp, "rules.so")
        with open(src, "w") as f:
            f.write(SOURCE)
        subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror", "-shared",
                        "-fPIC", f"-I{CSRC}", src, "-o", out], check=True)
        return ctypes.CDLL(out)


def _setting(over):
    v = (ctypes.c_double * 10)()
    _lib().defaults(v)
    for k, x in over.items():
        v[FIELDS.index(k)] = MODES[x] if k == "mode" else x
    return v


def _i64(x):
    return ctypes.c_int64(int(x))


def defaults():
    return dict(zip(FIELDS, _setting({})))


def tiles(f32, n, d, L, step=True, fill_only=False, write=False):
    """(tiles, packets of a flat tile or 0 for chunk tiles) of a fused step and
    its drift pass, or (step=False) of an aggregate or (write=True, too) a
    broadcast by itself; fill_only: a step of stale fill without drift."""
    out = (ctypes.c_int64 * 2)()
    _lib().tiles(int(f32), n, _i64(d), _i64(L), int(step), 2 if write else int(fill_only), out)
    return out[0], out[1]


def keeps(tiles, nbytes, fill=False, drift=False):
    """Whether an unpaced call (drift: a drift pass by itself) of so many tiles
    and bytes loads its rows with the plain cache policy."""
    return bool(_lib().keeps(int(fill), int(drift), _i64(tiles), ctypes.c_double(nbytes)))


def step_layout(f32, n, tiles, *, per_cu=5, lean=False, flat=False, fill=False, unlike=False,
                q=0.9, drift=True, vectors=3, **setting):
    """Schedule of a paced step (times in us, rounds in tiles), or None."""
    row = 4096.0
    out = (ctypes.c_double * 8)()
    grad = row * (1.08 * (1 + q) if fill else q) * (2 if unlike else 1)
    ok = _lib().step_layout(_setting(setting), int(f32), int(lean), int(flat), per_cu, n,
                            int(fill), int(drift), int(unlike), ctypes.c_double(grad), ctypes.c_double(row * q),
                            ctypes.c_double(row * (1 - q) if drift else 0.0),
                            ctypes.c_double(row * vectors * (1 if f32 else 2)), _i64(tiles), CUS,
                            ctypes.c_double(TICK_HZ), out)
    if not ok:
        return None
    us = 256.0 * TICK_HZ * 1e-6
    names = ("round", "off_g", "off_r", "off_s", "dg", "dr", "ds")
    return dict(per_round=int(out[0]), **{k: x / us for k, x in zip(names, out[1:])})


def write_layout(f32, n, tiles, *, per_cu=None, flat=False, **setting):
    """Schedule of a paced broadcast, or None (round: time between round starts
    if every row arrives; empty: if none does)."""
    out = (ctypes.c_double * 6)()
    ok = _lib().write_layout(_setting(setting), int(f32), int(flat),
                             per_cu or (16 if f32 else 8), n, ctypes.c_double(4096.0), ctypes.c_double(4096.0 * (1 if f32 else 2)),
                             _i64(tiles), CUS, ctypes.c_double(TICK_HZ), out)
    if not ok:
        return None
    us = 256.0 * TICK_HZ * 1e-6
    names = ("fixed", "off", "slot", "round", "empty")
    return dict(per_round=int(out[0]), **{k: x / us for k, x in zip(names, out[1:])})
