// Host arithmetic of the launches: which tiles a kernel runs on, whether and
// how its row accesses are paced.  Plain C++ without HIP, so that it can be
// compiled and checked by itself.
#pragma once

#include <stddef.h>
#include <stdint.h>

namespace lossy {

// ---------------------------------------------------------------------------
// Tiles
// ---------------------------------------------------------------------------
constexpr int kFlatMinPacket = 64;                // a group touches at most two packets
constexpr int64_t kFlatMaxPacket = 1ll << 30;     // 32-bit offsets within a packet

// Most packets that a run of `tile` elements can touch.
constexpr int flat_slots(int tile, int64_t L) {
    return (int)((tile - 2) / L) + 2;
}

constexpr size_t flat_lds_bytes(int ndir, int slots, int n) {
    return (size_t)slots * ((size_t)ndir * ((n + 63) / 64) * 8 + 8);
}

// Tiles of a kernel over fp32 or bf16 rows: chunks of one packet each (cpp per
// packet, slots = 0), or flat tiles (slots > 0) where a packet's chunks would
// start off the 128-byte lines or leave much of a workgroup idle.  A chunk
// tile's masks are wave-uniform, so it is the better one where it is full.
// Measured, chunk tiles against flat ones (us per step, Adam with drift, p =
// 0.1, d and N as given):
//   off the lines (L not a multiple of 64 elements)
//     bf16 N = 64, 16 M  L = 750: 3383 / 882   6000: 879 / 786   8184: 892 / 786
//     bf16 N = 8, 8 M    L = 750: 419 / 97     6000: 85 / 91     20000: 84 / 91
//     broadcast, bf16 N = 32, 8 M              6000: 114 / 92    8184: 122 / 92
//   on the lines, by the share of the threads that a packet's chunks fill
//     bf16 N = 64, 16 M  12%: 5960 / 916  75%: 1021 / 798  87%: 767 / 841 (L =
//                        1792), 799 / 788 (3584)  94%: 775 / -
//     bf16 N = 8, 8 M    12%: 279 / 103   75%: 89 / 92     87%: 86 / 93
//     fp32 N = 64, 8 M   25%: 3102 / 827  87%: 895 / 797   94%: 842 / 800
//     fp32 N = 16, 4 M   25%: 139 / 115   87%: 114 / 115
//     bf16 83% (L = 5120)  N = 8, 8 M: 85 / 92   N = 32: 211 / 216   N = 64, 16 M:
//                        913 / 784
// The share lies at 95% for fp32 rows and at 85% for bf16 rows, 80% below 48
// of them.  A multiple of 8 off the lines stays with chunk tiles below `few`
// rows: 12 in a step (and in the drift pass, whose partials are the step's),
// where little of the time is row traffic, and none in an aggregate or a
// broadcast by itself.  And a multiple of 8 stays with chunk tiles as long as
// they are so few that most run at once: then the time is one tile's, and a
// flat tile's code is the longer one (N = 64 bf16, L = 256: 0.2 M 30 / 49 with
// 782 chunk tiles, 0.8 M 85 / 63 with 3125; N = 16: 20 / 23 and 46 / 27; fp32
// N = 64, whose workgroups are half as large: 31 / 53 and 92 / 97).  Elements of
// 4 bytes are moved one by one well enough for that to hold of other lengths,
// too, while packets are short and there are 36 tiles or fewer, 64 of the shortest
// (fp32 rows, L = 375, 33 K: N = 8 17 / 19, N = 64 42 / 62, N = 96 56 / 88, N = 64
// aggregate 22 / 27, broadcast 13 / 26, drift 31 / 37; L = 511 42 / 55; L = 65, 66 K:
// N = 8 19 / 24, N = 64 45 / 85).  Beyond, steps of bf16 gradients under them (L =
// 375, N = 64: 33 K 60 / 72, 49 K 68 / 60) and an aggregate (L = 100: 33 K 24 / 27, 81
// K 25 / 23) gain on flat tiles, and a drift pass of longer packets (L = 750, 33 K:
// 41 / 36); bf16 rows do at once (L = 333, 33 K: N = 16 35 / 29, N = 64 80 / 77).
// Steps of stale fill without drift (kTileFill), whose flat tiles take two loads
// a row, stay with up to 2560 chunk tiles of bf16 rows that start on the lines (L =
// 256: N = 16, 0.5 M 18.0 / 21.7, N = 49, 0.34 M 27.4 / 41.4, N = 80, 0.46 M 112 / 117;
// L = 512: N = 24, 0.58 M 22.6 / 28.6, N = 94, 0.7 M 158 / 218; L = 1024: N = 24, 1.05 M
// 51.4 / 56.9, N = 20, 1.2 M 29.1 / 28.9, N = 9, 2.3 M 36.6 / 32.3); with drift they
// gain as others do (L = 256, N = 33, 0.65 M 59.7 / 47.4).
// A broadcast (kTileWrite) of few long bf16 rows that start on the lines writes
// them as well from a quarter of a workgroup: chunks of 512 to 1024 elements
// stay for 4 to 23 rows of more than 768 MiB in all (2.2 GB, L = 512: N = 2 890 / 693,
// N = 4 549 / 555, N = 8 440 / 480, N = 16 413 / 457, N = 20 407 / 456, 1.5 GB N = 48 266 /
// 261; L = 1024: N = 4 516 / 541, N = 12 424 / 458, N = 20 419 / 448, 1.5 GB N = 32 278 /
// 273; L = 256, 1.5 GB: N = 8 441 / 334; L = 1536: N = 8 448 / 471, N = 20 440 / 445, 1 GB
// N = 12 205 / 211, N = 20 196 / 190, 0.6 GB N = 12 122 / 124, N = 16 106 / 102).
constexpr int kFewStepRows = 12;
// Elements of a tile: 4 KiB of a row.
constexpr int tile_elems(bool f32_rows) { return f32_rows ? 1024 : 2048; }
enum TileCall { kTileAny, kTileFill, kTileWrite };
struct TileGrid {
    int64_t tiles;
    int cpp, slots;
    size_t lds;  // dynamic LDS of a flat tile
};
inline TileGrid tile_grid(bool f32_rows, int n, int64_t d, int64_t P, int64_t L, int ndir,
                          int few, TileCall call = kTileAny) {
    const int T = tile_elems(f32_rows);
    const int percent = f32_rows ? 95 : (n >= 48 ? 85 : 80);
    const int64_t cpp = (L + T - 1) / T;
    const bool full = L >= kFlatMaxPacket || 100 * L >= percent * cpp * T;
    const bool lines = L % 64 == 0 || (L % 8 == 0 && n < few);
    const int64_t line = f32_rows ? 4096 : (call == kTileFill && L % 64 == 0 ? 2560 : 1024);
    const bool small = L % 8 == 0 ? P * cpp <= line
                                  : f32_rows && L <= T / 2 && d <= (L <= T / 8 ? 64 : 36) * T;
    const bool writes = call == kTileWrite && !f32_rows && n >= 4 && n < 24 && L % 64 == 0 &&
                        L >= 512 && L <= 1024 && 2.0 * n * d > 768.0 * 1048576.0;
    if (L < kFlatMinPacket || L >= kFlatMaxPacket || (full && lines) || small || writes)
        return TileGrid{P * cpp, (int)cpp, 0, 0};
    const int slots = flat_slots(T, L);
    return TileGrid{(d + T - 1) / T, 0, slots, flat_lds_bytes(ndir, slots, n)};
}

// Whether an unpaced call that touches `bytes` in all, on `tiles` tiles, loads
// its rows with the plain cache policy instead of past the caches.  Up to half
// of the 256 MiB memory-side cache a program's rows may still be there, from the
// call or the kernel that wrote them, and plain loads find them sooner.  Streamed
// / plain, us, one set of buffers again and again; three in turn (p = 0.1):
//   steps   bf16 N = 6, 3.1 M (84 MiB) 22.1 / 16.8; 22.2 / 16.9
//           N = 8, 2.5 M (106) 28.0 / 23.7; 30.1 / 23.6   N = 5, 3.3 M (87) 40.2 /
//           40.2; 41.8 / 39.5   fp32 N = 6, 1.6 M (77) 23.6 / 20.3; 24.5 / 20.4
//           flat, N = 3, 5.7 M (109) 33.8 / 30.1; 33.9 / 30.6
//   larger  bf16 N = 3, 8.2 M (157) 70.4 / 66.2; 70.6 / 73.3   N = 12, 2.8 M (163)
//           54.9 / 54.6; 55.9 / 63.8   N = 4, 7.2 M (164) 43.3 / 41.3; 43.5 / 46.0
//   alone   drift bf16 N = 4, 3.9 M (45) 18.8 / 18.6; 19.3 / 18.3, N = 61, 0.2 M (24,
//           396 tiles) 28.7 / 25.6; 34.8 / 31.3, N = 3, 14 M (135) 43.5 / 40.8; 43.6
//           / 45.9   aggregate bf16 N = 4, 6.7 M (77) 24.1 / 22.9; 24.0 / 22.7
// With few tiles, each of many rows, streamed loads come back sooner whatever
// the size: steps N = 71, 0.3 M (159 tiles) 83.9 / 97.4, N = 47, 0.1 M fp32 (98) 25.7
// / 28.7; 25.7 / 32.8, N = 28, 0.5 M fp32 (512) 61.0 / 66.6; aggregate N = 77, 0.4 M
// (193) 74.8 / 87.9; drift N = 81, 0.4 M (217) 73.8 / 87.9.  Stale fill, which
// writes the rows that it reads, gains from fewer tiles and up to more bytes: bf16
// N = 9, 1.5 M (80, 709 tiles) 20.2 / 17.2; 20.6 / 17.9, N = 13, 2.3 M (187) 61.2 /
// 58.3; 63.1 / 58.3, 2.8 M (238) 62.3 / 48.3; 63.4 / 56.2, fp32 N = 55, 0.15 M (96,
// 586) 36.2 / 31.9; 37.2 / 32.3, but bf16 N = 4, 12.5 M (334) 94.1 / 87.3; 94.2 /
// 101.8.
constexpr double kMiB = 1048576.0;
enum KeepCall { kKeepStep, kKeepFill, kKeepDrift };  // (an aggregate alone is as a step)
inline bool keep_rows(KeepCall call, int64_t tiles, double bytes) {
    if (call == kKeepFill) return tiles >= 512 && bytes <= 256.0 * kMiB;
    return tiles >= (call == kKeepDrift ? 256 : 1024) && bytes <= 128.0 * kMiB;
}

// ---------------------------------------------------------------------------
// Pacing
// ---------------------------------------------------------------------------
// Slot schedule of the paced fused step (see ClockPace), times in 1/256
// clock ticks relative to each round's start.
struct PaceParams {
    int64_t per_round;             // workgroups (tiles) per round
    uint64_t round;                // time between round starts
    uint64_t off_g, off_r, off_s;  // gradient, replica and stale-read sweep starts
    uint64_t dg, dr, ds;           // slot lengths of the three sweeps
    uint64_t guard;                // longest wait, ticks
};

// Pacing modes and defaults: the schedule is laid out for kDefaultPaceRate
// bytes/s (kDefaultPaceRateF32 for steps with fp32 replica rows) with
// kDefaultPaceGapUs between the gradient and replica sweeps, and starts
// kPaceMarginUs after the anchor is written.  The rates (rows loaded
// non-temporally; N = 64, means of 20 to 80 steps in a row, the same to 0.2%
// in every run unless marked):
//   bf16 rows, 105 M  6.3e12 4888 us, 6.6e12 4685, 6.7e12 4622, 6.8e12 4560,
//                     6.9e12 4580-4720 (slips), 7.0e12 5300 (never kept)
//   fp32 rows, 48 M   one round streaming: 5.9e12 4696, 6.5e12 4336, 6.7e12
//                     4380 (slips); two: 6.2e12 4497, 6.4e12 4103 with 0.4 of
//                     the allowances, 6.6e12 3983 (25 M: slips)
enum { kPaceAuto = 0, kPaceAlways = 1, kPaceNever = 2 };
constexpr int64_t kPaceMaxRoundTiles = 1024;  // of fp32-row kernels
constexpr double kPaceF32Allowance = 0.4;
constexpr double kPaceFillCost = 1.08;  // time of a stale-fill sweep byte, in plain ones
// fp32 gradients under bf16 replicas: a thread's two loads of a row touch half
// lines each, so such a row is read with the plain policy and keeps 6.0e12 (0.9
// of the rate).  Unpaced, 6.7e12 (not kept), 6.3e12, 6.0e12, us, two cards:
//   with drift     N = 64 8 M 618 / 622 / 592 / 579, 26 M 1966 / 1955 / 1736-1870 /
//                  1788, 60 M 4521 / 4511 / 3972-4102 / 4080;  N = 48 20 M 1175 /
//                  1183 / 1141 / 1080;  N = 32 20 M 814 / 820 / 744-803 / 776
//   without drift  N = 64 60 M 4367 / 4345 / 3915-4052 / 3931;  N = 48 20 M 1128 /
//                  1135 / 1100 / 1030;  N = 32 10.6 M 407 / 422 / 417 / 410
constexpr double kPaceUnlikeRate = 0.9;
// A broadcast by itself, in rates of a step: 7.0e12 (N = 64, 26 M bf16: 511 us,
// 6.7e12 531, 6.0e12 585) and 6.8e12.
constexpr double kPaceWriteRate = 1.045;
constexpr double kPaceWriteRateF32 = 1.0625;
constexpr double kDefaultPaceRate = 6.7e12;
constexpr double kDefaultPaceRateF32 = 6.4e12;
constexpr double kDefaultPaceGapUs = 2.0;
constexpr double kDefaultPaceLeadUs = 4.0;
constexpr int kDefaultPaceOverlap = 1;
constexpr int kDefaultPaceResident = 1;
constexpr double kPaceMarginUs = 3.0;
constexpr double kDefaultPaceTailUs = 3.0;
constexpr int kDefaultPacePersistent = 0;
// Fraction of the resident workgroup places the rounds in flight may fill.
constexpr double kDefaultPaceHeadroom = 1.0;

// How the fused step is paced (process-wide; see ll_set_pacing).
struct PaceSetting {
    int mode;            // 0 auto, 1 always, 2 never
    double bytes_per_s;  // rate the schedule is laid out for
    double gap_us;       // allowance between the last gradient row and the first replica row
    double lead_us;      // allowance from a round's start to its first gradient row
    int overlap;         // rounds streaming at once (1 or 2)
    int resident;        // rounds the resident workgroup places are shared by (>= overlap)
    double headroom;     // fraction of the resident places the rounds may fill
    double tail_us;      // allowance after a round's last slot
    int persistent;      // 1: one round of workgroups loops over the rounds (plain steps)
    double bytes_per_s_f32;  // rate for steps whose replica rows are fp32
};

// Whether the layout of the rounds is left at its defaults.  Those are the
// best of bf16 rows; fp32 rows then take their own (two rounds streaming,
// kPaceF32Allowance of the times).  A setting that differs in any of the five
// is taken as it is for both.
inline bool default_layout(const PaceSetting& st) {
    return st.overlap == kDefaultPaceOverlap && st.resident == kDefaultPaceResident &&
           st.gap_us == kDefaultPaceGapUs && st.lead_us == kDefaultPaceLeadUs &&
           st.tail_us == kDefaultPaceTailUs;
}

// Schedule of a kernel with a single sweep, the broadcast (see SweepPace).
struct SweepParams {
    int64_t per_round;
    uint64_t fixed;        // of a round besides its slots, 1/256 ticks
    uint64_t off;          // first slot after the round's start, 1/256 ticks
    uint64_t slot;         // slot length if every row arrived, 1/256 ticks
    uint64_t vectors;      // time of the vectors' bytes, 1/256 ticks
    uint64_t rows, share;  // rows; rounds that share the places
    uint64_t streams;      // rounds streaming at once
    uint64_t guard;        // ticks
};

// Time between round starts if a row's slot lasts `delta`: no less than the
// round's bytes take at its share of the rate, and enough for its places to be
// free again (as in pace_layout).  Evaluated on the device, where the share of
// arrived rows is known.
constexpr uint64_t sweep_spacing(const SweepParams& q, uint64_t delta) {
    const uint64_t places = (q.fixed + q.rows * delta) / q.share;
    const uint64_t stream = (q.vectors + q.rows * delta) / q.streams;
    return stream > places ? stream : places;
}

// What one tile of a paced kernel is expected to move: bytes per row slot of
// each sweep, and of master and moments before and after the first sweep.
struct PaceTile {
    int n;
    bool fill;    // stale fill
    bool flat;    // flat tiles
    bool drift;   // with drift
    bool unlike;  // fp32 gradients, bf16 replicas
    double grad, rep, stale;
    double in, out;
};

// Whether LL_PACE_AUTO paces a step of n rows in `rounds` rounds.  Many rows
// gain most: unpaced, the chip reads pieces of all of them at once.  Few rounds
// lose the start and the end of the schedule, and few rows make rounds so short
// that the allowances count.  Unpaced / paced, us per step with drift, p = 0.1,
// on three sets of buffers in turn (nothing left in the caches):
//   bf16 rows  N = 96: 4 M (2 rounds) 287 / 277, 8 M (4) 604 / 530
//              N = 64: 3 M (2) 153 / 173, 5.2 M (3) 261 / 261, 8 M (4) 409 / 380,
//                      13 M (6) 776 / 681, 33 M (13) 1757 / 1474, 105 M 5520 / 4622
//              N = 48: 5.2 M (3) 200 / 211, 8 M (4) 310 / 306, 13 M (5) 520 / 471
//              N = 32: 8 M (4) 218 / 230, 13 M (5) 369 / 350, 20 M (8) 578 / 530
//              N = 24: 16 M (7) 351 / 362, 33 M (13) 721 / 715
//              N = 16: 16 M 270 / 287, 100 M 1515 / 1646
//   stale fill, bf16 rows with drift (rounds of 1280 tiles)
//              N = 64: 8 M (4) 617 / 577, 26 M 1856 / 1783
//              N = 48: 5.3 M (3) 308 / 311, 5.6 M (3) 324 / 322, 7 M (3) 401 / 381
//              N = 40: 5.3 M (3) 259 / 268, 5.9 M (3) 286 / 289, 7 M (3) 339 / 330
//              N = 32: 5.3 M (3) 211 / 226, 6 M (3) 237 / 245, 7 M (3) 274 / 276,
//                      7.4 M (3) 301 / 290, 7.9 M (4) 318 / 320, 8.4 M (4) 358 / 332
//              N = 16: 33 M 684 / 767
//   the same without drift (of 1536)
//              N = 48: 7 M (3) 380 / 367
//              N = 36: 6.3 M (3) 263 / 269, 7 M (3) 289 / 289, 7.9 M (3) 336 / 319
//              N = 32: 7 M (3) 259 / 263, 7.4 M (3) 280 / 276, 8 M (3) 306 / 291
//   fp32 rows  N = 64: 4 M (4) 382 / 425, 8 M (8) 802 / 756, 50 M 4725 / 4220
//              N = 32: 8 M (8) 412 / 413, 16 M (16) 844 / 769
//              N = 24: 16 M (16) 598 / 605, 25 M (24) 1035 / 908
//              N = 16: 16 M 425 / 440, 33 M (32) 932 / 856
//              N = 14: 26 M (25) 648 / 619, 60 M 1503 / 1376
//              N = 12: 25.5 M (25) 565 / 546, 33 M 723 / 694, 50 M 1120 / 1030, 80 M
//                      1765 / 1625;  N = 10: 70 M 1335 / 1257
//              N = 8: 33 M 530 / 531, 60 M 962 / 937, 100 M 1485 / 1538
//   stale fill, fp32 rows  N = 32: 16 M 1129 / 1144
// Three rounds of stale fill gain from 115000 row tiles (rows x tiles) on; on
// flat tiles, without drift, for the most part from the start (L = 750: N = 32 5.3
// M 213 / 210, 6.3 M 246 / 257, 7.4 M 295 / 285; N = 40 5.3 M 265 / 250).
// Flat tiles with drift gain nothing at any size: their stale rows are read
// vector by vector, so that the last sweep is no stream (bf16 rows, L = 750: N =
// 32 10 M 319 / 334, 80 M 2357 / 2369; N = 48 6.4 M 273 / 307; N = 64 5 M 284 /
// 314, 13 M 727 / 750, 80 M 4371 / 4493; N = 96 26 M 2119 / 2168; N = 300 5 M
// 1257 / 1337; L = 256, N = 64 16 M 878 / 931; L = 6000 866 / 868; fp32 rows, L =
// 750: N = 16 26 M 756 / 768, N = 64 8 M 832 / 848, 40 M 4126 / 4124).  Without
// drift they gain like chunks for the most part (L = 750: N = 32 10 M 290 / 270,
// N = 64 8 M 416 / 366, 13 M 680 / 698, 80 M 4131 / 4175, N = 96 13 M 1005 / 1035;
// L = 2250, N = 64 16 M 827 / 703; fp32 rows, N = 16 50 M 1399 / 1227).
constexpr int64_t kFillRowTiles = 115000;
inline bool pace_pays(bool f32_rows, const PaceTile& w, int64_t tiles, int64_t rounds) {
    const int n = w.n;
    const bool fill = w.fill;
    if (w.flat && w.drift) return false;
    if (f32_rows)
        return (n >= 48 && rounds >= 8) ||
               (!fill && ((n >= 32 && rounds >= 16) || (n >= 12 && rounds >= 24)));
    return (n >= 64 && rounds >= 3) || (n >= 48 && rounds >= 4) || (n >= 32 && rounds >= 5) ||
           (fill && n >= 32 && rounds >= 3 && (w.flat || n * tiles >= kFillRowTiles));
}

// Whether LL_PACE_AUTO paces a broadcast of `tiles` tiles in rounds of at most
// `places` (masks in memory, p = 0.1, three sets of buffers in turn, unpaced /
// paced, us):
//   bf16 rows  N = 64: 3 M (1 round) 70 / 67, 8 M (2) 178 / 160, 26 M 615 / 511
//              N = 40: 14 M (4) 189 / 189, 18 M (5) 245 / 246, 25 M (6) 368 / 322
//              N = 32: 18 M (5) 196 / 207, 21 M (5.05 rounds) 228 / 239, 22.6 M
//                      (5.4) 268 / 252, 33 M (8) 401 / 359
//              N = 28: 21 M (5.05) 200 / 217, 22.6 M (5.4) 228 / 228, 25 M 268 / 245
//              N = 24: 13 M (4) 106 / 125, 25 M (6.06) 251 / 230, 33 M 310 / 290
//              N = 16: 50 M (12) 335 / 329
//              flat tiles, N = 28: 21 M (5.05) 238 / 227;  N = 32: 270 / 251
//   fp32 rows  N = 64: 8 M (8) 346 / 333, 25 M (24) 1108 / 950
//              N = 48: 10 M (10) 381 / 352
//              N = 32: 8 M (8) 175 / 180, 16 M (16) 340 / 333
//              N = 16: 33 M (32) 407 / 366
// One round of very many bf16 rows gains if a row's slot is longer than the
// wait for it (about 0.1 us, 0.23 us on flat tiles) and all of them outweigh
// the anchor launch and the lead, 12 us:
//   chunks     N = 160: 1 tile 17 / 29, 500 tiles 58 / 59, 818 95 / 86
//              N = 400: 200 57 / 59, 327 96 / 88;  N = 800: 100 57 / 88, 163 92 / 89
//              N = 1024: 127 86 / 108, 195 138 / 123
//   flat       N = 160: 500 75 / 65;  N = 400: 200 81 / 106, 275 123 / 120
//              N = 800: 200 152 / 192, 325 274 / 269;  N = 1024: 253 241 / 244
// An aggregate or a drift pass by itself gains nothing at any rate from 6.0 to
// 7.0e12 (N = 64, 26 M: 624 / 622 and 672 / 690): rows read non-temporally are
// served as well unpaced.
constexpr int kSweepOneRoundRows = 160;
inline bool sweep_pays(bool f32_rows, bool flat, int n, int64_t tiles, int64_t places) {
    const int64_t rounds = (tiles + places - 1) / places;
    if (f32_rows) return n >= 16 && rounds >= 8 && n * rounds >= 450;
    if (rounds < 2)
        return n >= kSweepOneRoundRows &&
               (flat ? tiles >= 272 : tiles >= 160 && n * tiles >= 131072);
    // (5.3 rounds of few rows on chunk tiles: shorter ones are served well
    // unpaced, up to 5.8 TB/s)
    return n >= 64 || (n >= 24 && n * rounds >= 160 &&
                       (flat || n >= 40 || 10 * tiles >= 53 * places));
}

// The schedule of one sweep of writes over n rows of `row` bytes a tile, after
// `in` bytes of vectors; false: unpaced.
inline bool sweep_layout(const PaceSetting& st, bool f32_rows, bool flat, int per_cu, int n,
                         double row, double in, int64_t tiles, int cus, double tick_hz,
                         SweepParams* q, uint64_t* margin) {
    const bool pair = f32_rows && default_layout(st);
    const int k = st.overlap > 1 || pair ? 2 : 1;
    const int res = st.resident < k ? k : st.resident;
    int64_t gmax = (int64_t)(st.headroom * per_cu * cus / res);
    if (f32_rows && gmax > kPaceMaxRoundTiles) gmax = kPaceMaxRoundTiles;
    if (gmax < 1) return false;
    const int64_t rounds = (tiles + gmax - 1) / gmax;
    if (st.mode == kPaceAuto && !sweep_pays(f32_rows, flat, n, tiles, gmax)) return false;
    const int64_t g = (tiles + rounds - 1) / rounds;
    // writes alone keep a higher rate than the step's sweeps of either kind
    const double rate =
        f32_rows ? kPaceWriteRateF32 * st.bytes_per_s_f32 : kPaceWriteRate * st.bytes_per_s;
    const double fp = 256.0 * tick_hz * k / rate;
    const double us = 1e-6 * tick_hz * 256.0 * (pair ? kPaceF32Allowance : 1.0);
    const double slot = g * row * fp;
    const double off = st.lead_us * us + g * in * fp;
    const double fixed = off + st.tail_us * us;
    if (!(fixed + n * slot < 1e15)) return false;
    q->per_round = g;
    q->fixed = (uint64_t)fixed;
    q->off = (uint64_t)off;
    q->slot = (uint64_t)slot;
    q->vectors = (uint64_t)(g * in * fp);
    q->rows = (uint64_t)n;
    q->share = (uint64_t)res;
    q->streams = (uint64_t)k;
    *margin = (uint64_t)(kPaceMarginUs * 1e-6 * tick_hz) + 1;
    q->guard = 2 * ((uint64_t)(fixed + n * slot) >> 8) + 2 * *margin + 1;
    return true;
}

// Lay out the schedule of a paced kernel with `tiles` tiles, `per_cu`
// workgroups of it resident per compute unit, or return false to run it
// unpaced.  `overlap` rounds stream at once, each covering *grid
// adjacent tiles (`resident` rounds fill at most kPaceHeadroom of the
// resident workgroup places; rounds are balanced) and laid out for its
// share, rate / overlap, of the bandwidth.  A round is: a
// lead for the workgroups to start, draw masks and read their master and
// moments; the gradient sweep; the gap for the update and the master and
// moment writes; the replica sweep; the stale-read sweep.  Each sweep's slot
// lasts as long as the rows that slot is expected to move take at the
// round's share.  Rounds start round / overlap apart, so with two in flight
// one round's gradient sweep runs beside the previous round's replica sweep
// and each round's lead, gap and tail are covered by the other's streams.
inline bool pace_layout(const PaceSetting& st, bool f32_rows, bool lean, int per_cu,
                        const PaceTile& w, int64_t tiles, int cus, double tick_hz, PaceParams* q,
                        int64_t* grid, uint64_t* margin) {
    // Rounds of fp32-row kernels hold half of the 2048 places (one row slot
    // streams 4 MiB; rounds of all places were measured slower), so the
    // other half takes the next round while one streams: two rounds stream at
    // once, and since each covers the other's lead, gap and tail, 0.4 of
    // those is enough (unless the caller sets a layout of its own).  Rounds of
    // bf16-row kernels take every place (1280 with drift, 1536 without): two
    // rounds at once fall behind their schedule there.
    const bool pair = f32_rows && !lean && default_layout(st);
    const double rate = f32_rows   ? st.bytes_per_s_f32
                        : w.unlike ? kPaceUnlikeRate * st.bytes_per_s
                                   : st.bytes_per_s;
    const int k = st.overlap > 1 || pair ? 2 : 1;
    const int res = st.resident < k ? k : st.resident;
    int64_t gmax = (int64_t)(st.headroom * per_cu * cus / res);
    if (f32_rows && gmax > kPaceMaxRoundTiles) gmax = kPaceMaxRoundTiles;
    if (gmax < 1) return false;
    const int64_t rounds = (tiles + gmax - 1) / gmax;
    if (st.mode == kPaceAuto && !pace_pays(f32_rows, w, tiles, rounds)) return false;
    const int64_t g = (tiles + rounds - 1) / rounds;
    const double fp = 256.0 * tick_hz * k / rate;             // 1/256 ticks per byte of a round
    const double allow = pair ? kPaceF32Allowance : 1.0;
    const double us = 1e-6 * tick_hz * 256.0 * allow;         // 1/256 ticks per allowed microsecond
    const double n = (double)w.n;
    const double dg = g * w.grad * fp, dr = g * w.rep * fp, ds = g * w.stale * fp;
    const double off_g = st.lead_us * us + g * w.in * fp;
    const double off_r = off_g + n * dg + g * w.out * fp + st.gap_us * us;
    const double off_s = off_r + n * dr;
    // A round's workgroups leave a little after its last slot: the last rows
    // they read must arrive and the drift partial be folded.
    const double length = off_s + n * ds + st.tail_us * us;
    // Rounds start `spacing` apart: no closer than the round's bytes at its
    // share allow with k rounds streaming (stream / k), and far enough apart
    // that a round's workgroups find places when it starts, res rounds
    // sharing the resident places (length / res).  With k = 2 and res = 3
    // the lead, gap and tail of each round are covered by the other rounds'
    // streams.
    const double stream = n * (dg + dr + ds) + g * (w.in + w.out) * fp;
    const double spacing = stream / k > length / res ? stream / k : length / res;
    if (!(length < 1e15)) return false;
    q->per_round = g;
    q->dg = (uint64_t)dg;
    q->dr = (uint64_t)dr;
    q->ds = (uint64_t)ds;
    q->off_g = (uint64_t)off_g;
    q->off_r = (uint64_t)off_r;
    q->off_s = (uint64_t)off_s;
    q->round = (uint64_t)spacing;
    *margin = (uint64_t)(kPaceMarginUs * 1e-6 * tick_hz) + 1;
    q->guard = 2 * ((uint64_t)length >> 8) + 2 * *margin + 1;
    *grid = g;
    return true;
}

}  // namespace lossy
