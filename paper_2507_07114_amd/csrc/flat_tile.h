// Flat tiles: the geometry of packet lengths that do not fill the chunks of
// one packet.  Building blocks like those of lossy_device.h, with the same
// arithmetic in the same order per element.
#pragma once

#include "lossy_device.h"

namespace lossy {

// ---------------------------------------------------------------------------
// Flat tiles: NT * 8 consecutive elements of the shard whatever packets they
// belong to, for packet lengths that fill a chunk badly (a 750-element packet
// has 94 of 256 threads busy) or leave rows unaligned (1500-byte packets start
// on a 16-byte boundary once in four).  A flat tile starts on a multiple of
// its size, so every access of it is a vector whatever the packet length; its
// masks are kept per packet ("slot"), and a lane takes part in a row by the
// mask of its own packet.  A thread's group of elements may straddle two
// packets: each lane carries an 8-bit element mask per row.
// ---------------------------------------------------------------------------
// Byte offset past the end of every buffer resource of a tile: a load there
// gives zeros and a store is dropped, with no memory access.
constexpr int kBufferPast = 1 << 30;

template <bool SPLIT>
struct Flat {
    static constexpr int Q = SPLIT ? 4 : 2;  // packets a thread's elements can be in
    Chunk<SPLIT> ch;  // k: packet of the tile's first element
    int n, nw;
    int cap;          // slots of the LDS arrays
    int slots;        // packets of this tile
    int off;          // position of the tile's first element in packet k
    // packets of this thread's elements and which of its 8 elements are in
    // each, one byte per q (a tile has at most 33 packets)
    uint32_t slot_bytes, own_bytes;
    __device__ __forceinline__ int slot(int q) const { return (slot_bytes >> (8 * q)) & 0xFFu; }
    __device__ __forceinline__ uint32_t own(int q) const { return (own_bytes >> (8 * q)) & 0xFFu; }
    int first[SPLIT ? 2 : 1], last[SPLIT ? 2 : 1];  // slots of this wavefront's elements
    // value of element j, from one value per slot of the thread
    template <class T>
    __device__ __forceinline__ T pick(const T (&x)[Q], int j) const {
        const int q = SPLIT && j >= 4 ? 2 : 0;
        return ((own_bytes >> (8 * (q + 1) + j)) & 1u) ? x[q + 1] : x[q];
    }
    // the tile in which packet k + s starts keeps its books
    __device__ __forceinline__ bool starts_here(int s) const { return s > 0 || off == 0; }
};

// LDS of a flat tile.
struct FlatLds {
    uint64_t* words;  // [direction][slot][word]
    float* invq;      // [slot] Horvitz-Thompson weight
    uint32_t* sure;   // [slot] 1: no row of the packet can be lost
    __device__ __forceinline__ FlatLds(uint64_t* base, int ndir, int cap, int nw)
        : words(base),
          invq(reinterpret_cast<float*>(base + (size_t)ndir * cap * nw)),
          sure(reinterpret_cast<uint32_t*>(invq + cap)) {}
};

template <int NT, bool SPLIT>
__device__ __forceinline__ Flat<SPLIT> flat_at(int64_t b, int64_t d, int64_t L, int n, int cap) {
    constexpr int G = SPLIT ? 4 : 8;
    Flat<SPLIT> f;
    Chunk<SPLIT>& ch = f.ch;
    ch.c0 = b * (NT * kElems);
    ch.k = ch.c0 / L;
    ch.c = 0;
    const int64_t cv = d - ch.c0;
    ch.cv = cv >= NT * kElems ? NT * kElems : (int)cv;
    ch.lane = (int)threadIdx.x * G;
    ch.hi = ch.lane + (SPLIT ? NT * 4 : 4);
    const int lo_v = ch.cv - ch.lane, hi_v = ch.cv - ch.hi;
    ch.nv = (lo_v <= 0 ? 0 : lo_v >= 4 ? 4 : lo_v) + (hi_v <= 0 ? 0 : hi_v >= 4 ? 4 : hi_v);
    ch.whole = ch.cv % 8 == 0;
    f.n = n;
    f.nw = (n + 63) >> 6;
    f.cap = cap;
    f.off = (int)(ch.c0 - ch.k * L);
    const uint32_t len = (uint32_t)L, off = (uint32_t)f.off;
    f.slots = (int)((off + (uint32_t)ch.cv - 1) / len) + 1;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    f.slot_bytes = f.own_bytes = 0;
#pragma unroll
    for (int h = 0; h < (SPLIT ? 2 : 1); ++h) {
        const int e0 = h ? ch.hi : ch.lane;
        const int valid = ch.cv - e0 <= 0 ? 0 : (ch.cv - e0 >= G ? G : ch.cv - e0);
        const int s = (int)((off + (uint32_t)e0) / len);
        const int in_a = (int)((uint32_t)(s + 1) * len - off) - e0;  // elements left in packet s
        const uint32_t all = (1u << valid) - 1, a = in_a >= G ? all : all & ((1u << in_a) - 1);
        const uint32_t sa = s < f.slots ? s : f.slots - 1;
        const uint32_t sb = s + 1 < f.slots ? s + 1 : f.slots - 1;
        f.slot_bytes |= (sa | (sb << 8)) << (16 * h);
        f.own_bytes |= ((a << (4 * h)) | ((all & ~a) << (4 * h + 8))) << (16 * h);
        const uint32_t w0 = (uint32_t)(wave * 64 * G + (h ? NT * 4 : 0));
        const int first = (int)((off + w0) / len), last = (int)((off + w0 + 64 * G - 1) / len);
        f.first[h] = first < f.slots ? first : f.slots - 1;
        f.last[h] = last < f.slots ? last : f.slots - 1;
    }
    return f;
}

// Masks of the tile's packets into lds.words, like stage_masks.  A wavefront's
// ballot covers 64 rows of one packet or, with few rows, one packet per power
// of two of rows; the directions start on different wavefronts, so that with
// few packets their draws or loads run side by side.
template <int NT, int NDIR, bool SPLIT, class Fetch = NoFetch>
__device__ __forceinline__ void stage_flat(const MaskSource* src, const Flat<SPLIT>& f, int64_t P,
                                           uint64_t step, const int* dirs, uint64_t* words,
                                           const Fetch& fetch = Fetch()) {
    constexpr int NW = NT / 64, B = 4;
    const int n = f.n, nw = f.nw, lane = (int)threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int rows = n > 32 ? 64 : (n > 1 ? 1 << (32 - __builtin_clz((unsigned)n - 1)) : 1);
    const int per = 64 / rows;  // packets per ballot
    const int jobs = nw > 1 ? f.slots * nw : (f.slots + per - 1) / per;
    struct At {
        int slot, i, w;
    };
    auto where = [&](int job) {
        At a;
        if (nw > 1) {
            a.slot = job / nw;
            a.w = job - a.slot * nw;
            a.i = a.w * 64 + lane;
        } else {
            a.slot = job * per + lane / rows;
            a.w = 0;
            a.i = lane & (rows - 1);
        }
        return a;
    };
    auto put = [&](int s, const At& a, bool arrived) {
        const uint64_t word = __ballot(arrived);
        if ((lane & (rows - 1)) == 0 && a.slot < f.slots)
            words[((size_t)s * f.cap + a.slot) * nw + a.w] =
                rows == 64 ? word : (word >> lane) & ((1ull << rows) - 1);
    };
#pragma unroll
    for (int s = 0; s < NDIR; ++s) {
        const MaskSource& m = src[s];
        const int start = (wave + NW - (s * jobs) % NW) % NW;
        auto sure = [&](const At& a) {
            return a.i == m.owner || (m.reliable != nullptr && m.reliable[f.ch.k + a.slot] != 0);
        };
        if (m.draw) {
#pragma unroll 1
            for (int job = start; job < jobs; job += NW) {
                const At a = where(job);
                bool arrived = false;
                if (a.slot < f.slots && a.i < n)
                    arrived = bernoulli_arrived((uint64_t)(f.ch.k + a.slot), (uint64_t)a.i, step,
                                                (uint64_t)dirs[s], m.seed, m.thr) || sure(a);
                put(s, a, arrived);
            }
            if (s == 0) fetch();
        } else {
            for (int job0 = start; job0 < jobs; job0 += NW * B) {
                uint8_t byte[B];
#pragma unroll
                for (int u = 0; u < B; ++u) {
                    const At a = where(job0 + u * NW);
                    const int i = a.i < n ? a.i : n - 1;
                    const int t = a.slot < f.slots ? a.slot : f.slots - 1;
                    byte[u] = m.mem[(int64_t)i * P + f.ch.k + t];
                }
                if (s == 0 && job0 == start) fetch();
#pragma unroll
                for (int u = 0; u < B; ++u) {
                    if (job0 + u * NW >= jobs) break;
                    const At a = where(job0 + u * NW);
                    const bool live = a.slot < f.slots && a.i < n;
                    put(s, a, live && (byte[u] != 0 || sure(a)));
                }
            }
        }
    }
    __syncthreads();
}

// Ascending walk over the rows that some lane of the wavefront takes part in:
// rows whose bit is set or, with INVERT, clear in the mask of a packet of the
// wavefront's elements; row `drop` (or -1) is left out of packets that can be
// lost.  next() gives the row (-1 after the last) and this lane's elements of
// it.  Masks are walked 32 rows at a time: half the registers of a 64-row
// word, and no 64-bit shifts.
template <bool SPLIT, bool INVERT>
struct FlatWalk {
    static constexpr int Q = Flat<SPLIT>::Q;
    const Flat<SPLIT>& f;
    const uint32_t* words;  // [slot][2 * nw] of one direction
    const uint32_t* sure;
    int drop, w;
    uint32_t bits, mine[Q];
    __device__ __forceinline__ uint32_t word(int s, int i) const {
        uint32_t x = words[s * 2 * f.nw + i];
        if (INVERT) {
            x = ~x;
            const int rest = f.n - i * 32;
            if (rest < 32) x &= rest > 0 ? (1u << rest) - 1 : 0u;
        }
        if (drop >= 0 && (drop >> 5) == i && !sure[s]) x &= ~(1u << (drop & 31));
        return x;
    }
    __device__ __forceinline__ void load(int i) {
        w = i;
        uint32_t any = 0;
#pragma unroll
        for (int h = 0; h < (SPLIT ? 2 : 1); ++h)
            for (int s = f.first[h]; s <= f.last[h]; ++s) any |= word(s, i);
        bits = __builtin_amdgcn_readfirstlane(any);
#pragma unroll
        for (int q = 0; q < Q; ++q) mine[q] = word(f.slot(q), i);
    }
    __device__ __forceinline__ FlatWalk(const Flat<SPLIT>& f_, const uint64_t* words_, int drop_,
                                        const uint32_t* sure_)
        : f(f_), words(reinterpret_cast<const uint32_t*>(words_)), sure(sure_), drop(drop_) {
        load(0);
    }
    __device__ __forceinline__ int next(uint32_t& elems) {
        elems = 0;
        while (bits == 0) {
            if ((w + 1) * 32 >= f.n) return -1;
            load(w + 1);
        }
        const int b = __builtin_ctz(bits);
        bits &= bits - 1;
#pragma unroll
        for (int q = 0; q < Q; ++q) elems |= ((mine[q] >> b) & 1u) ? f.own(q) : 0u;
        return w * 32 + b;
    }
};

__device__ __forceinline__ uint32_t elem_bits(float x) { return __float_as_uint(x); }
__device__ __forceinline__ uint32_t elem_bits(uint16_t x) { return x; }

__device__ __forceinline__ void set_raw(const uint32_t (&w)[8], Raw8<F32>& r) {
    r.a = u32x4{w[0], w[1], w[2], w[3]};
    r.b = u32x4{w[4], w[5], w[6], w[7]};
}
__device__ __forceinline__ void set_raw(const uint32_t (&w)[8], Raw8<BF16>& r) {
    r.a = u32x4{w[0] | (w[1] << 16), w[2] | (w[3] << 16), w[4] | (w[5] << 16),
                w[6] | (w[7] << 16)};
}

__device__ __forceinline__ void put_elem(float* p, const Raw8<F32>& r, int j) {
    const uint32_t w[8] = {r.a.x, r.a.y, r.a.z, r.a.w, r.b.x, r.b.y, r.b.z, r.b.w};
    *p = __uint_as_float(w[j]);
}
__device__ __forceinline__ void put_elem(uint16_t* p, const Raw8<BF16>& r, int j) {
    const uint32_t w[4] = {r.a.x, r.a.y, r.a.z, r.a.w};
    *p = (uint16_t)(w[j >> 1] >> (16 * (j & 1)));
}

// All ones where an element is in `elems`, 0 elsewhere, in the layout of r.
__device__ __forceinline__ uint32_t elem_on(uint32_t elems, int j) {
    return 0u - ((elems >> j) & 1u);
}
__device__ __forceinline__ void keep_elems(uint32_t e, Raw8<F32>& r) {
    r.a &= u32x4{elem_on(e, 0), elem_on(e, 1), elem_on(e, 2), elem_on(e, 3)};
    r.b &= u32x4{elem_on(e, 4), elem_on(e, 5), elem_on(e, 6), elem_on(e, 7)};
}
__device__ __forceinline__ uint32_t pair_on(uint32_t e, int j) {
    return (elem_on(e, j) & 0xFFFFu) | (elem_on(e, j + 1) & 0xFFFF0000u);
}
__device__ __forceinline__ void keep_elems(uint32_t e, Raw8<BF16>& r) {
    r.a &= u32x4{pair_on(e, 0), pair_on(e, 2), pair_on(e, 4), pair_on(e, 6)};
}
// some but not all of the 8
__device__ __forceinline__ bool some_elems(uint32_t e) { return e - 1u < 0xFEu; }

__device__ __forceinline__ void merge(const Raw8<F32>& y, Raw8<F32>& x) {
    x.a |= y.a;
    x.b |= y.b;
}
__device__ __forceinline__ void merge(const Raw8<BF16>& y, Raw8<BF16>& x) { x.a |= y.a; }

// Two accesses of a row by every thread (or one, where a thread's 8 elements
// are adjacent and one vector holds them), each at its own byte offset.
template <int POLICY, bool SPLIT>
__device__ __forceinline__ void load_at(__amdgpu_buffer_rsrc_t r, int lo, int hi, Raw8<F32>& x) {
    x.a = __builtin_amdgcn_raw_buffer_load_b128(r, lo, 0, POLICY);
    x.b = __builtin_amdgcn_raw_buffer_load_b128(r, hi, 0, POLICY);
}
template <int POLICY, bool SPLIT>
__device__ __forceinline__ void load_at(__amdgpu_buffer_rsrc_t r, int lo, int hi, Raw8<BF16>& x) {
    if (SPLIT) {
        const u32x2 a = __builtin_amdgcn_raw_buffer_load_b64(r, lo, 0, POLICY);
        const u32x2 b = __builtin_amdgcn_raw_buffer_load_b64(r, hi, 0, POLICY);
        x.a = u32x4{a.x, a.y, b.x, b.y};
    } else {
        x.a = __builtin_amdgcn_raw_buffer_load_b128(r, lo, 0, POLICY);
    }
}
template <int POLICY, bool SPLIT>
__device__ __forceinline__ void store_at(__amdgpu_buffer_rsrc_t r, int lo, int hi,
                                         const Raw8<F32>& x) {
    __builtin_amdgcn_raw_buffer_store_b128(x.a, r, lo, 0, POLICY);
    __builtin_amdgcn_raw_buffer_store_b128(x.b, r, hi, 0, POLICY);
}
template <int POLICY, bool SPLIT>
__device__ __forceinline__ void store_at(__amdgpu_buffer_rsrc_t r, int lo, int hi,
                                         const Raw8<BF16>& x) {
    if (SPLIT) {
        __builtin_amdgcn_raw_buffer_store_b64(u32x2{x.a.x, x.a.y}, r, lo, 0, POLICY);
        __builtin_amdgcn_raw_buffer_store_b64(u32x2{x.a.z, x.a.w}, r, hi, 0, POLICY);
    } else {
        __builtin_amdgcn_raw_buffer_store_b128(x.a, r, lo, 0, POLICY);
    }
}

// Elements `elems` of a row: in whole tiles (W) every vector that holds one of
// them, with its other elements as they are in memory; else those elements
// alone.  What is not loaded reads as 0.
template <class E, bool W, bool STREAM, bool SPLIT>
__device__ __forceinline__ void load_flat(const typename E::T* row, const Chunk<SPLIT>& ch,
                                          uint32_t elems, Raw8<E>& x) {
    if (W) {
        const int es = (int)sizeof(typename E::T);
        const int lo = (SPLIT ? (elems & 0x0Fu) : elems) ? ch.lane * es : kBufferPast;
        const int hi = (SPLIT ? (elems & 0xF0u) : elems) ? ch.hi * es : kBufferPast;
        load_at<row_policy<E, SPLIT, STREAM>(), SPLIT>(chunk_rsrc(row, ch), lo, hi, x);
    } else {
        uint32_t w[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) w[j] = ((elems >> j) & 1u) ? elem_bits(row[ch.at(j)]) : 0u;
        set_raw(w, x);
    }
}

// Writes elements `elems` of a row and no others.
template <class E, bool W, bool SPLIT>
__device__ __forceinline__ void store_flat(typename E::T* row, const Chunk<SPLIT>& ch,
                                           uint32_t elems, const Raw8<E>& x) {
    uint32_t rest = elems;
    if (W) {
        constexpr bool kOne = sizeof(typename E::T) == 2 && !SPLIT;  // one vector per thread
        const int es = (int)sizeof(typename E::T);
        const uint32_t lo_all = kOne ? 0xFFu : 0x0Fu, hi_all = kOne ? 0xFFu : 0xF0u;
        const bool lo = (elems & lo_all) == lo_all, hi = (elems & hi_all) == hi_all;
        store_at<row_policy<E, SPLIT>(), SPLIT>(chunk_rsrc(row, ch), lo ? ch.lane * es : kBufferPast,
                                                hi ? ch.hi * es : kBufferPast, x);
        rest &= ~((lo ? lo_all : 0u) | (hi ? hi_all : 0u));
    }
    if (rest == 0) return;
#pragma unroll
    for (int j = 0; j < 8; ++j)
        if ((rest >> j) & 1u) put_elem(row + ch.at(j), x, j);
}

// stream_rows over the rows of a FlatWalk: use(raw, elems) with what load_flat
// gives for the lane's elements of each row.
template <int D, class E, bool W, bool STREAM, bool SPLIT, class Walk, class PaceFn, class UseFn>
__device__ __forceinline__ void stream_flat(const typename E::T* rows, int64_t ld,
                                            const Chunk<SPLIT>& ch, Walk& walk, const PaceFn& pace,
                                            const UseFn& use) {
    int r[D];
    uint32_t elems[D];
    Raw8<E> b[D];
#pragma unroll
    for (int u = 0; u < D; ++u) r[u] = walk.next(elems[u]);
    if (r[0] < 0) return;
    const int first = r[0];
    // past the last row the ring issues loads of no element
    auto issue = [&](int row, uint32_t e, Raw8<E>& x) {
        const int at = __builtin_amdgcn_readfirstlane(row >= 0 ? row : first);
        load_flat<E, W, STREAM>(rows + (int64_t)at * ld, ch, e, x);
    };
#pragma unroll
    for (int u = 0; u < D; ++u) {
        if (r[u] >= 0) pace(r[u]);
        issue(r[u], elems[u], b[u]);
    }
    for (;;) {
#pragma unroll
        for (int u = 0; u < D; ++u) {
            if (r[u] >= 0) {
                use(b[u], elems[u]);
                r[u] = walk.next(elems[u]);
                if (r[u] >= 0) pace(r[u]);
            }
            issue(r[u], elems[u], b[u]);
        }
        if (r[0] < 0) return;
    }
}

// Rows in flight per thread of a flat tile's sweeps.  Stale rows are few and
// their sweep holds the drift sums, the kernel's most registers: with two rows
// in flight it keeps 4 wavefronts per SIMD (bf16 rows 101 VGPRs, fp32 rows
// 122; with four 117 and 144, 3 per SIMD).  The one tile at a shard's ragged
// end goes row by row.
template <class Pace, bool W>
struct FlatDepth {
    static constexpr int grad = W ? RingDepth<Pace>::grad : 1, stale = W ? 2 : 1;
};

// Horvitz-Thompson weights and sure packets of the tile, by the last
// wavefront; a barrier (stage_flat's) comes before they are read.
template <int NT, bool SPLIT>
__device__ __forceinline__ void flat_weights(const AggVariant& var, uint64_t step, int64_t P,
                                             const Flat<SPLIT>& f, const FlatLds& lds) {
    const int s = (int)threadIdx.x - (NT - 64);
    if (var.kind != kEstHorvitzThompson || s < 0 || s >= f.slots) return;
    const int64_t k = f.ch.k + s;
    const bool sure = var.reliable != nullptr && var.reliable[k] != 0;
    float invq = var.invq;
    if (var.parity_group > 0 && !sure) invq = parity_invq(var, k, P);
    if (var.ge_derived && !sure) invq = ge_invq(var, step, k, P);
    lds.invq[s] = invq;
    lds.sure[s] = sure ? 1u : 0u;
}

template <bool SPLIT>
__device__ __forceinline__ int flat_count(const uint64_t* words, const Flat<SPLIT>& f, int s) {
    int c = 0;
    for (int i = 0; i < f.nw; ++i) c += __popcll(words[(size_t)s * f.nw + i]);
    return c;
}

// aggregate8 over a flat tile: the same sums, each element with the masks and
// weights of its own packet.  `words`: the gradient direction's masks.
template <class E, bool W, bool SPLIT, class Pace>
__device__ __forceinline__ void aggregate_flat(const typename E::T* grads, int64_t ld,
                                               const Flat<SPLIT>& f, const FlatLds& lds, float lam,
                                               const float (&th)[8], const AggVariant& var,
                                               const Pace& pace, float (&g)[8]) {
    constexpr int Q = Flat<SPLIT>::Q;
    constexpr bool kStream = kStreamRows<Pace>;
    const Chunk<SPLIT>& ch = f.ch;
    const uint64_t* words = lds.words;
    const float nf = (float)f.n;
#pragma unroll
    for (int j = 0; j < 8; ++j) g[j] = 0.0f;
    uint32_t all = 0;
#pragma unroll
    for (int q = 0; q < Q; ++q) all |= f.own(q);
    if (var.kind == kEstStaleFill) {
        // every row, arrived elements from grads and lost ones from g_prev;
        // two rows (four loads) in flight, as more cost the whole kernel
        // registers
        constexpr int B = 2;
        typename E::T* prev = reinterpret_cast<typename E::T*>(var.g_prev);
        uint32_t mine[Q];
        const uint32_t* half = reinterpret_cast<const uint32_t*>(words);
        for (int i0 = 0; i0 < f.n; i0 += B) {
            if ((i0 & 31) == 0) {
#pragma unroll
                for (int q = 0; q < Q; ++q)
                    mine[q] = half[f.slot(q) * 2 * f.nw + (i0 >> 5)];
            }
            Raw8<E> x[B], y[B];
            uint32_t here[B];
#pragma unroll
            for (int u = 0; u < B; ++u) {
                const int row = i0 + u < f.n ? i0 + u : i0;
                here[u] = 0;
#pragma unroll
                for (int q = 0; q < Q; ++q)
                    here[u] |= ((mine[q] >> (row & 31)) & 1u) ? f.own(q) : 0u;
                pace.grad(row);
                load_flat<E, W, kStream>(grads + (int64_t)row * ld, ch, here[u], x[u]);
                load_flat<E, W, kStream>(prev + (int64_t)row * ld, ch, all & ~here[u], y[u]);
            }
#pragma unroll
            for (int u = 0; u < B; ++u) {
                if (i0 + u < f.n) {
                    if (some_elems(here[u])) {
                        keep_elems(here[u], x[u]);
                        keep_elems(all & ~here[u], y[u]);
                    }
                    merge(y[u], x[u]);
                    float v[8];
                    unpack(x[u], v);
#pragma unroll
                    for (int j = 0; j < 8; ++j) g[j] += v[j];
                    store_flat<E, W>(prev + (int64_t)(i0 + u) * ld, ch, here[u], x[u]);
                }
            }
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) g[j] = g[j] / nf;
        return;
    }
    const bool ht = var.kind == kEstHorvitzThompson;
    const int owner = ht ? var.owner : -1;
    FlatWalk<SPLIT, false> walk(f, words, owner, lds.sure);
    stream_flat<FlatDepth<Pace, W>::grad, E, W, kStream>(
        grads, ld, ch, walk, [&](int row) { pace.grad(row); },
        [&](Raw8<E>& raw, uint32_t elems) {
            if (W && some_elems(elems)) keep_elems(elems, raw);
            float x[8];
            unpack(raw, x);
#pragma unroll
            for (int j = 0; j < 8; ++j) g[j] += x[j];
        });
    if (ht) {
        float invq[Q];
        bool sure[Q];
        uint32_t lossy = 0;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            invq[q] = lds.invq[f.slot(q)];
            sure[q] = lds.sure[f.slot(q)] != 0;
            if (!sure[q]) lossy |= f.own(q);
        }
        float mine[8] = {0, 0, 0, 0, 0, 0, 0, 0};
        if (owner >= 0) {
            pace.grad(owner);
            Raw8<E> raw;
            load_flat<E, W, kStream>(grads + (int64_t)owner * ld, ch, lossy, raw);
            unpack(raw, mine);
        }
#pragma unroll
        for (int j = 0; j < 8; ++j)
            g[j] = f.pick(sure, j) ? g[j] / nf : (g[j] * f.pick(invq, j) + mine[j]) / nf;
        return;
    }
    int K[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) K[q] = flat_count(words, f, f.slot(q));
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int k = f.pick(K, j);
        g[j] = k > 0 ? g[j] / (float)k : lam * th[j];
    }
}

// The arrived rows' elements of a flat tile take the values r.
template <class R, bool W, bool SPLIT, class PaceFn>
__device__ __forceinline__ void broadcast_flat(typename R::T* reps, int64_t ld,
                                               const Flat<SPLIT>& f, const uint64_t* words,
                                               const Raw8<R>& r, const PaceFn& pace) {
    FlatWalk<SPLIT, false> walk(f, words, -1, nullptr);
    uint32_t elems;
    for (int i = walk.next(elems); i >= 0; i = walk.next(elems)) {
        pace(i);
        const int at = __builtin_amdgcn_readfirstlane(i);
        store_flat<R, W>(reps + (int64_t)at * ld, f.ch, elems, r);
    }
}

}  // namespace lossy
