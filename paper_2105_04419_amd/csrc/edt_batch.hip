// edt_batch.hip -- global transform of many dense maps in one launch.
//
// Every map goes through the same three separable passes as the single-map
// transform (x from the occupancy bytes, then the windowed minimum along y
// and z; d_max <= 64).  Two neighbouring voxels of a row travel together: the
// intermediates are rows of pairs, g1 two distances in 16 bits, g2 two values
// in 32, rows padded to whole groups of four voxels (np pairs a row).
//
// Work items (per map, in map order; maps are ordered largest first):
//   phase 0 (x)  60 words of 32 voxels, in row order
//   phase 1 (y)  64 pair columns (in order of z, x) and 8 lrun rows along y
//   phase 2 (z)  64 pair columns (in order of y, x) and 8 lrun rows along z
// The columns of an item run on over the ends of rows, so no lane is left
// idle at a map's edge, whatever its sides.
// FUSED runs all three phases of all maps in one cooperative persistent
// launch: waves take items from a per-phase queue (chunks of `chunk` items
// through one atomic, or a static stride), and a grid-wide barrier separates
// the phases, so a map's y pass starts only after every x item is written.
// PHASED runs the same schedule as three plain launches, one per phase, each
// a kernel of its own phase only (its own register and LDS footprint; the
// kernel boundary replaces the grid barrier).  PER_MAP launches the phase
// kernels three times per map.
#include <hip/hip_cooperative_groups.h>
#include <hip/hip_runtime.h>
#include <stdlib.h>
#include <string.h>

#include "edt.h"
#include "edt_row.h"
#include "edt_win.h"

namespace {

using namespace edt;

struct MapDev {
    int nx, ny, nz;
    int nby, nbz;            // rows along y / z in eights
    int nw;                  // words of 32 voxels in a row
    int np;                  // pairs in a row of g1 / g2 (even)
    int ps;                  // pairs between rows y, y + 1 of g2
    int64_t occ_off;         // bytes into the occupancy input
    int64_t out_off;         // int32 elements into the output
    int64_t pair_off;        // pairs into g1 ([z][y][pair])
    int64_t pair2_off;       // pairs into g2 ([y][z][pair]; 64 bytes: read as four words)
};

// Pairs from one item of phase 2 to the next along a plane.  The items of
// planes with rows of 32 or more overlap by 20 pairs (at least 31 voxels, as
// at most two row ends of three unused values each lie in them), so that each
// can store whole 128-byte lines (item_z).
__host__ __device__ inline int z_step(const MapDev& m) { return m.nx >= 32 ? 44 : 64; }
__host__ __device__ inline int z_chunks(const MapDev& m) {
    const int cols = m.ny * m.np, step = z_step(m);
    return cols <= 64 ? 1 : 1 + (cols - 64 + step - 1) / step;
}

// Work items of a map per phase.
constexpr int XWORDS = 60;   // words a wave of phase 0 writes (two lanes of context a side)
__host__ __device__ inline int64_t phase_items(const MapDev& m, int phase, int lrun) {
    if (phase == 0) return ((int64_t)m.ny * m.nz * m.nw + XWORDS - 1) / XWORDS;
    if (phase == 1)
        return (((int64_t)m.nz * m.np + 63) / 64) * ((m.nby + lrun - 1) / lrun);
    return (int64_t)z_chunks(m) * ((m.nbz + lrun - 1) / lrun);
}

struct BArgs {
    const MapDev* maps;
    const int32_t* pref;     // [3][n_maps + 1] item prefix sums (phase-major)
    int32_t* queues;         // [3][n_maps + 1] grab counters
    const int32_t* itemmap;  // [3][icap] map of each work item
    int64_t icap;
    const uint8_t* occ;
    int32_t* out;
    uint16_t* g1;            // distances along x, min(d, d_max), a byte per voxel of the pair
    uint32_t* g2;            // two 16-bit values in the window's representation
    int n_maps;
    int dmax, D, M;
    int lrun, chunk, schedule;
};

// Two 8-bit distances (at most 64) to their squares in the window's
// representation.  v_perm gives each half the high byte 0x64 (F16: 0x64nn is
// the binary16 of 1024 + n, exact, so subtracting 1024 leaves n, and n^2 <=
// 1600 is exact) or zero (integer squares <= 4096).
template <bool F16>
__device__ inline uint32_t pair_squares(uint32_t w) {
    const uint32_t x = __builtin_amdgcn_perm(F16 ? 0x64646464u : 0u, w, 0x04010400u);
    if (F16) {
        const h16x2 f = as_h16x2(as_u16x2(x)) - (h16x2){(_Float16)1024, (_Float16)1024};
        return as_u32(as_u16x2(f * f));
    }
    const u16x2 v = as_u16x2(x);
    return as_u32(v * v);
}

// each 16-bit half of t: all ones if its bit 15 is set, else zero.  Written
// as the instruction itself: as plain code the compiler turns the masks into
// per-half compares and selects, three times the work of this one operation.
__device__ inline uint32_t pk_sign_mask(uint32_t t) {
    uint32_t r;
    // op_sel_hi:[0,1]: the high half shifts by the constant's low half too
    asm("v_pk_ashrrev_i16 %0, 15, %1 op_sel_hi:[0,1]" : "=v"(r) : "v"(t));
    return r;
}

// phase 0: distances along x.  One lane per word of 32 voxels of a row, words
// in row order; a distance above 64 does not count, so the two words on either
// side, from the lanes beside, are all the context there is, and a wave's
// outer two lanes a side are context only.  The words of a wave are one run of
// the map's bytes: it is read in aligned 16-byte pieces, which become bits in
// LDS, and each lane cuts its word out of them.  The lane sweeps the word with
// carried distances in packed 16-bit halves, voxels x and x + 16 at once, and
// min(d, d_max), a byte per voxel, goes out through LDS in whole lines.
// (Loads and stores of 32 bytes a lane at any alignment keep the address unit
// busy 90% of the time.)  Bound by memory and issue about equally: 104 us for
// 206 M voxels (1 byte read and 1 written each); a byte load and a ballot per
// row took 185 us.
constexpr int XBITS = 144;                     // 16-bit pieces of a wave's bits
constexpr int XSLICE = XBITS * 2 + 64 * 32;    // LDS bytes of a wave
extern __shared__ __align__(16) unsigned char xlds[];

__device__ inline void item_x(const BArgs& a, const MapDev& m, int li) {
    unsigned char* slice = xlds + (threadIdx.x >> 6) * XSLICE;
    uint16_t* bits = (uint16_t*)slice;
    uint32_t* outw = (uint32_t*)(slice + XBITS * 2);
    const int lane = threadIdx.x & 63;
    const int64_t words = (int64_t)m.ny * m.nz * m.nw;
    const int64_t i0 = (int64_t)li * XWORDS - 2, i = i0 + lane;
    const bool ok = i >= 0 && i < words;
    const int64_t ic = i < 0 ? 0 : (i < words ? i : words - 1);
    const int row = (int)((uint32_t)ic / (uint32_t)m.nw);
    const int w = (int)(ic - (int64_t)row * m.nw);
    const int64_t total = (int64_t)m.ny * m.nz * m.nx;
    const int64_t at = (int64_t)row * m.nx + 32 * w;          // byte of the map
    const uint8_t* map = a.occ + m.occ_off;
    // the wave's bytes start at lane 0's word; rounded down to 16 in memory
    const int64_t at0 = __shfl(at, 0);
    const int head = (int)((uintptr_t)(map + at0) & 15);
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const int c = 64 * k + lane;                          // piece: bytes 16 c - head on
        if (c >= 130) continue;
        const int64_t b = at0 - head + 16 * c;
        uint32_t v = 0u;
        if (b >= 0 && b + 16 <= total) {
            const uint4 q = *(const uint4*)(map + b);
            v = bytes8_bits(q.x, q.y) | (bytes8_bits(q.z, q.w) << 8);
        } else if (b + 16 > 0 && b < total) {                 // an end of the map
            for (int k2 = 0; k2 < 16; ++k2)
                if (b + k2 >= 0 && b + k2 < total && map[b + k2]) v |= 1u << k2;
        }
        bits[c] = (uint16_t)v;
    }
    __builtin_amdgcn_wave_barrier();
    const int bit = (int)(at - at0) + head;
    // (two words of the pieces: copied, since a 32-bit read of 16-bit objects is
    // the compiler's to move in front of their stores)
    uint32_t b32[2];
    __builtin_memcpy(b32, __builtin_assume_aligned(slice + 4 * (bit >> 5), 4), 8);
    const int here = min(32, m.nx - 32 * w);                  // voxels of the word in the row
    uint32_t word = __builtin_amdgcn_alignbit(b32[1], b32[0], bit & 31) &
                    (here == 32 ? ~0u : (1u << here) - 1u);
    if (!ok) word = 0u;
    // words w - 2, w - 1, w + 1, w + 2 of the row (0 past its ends)
    const uint32_t l2 = __shfl_up(word, 2), l1 = __shfl_up(word, 1);
    const uint32_t r1 = __shfl_down(word, 1), r2 = __shfl_down(word, 2);
    // distances from the last voxel before the word back to the nearest
    // obstacle at or before it, and from the first one after it onwards
    constexpr uint32_t FAR = 0x100u;
    const uint32_t pl = w > 0 ? l1 : 0u, pl2 = w > 1 ? l2 : 0u;
    const uint32_t pr = w + 1 < m.nw ? r1 : 0u, pr2 = w + 2 < m.nw ? r2 : 0u;
    const uint32_t L = pl ? (uint32_t)__clz(pl) : (pl2 ? 32u + (uint32_t)__clz(pl2) : FAR);
    const uint32_t R =
        pr ? (uint32_t)__ffs(pr) - 1u : (pr2 ? 32u + (uint32_t)__ffs(pr2) - 1u : FAR);
    // the same from voxel 15 back and from voxel 16 on
    const uint32_t wl = word & 0xffffu, wh = word >> 16;
    const uint32_t L16 = wl ? (uint32_t)__clz(wl) - 16u : L + 16u;
    const uint32_t R16 = wh ? (uint32_t)__ffs(wh) - 1u : R + 16u;
    const u16x2 one = {1, 1};
    const u16x2 dmp = {(unsigned short)a.dmax, (unsigned short)a.dmax};
    uint32_t mk[16];
    u16x2 d[16];
#pragma unroll
    for (int x = 0; x < 16; ++x) {
        // bits x and x + 16 into bit 15 of the two halves: all ones where set
        mk[x] = pk_sign_mask(as_u32(as_u16x2(word) << (u16x2){(unsigned short)(15 - x),
                                                              (unsigned short)(15 - x)}));
    }
    uint32_t c = L | (L16 << 16);
#pragma unroll
    for (int x = 0; x < 16; ++x) {
        c = as_u32(as_u16x2(c) + one) & ~mk[x];
        d[x] = as_u16x2(c);
    }
    c = R16 | (R << 16);
#pragma unroll
    for (int x = 15; x >= 0; --x) {
        c = as_u32(as_u16x2(c) + one) & ~mk[x];
        d[x] = __builtin_elementwise_min(__builtin_elementwise_min(d[x], as_u16x2(c)), dmp);
    }
    // voxels 4 q .. 4 q + 3 from the low halves, 16 more on from the high ones
    uint32_t v[8];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const uint32_t e0 = as_u32(d[4 * q]), e1 = as_u32(d[4 * q + 1]);
        const uint32_t e2 = as_u32(d[4 * q + 2]), e3 = as_u32(d[4 * q + 3]);
        // bytes 0 and 2 of two words: lo0 lo1 hi0 hi1
        const uint32_t p = __builtin_amdgcn_perm(e1, e0, 0x06020400u);
        const uint32_t r = __builtin_amdgcn_perm(e3, e2, 0x06020400u);
        v[q] = (p & 0xffffu) | (r << 16);
        v[q + 4] = (p >> 16) | (r & 0xffff0000u);
    }
    // the row's share of the word, in words of four voxels; the wave's words
    // (lanes 2 .. 61) follow each other in g1
    const bool mine = ok && lane >= 2 && lane < 62;
    const int64_t o = ((m.pair_off + (int64_t)row * m.np) >> 1) + 8 * w;
    const int left = mine ? min(8, m.np / 2 - 8 * w) : 0;
    const int64_t o0 = __shfl(o, 2);
    const int n = (int)min((int64_t)li * XWORDS + XWORDS, words) - 1 - (int)i0;   // last lane
    const int count = (int)(__shfl(o + left, n) - o0);
    uint32_t* lo = outw + (int)(o - o0);
#pragma unroll
    for (int q = 0; q < 8; ++q)
        if (q < left) lo[q] = v[q];
    __builtin_amdgcn_wave_barrier();
    uint32_t* dst = (uint32_t*)a.g1 + o0;
    for (int k = lane; k < count; k += 64) dst[k] = outw[k];
    __builtin_amdgcn_wave_barrier();
}

// Windowed minimum of one pair column per lane, rows first .. first + 8 steps
// - 1 of a column (both values of a pair at once, in packed 16 bits):
//   out(i) = min over |k| <= 8 M - 1 of in(i + k) + k^2.
// load(i, v): rows i .. i + 7 as stored (callers give rows past the column's
// ends d_max or D); conv turns one into the window's representation, Dp is D
// in it; emit(r, acc): outputs of rows r .. r + 7.  Eight outputs a step,
// offsets outward.  The 24 rows within 8 of the outputs stay in registers, the
// next 8 on their way; rows further off are read when some output is still
// larger than the square of their offset, which dense maps seldom need: so the
// radius costs no registers.
//   Nearly empty maps need them at every step.  An item without a value below
// D within its reach is therefore told at its start, from one read of its rows
// (16 empty maps of 128 voxels a side at d_max 64: 309 -> 94 us), and the first
// rows outside the registers are the ones on their way (24 maps of 32 to 256 a
// side at d_max 24 with walls alone 404 -> 386 us, with one obstacle in 2,000
// voxels 451 -> 434).  Remembering such rows one group of eight at a time, inside
// the loop, cost maps with one obstacle in 50 voxels 2 to 4%.
template <bool F16, class Load, class Conv, class Emit>
__device__ inline void column_min(int first, int steps, int M, uint32_t Dp, Load&& load,
                                  Conv&& conv, Emit&& emit) {
    u16x2 P[24];                                 // rows r - 8 .. r + 15
    {
        uint32_t v[3][8];
#pragma unroll
        for (int h = 0; h < 3; ++h) load(first - 8 + 8 * h, v[h]);
#pragma unroll
        for (int q = 0; q < 24; ++q) P[q] = as_u16x2(conv(v[q >> 3][q & 7]));
    }
    // nothing below D in the item's rows and those within the radius of them
    if (M > 1 && !__any(as_u32(min8<F16>(P + 8)) != Dp)) {
        bool away = true;
#pragma unroll 1
        for (int g = -M; g < steps + M && away; ++g) {
            uint32_t v[8];
            u16x2 c[8];
            load(first + 8 * g, v);
#pragma unroll
            for (int u = 0; u < 8; ++u) c[u] = as_u16x2(conv(v[u]));
            away = !__any(as_u32(min8<F16>(c)) != Dp);
        }
        if (away) {
            u16x2 acc[8];
#pragma unroll
            for (int o = 0; o < 8; ++o) acc[o] = as_u16x2(Dp);
#pragma unroll 1
            for (int s = 0; s < steps; ++s) emit(first + 8 * s, acc);
            return;
        }
    }
    // some output is larger than lim (binary16 patterns order like their values)
    auto over = [](u16x2 mx, uint32_t lim) {
        return __any((uint32_t)mx.x > lim || (uint32_t)mx.y > lim) != 0;
    };
    auto bits = [](uint32_t n) -> uint32_t {     // n <= 2048, in the window's representation
        return F16 ? (uint32_t)__builtin_bit_cast(unsigned short, (_Float16)(int)n) : n;
    };
    // offsets t0 .. t1 - 1 (added to 8 G) of the eight outputs: A[8 + o - t]
    // and B[o + t] are the rows at -(8 G + t) and +(8 G + t); sq(t) their
    // squares
    auto offsets = [&](u16x2* acc, const u16x2* A, const u16x2* B, int t0, int t1, auto&& sq) {
#pragma unroll
        for (int t = t0; t < t1; ++t) {
            const uint32_t k2 = sq(t);
            const u16x2 kk = {(unsigned short)k2, (unsigned short)k2};
#pragma unroll
            for (int o = 0; o < 8; ++o) {
                const u16x2 c = __builtin_elementwise_min(A[8 + o - t], B[o + t]);
                if (F16)
                    acc[o] = as_u16x2(__builtin_elementwise_minimum(as_h16x2(acc[o]),
                                                                    as_h16x2(c) + as_h16x2(kk)));
                else
                    acc[o] = __builtin_elementwise_min(acc[o], c + kk);
            }
        }
    };
    for (int s = 0; s < steps; ++s) {
        const int r = first + 8 * s;
        uint32_t N[8];
        load(r + 16, N);
        u16x2 acc[8];
#pragma unroll
        for (int o = 0; o < 8; ++o) acc[o] = P[8 + o];
        auto near2 = [](int t) -> uint32_t { return F16 ? f16_bits(t * t) : (uint32_t)(t * t); };
        offsets(acc, P, P + 8, 1, 4, near2);
        u16x2 mx = max8<F16>(acc);
        if (over(mx, near2(4))) {
            offsets(acc, P, P + 8, 4, 8, near2);
            mx = max8<F16>(acc);
        }
        if (M > 1 && over(mx, near2(8))) {
            u16x2 A[16], B[16];
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                A[q] = P[q];
                B[q] = P[8 + q];
            }
            u16x2 m0 = __builtin_elementwise_min(min8<F16>(P), min8<F16>(P + 16));
#pragma unroll 1
            for (int G = 1; G < M; ++G) {
                uint32_t a8[8], b8[8];
                load(r - 8 * G - 8, a8);
                if (G == 1) {
#pragma unroll
                    for (int u = 0; u < 8; ++u) b8[u] = N[u];
                } else {
                    load(r + 8 * G + 8, b8);
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    A[8 + u] = A[u];
                    B[u] = B[8 + u];
                    A[u] = as_u16x2(conv(a8[u]));
                    B[8 + u] = as_u16x2(conv(b8[u]));
                }
                // no lane can gain when its least row plus (8 G)^2 is no
                // less than its largest output
                const u16x2 m1 = __builtin_elementwise_min(min8<F16>(A), min8<F16>(B + 8));
                u16x2 lb = __builtin_elementwise_min(m0, m1);
                m0 = m1;
                const uint32_t g2 = bits(64u * G * G);
                const u16x2 gg = {(unsigned short)g2, (unsigned short)g2};
                lb = F16 ? as_u16x2(as_h16x2(lb) + as_h16x2(gg)) : lb + gg;
                if (__any(lb.x < mx.x || lb.y < mx.y)) {
                    offsets(acc, A, B, 0, 8,
                            [&](int t) { return bits((uint32_t)((8 * G + t) * (8 * G + t))); });
                    mx = max8<F16>(acc);
                }
                if (G + 1 < M && !over(mx, bits((uint32_t)(64 * (G + 1) * (G + 1))))) break;
            }
        }
        emit(r, acc);
#pragma unroll
        for (int q = 0; q < 16; ++q) P[q] = P[q + 8];
#pragma unroll
        for (int u = 0; u < 8; ++u) P[16 + u] = as_u16x2(conv(N[u]));
    }
}

// Rows i .. i + 7 of a column: row j of this lane at at + j * stride + lane
// (bytes; at and stride are uniform, so a row's address is scalar but for the
// lane's offset), `none` for rows outside 0 .. n - 1.
template <class T>
__device__ inline void load_rows(const char* at, uint32_t stride, uint32_t lane, int i, int n,
                                 uint32_t none, uint32_t (&v)[8]) {
    if (i >= 0 && i + 8 <= n) {
        const char* p = at + (uint32_t)i * stride;
#pragma unroll
        for (int u = 0; u < 8; ++u, p += stride) v[u] = *(const T*)(p + lane);
        return;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        v[u] = none;
        if (i + u >= 0 && i + u < n) v[u] = *(const T*)(at + (uint32_t)(i + u) * stride + lane);
    }
}

// phase 1: g1 -> g2 along y.  Lane = pair column c = (z, pair) in that order.
// g2 is laid out by y first, so that a wave's row is one whole run of 256
// aligned bytes (178 -> 138 us on 206 M voxels against rows in [z][y] order).
template <bool F16>
__device__ inline void item_y(const BArgs& a, const MapDev& m, int li, uint32_t Dp) {
    const int cols = m.nz * m.np, nc = (cols + 63) / 64;
    const int seg = li / nc;
    const int c = min((li - seg * nc) * 64 + (int)(threadIdx.x & 63), cols - 1);
    const int z = (int)((uint32_t)c / (uint32_t)m.np), p = c - z * m.np;
    // offsets of a lane: g1 from the first lane's z on (a map's g1 is below
    // 4 GB), g2 from the item's first pair
    const int z0 = __builtin_amdgcn_readfirstlane(z), c0 = __builtin_amdgcn_readfirstlane(c);
    const char* src = (const char*)(a.g1 + m.pair_off + (int64_t)z0 * m.ny * m.np);
    const uint32_t lane_src = 2u * ((uint32_t)(z - z0) * (uint32_t)(m.ny * m.np) + (uint32_t)p);
    char* dst = (char*)(a.g2 + m.pair2_off + c0);
    const uint32_t lane_dst = 4u * (uint32_t)(c - c0);
    const uint32_t none = (uint32_t)a.dmax * 0x0101u;
    auto load = [&](int i, uint32_t (&v)[8]) {
        load_rows<uint16_t>(src, 2u * m.np, lane_src, i, m.ny, none, v);
    };
    auto conv = [](uint32_t w) { return pair_squares<F16>(w); };
    auto emit = [&](int r, const u16x2* acc) {
        char* d = dst + (int64_t)r * m.ps * 4;
#pragma unroll
        for (int o = 0; o < 8; ++o, d += 4 * (int64_t)m.ps)
            if (r + o < m.ny) *(uint32_t*)(d + lane_dst) = as_u32(acc[o]);
    };
    const int b0 = seg * a.lrun;
    column_min<F16>(8 * b0, min(a.lrun, m.nby - b0), a.M, Dp, load, conv, emit);
}

// phase 2: g2 -> int32 field along z.  Lane = pair column c = (y, pair).
// The planes of the field follow each other at any alignment, and a store
// that covers part of a 128-byte line costs about as much as one that covers
// all of it (a plain fill runs at 3.1 to 3.6 TB/s in unaligned runs of 256 or
// 512 bytes, at 5.4 in aligned ones).  So an item stores, of every plane, the
// lines that start among its own voxels: its last 20 pairs are also the next
// item's first, eight rows go through LDS in the plane's order, and the lanes
// take them from there two by two from the first line's start on: 322 -> 271
// us on 206 M voxels, for 45% more columns to compute.
constexpr int ZROW = 132;                      // LDS halfwords of a row (130, 131: unused pairs)
// (a lane reads up to halfword 31 + 2 * 63 + 1 of its row before it drops what
// lies past the item: 26 past the last row)
static_assert((8 * ZROW + 32) * 2 <= XSLICE, "rows of phase 2");

template <bool F16>
__device__ inline void item_z(const BArgs& a, const MapDev& m, int li, uint32_t Dp) {
    uint16_t* buf = (uint16_t*)(xlds + (threadIdx.x >> 6) * XSLICE);
    const int lane = threadIdx.x & 63;
    const int cols = m.ny * m.np, nc = z_chunks(m), step = z_step(m);
    const int seg = li / nc, k = li - seg * nc;
    const int c = min(k * step + lane, cols - 1);
    const int y = (int)((uint32_t)c / (uint32_t)m.np), x = 2 * (c - y * m.np);
    const int y0 = __builtin_amdgcn_readfirstlane(y);
    const char* src = (const char*)(a.g2 + m.pair2_off + (int64_t)y0 * m.ps);
    const uint32_t lane_src = 4u * ((uint32_t)(y - y0) * (uint32_t)m.ps + (uint32_t)(x >> 1));
    const int plane = m.nx * m.ny;             // 4096^2 at most
    // voxel of the plane behind pair c (the next row's first for unused pairs)
    auto voxel = [&](int pc) {
        const int yy = (int)((uint32_t)pc / (uint32_t)m.np);
        return yy * m.nx + min(2 * (pc - yy * m.np), m.nx);
    };
    const int e = y * m.nx + min(x, m.nx);
    const int e0 = __builtin_amdgcn_readfirstlane(voxel(k * step));
    const int e1 = __builtin_amdgcn_readfirstlane(k + 1 < nc ? voxel((k + 1) * step) : plane);
    const bool lo = k * step + lane < cols && x < m.nx, hi = lo && x + 1 < m.nx;
    uint16_t* plo = buf + (lo ? e - e0 : 130);
    uint16_t* phi = buf + (hi ? e - e0 + 1 : 131);
    int32_t* field = a.out + m.out_off;
    // an item's voxels of a plane: from the first line that starts in it (from
    // its first voxel for a plane's first item, or without lines) to the next
    // item's first
    const uint32_t first = step < 64 && k > 0 ? 31u : 0u;
    const uint32_t last = step < 64 && k + 1 < nc ? 31u : 0u;
    const bool edge = first == 0u || last == 0u;
    const uint32_t place = (uint32_t)((uintptr_t)field >> 2) + (uint32_t)e0;
    const int own = e1 - e0, room = plane - e0;
    auto load = [&](int i, uint32_t (&v)[8]) {
        load_rows<uint32_t>(src, 4u * m.np, lane_src, i, m.nz, Dp, v);
    };
    auto conv = [](uint32_t w) { return w; };
    auto emit = [&](int r, const u16x2* acc) {
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int o = 0; o < 8; ++o) {
            plo[o * ZROW] = acc[o].x;
            phi[o * ZROW] = acc[o].y;
        }
        __builtin_amdgcn_wave_barrier();
        // voxels s .. t - 1 of the item are its own in a plane; `at` is the
        // place in a line of the item's first.  All rows are read before any is
        // stored, so that one wait covers them
        uint32_t at = place + (uint32_t)r * (uint32_t)plane;
        uint32_t v0[8], v1[8];
#pragma unroll
        for (int o = 0; o < 8; ++o) {
            const uint16_t* b = buf + o * ZROW + 2 * lane + ((0u - at - o * plane) & first);
            v0[o] = b[0];
            v1[o] = b[1];
        }
        __builtin_amdgcn_wave_barrier();
        const char* p = (const char*)(field + (int64_t)r * plane + e0);
#pragma unroll
        for (int o = 0; o < 8; ++o, at += plane, p += 4 * (int64_t)plane) {
            if (r + o >= m.nz) break;
            const uint32_t s = (0u - at) & first;
            const int t = min(own + (int)((0u - at - (uint32_t)own) & last), room);
            const int n = t - (int)s;                               // at most 128
            const int32_t v[2] = {F16 ? f16_int(v0[o]) : (int)v0[o],
                                  F16 ? f16_int(v1[o]) : (int)v1[o]};
            char* d = (char*)p + (8u * (uint32_t)lane + 4u * s);
            if (2 * lane + 1 < n) __builtin_memcpy(d, v, 8);
            if (edge)
                if (2 * lane + 1 == n) *(int32_t*)d = v[0];
        }
    };
    const int b0 = seg * a.lrun;
    column_min<F16>(8 * b0, min(a.lrun, m.nbz - b0), a.M, Dp, load, conv, emit);
}

// The item -> map table, the map records and the item offsets are read-only
// while the batch runs, and an item's index is wave-uniform: read through
// the constant address space they become scalar loads, so the map record and
// everything derived from it stay in scalar registers.
template <typename T>
__device__ inline const __attribute__((address_space(4))) T* as_const(const T* p) {
    return (const __attribute__((address_space(4))) T*)p;
}

typedef int i32x4 __attribute__((ext_vector_type(4)));
__device__ inline MapDev load_map(const MapDev* maps, int mi) {
    static_assert(sizeof(MapDev) == 4 * sizeof(i32x4), "map record size");
    const auto* p = as_const((const i32x4*)(maps + mi));
    struct { i32x4 w0, w1, w2, w3; } r = {p[0], p[1], p[2], p[3]};
    return __builtin_bit_cast(MapDev, r);
}

template <bool F16, int PHASE>
__device__ inline void run_item(const BArgs& a, int gi, uint32_t Dp) {
    const int mi = as_const(a.itemmap)[PHASE * a.icap + gi];
    const MapDev m = load_map(a.maps, mi);
    const int li = gi - as_const(a.pref)[PHASE * (a.n_maps + 1) + mi];
    if (PHASE == 0) {
        item_x(a, m, li);
    } else if (PHASE == 1) {
        item_y<F16>(a, m, li, Dp);
    } else {
        item_z<F16>(a, m, li, Dp);
    }
}

// Items [lo, hi) of phase PHASE; one wave per item.  Dynamic schedule: after
// its first, a wave takes `chunk` items per atomic on the phase's counter (cidx); static:
// wave w takes items lo + w, lo + w + nwaves, ...
template <bool F16, int PHASE>
__device__ void run_phase(const BArgs& a, int lo, int hi, int cidx) {
    const int lane = threadIdx.x & 63;
    const int wpb = blockDim.x >> 6;
    // item indices are wave-uniform: kept in scalar registers, so the map
    // record, the item's block coordinates and the row addresses derived
    // from them are scalar too
    const int wid = __builtin_amdgcn_readfirstlane(blockIdx.x * wpb + (threadIdx.x >> 6));
    const int nwaves = gridDim.x * wpb;
    const uint32_t Dw = F16 ? f16_bits((uint32_t)a.D) : (uint32_t)a.D;
    const uint32_t Dp = Dw | (Dw << 16);        // D in the window's representation
    if (a.schedule == 0) {
        // phase 0's items are the smallest: two for each of the others'.  No more
        // than a wave's share at a time, so that few items still reach all
        // waves, and the first chunk of every wave without asking: the counter
        // is one address, and a batch with no more than one chunk a wave leaves
        // it alone
        const int chunk = max(1, min((PHASE == 0 ? 2 : 1) * a.chunk, (hi - lo) / nwaves));
        const int64_t given = (int64_t)nwaves * chunk;
        int64_t base = lo + (int64_t)wid * chunk;
        while (base < hi) {
            const int end = (int)min(base + chunk, (int64_t)hi);
            for (int i = (int)base; i < end; ++i) run_item<F16, PHASE>(a, i, Dp);
            if (given >= hi - lo) break;
            int grab = 0;
            if (lane == 0) grab = atomicAdd(&a.queues[cidx], chunk);
            base = lo + given + __builtin_amdgcn_readfirstlane(grab);   // lane 0's grab
        }
    } else {
        for (int i = lo + wid; i < hi; i += nwaves) run_item<F16, PHASE>(a, i, Dp);
    }
}

// FUSED: phases 0..2 of all maps, grid barrier between phases.
template <bool F16>
__global__ void __launch_bounds__(512) k_batch_fused(BArgs a) {
    namespace cg = cooperative_groups;
    cg::grid_group grid = cg::this_grid();
    const int n = a.n_maps;
    run_phase<F16, 0>(a, a.pref[0], a.pref[n], n);
    grid.sync();
    run_phase<F16, 1>(a, a.pref[n + 1], a.pref[2 * n + 1], 2 * n + 1);
    grid.sync();
    run_phase<F16, 2>(a, a.pref[2 * n + 2], a.pref[3 * n + 2], 3 * n + 2);
}

// PHASED: one phase of all maps (map = -1), PER_MAP: one phase of one map.
template <bool F16, int PHASE>
__global__ void __launch_bounds__(512, 5) k_batch_phase(BArgs a, int map) {
    const int n = a.n_maps;
    const int* pref = a.pref + PHASE * (n + 1);
    if (map < 0) run_phase<F16, PHASE>(a, pref[0], pref[n], PHASE * (n + 1) + n);
    else run_phase<F16, PHASE>(a, pref[map], pref[map + 1], PHASE * (n + 1) + map);
}

// Item prefix sums of the three phases over the maps (processing order), one
// workgroup of 1024 threads: every thread counts one map's items, a scan
// across the workgroup gives the offsets, chunks of 1024 maps carry on.
__global__ void __launch_bounds__(1024) k_batch_prefix(const MapDev* maps, int n, int lrun,
                                                       int32_t* pref) {
    __shared__ int wsum[16][3];
    __shared__ int carry[3];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    if (t < 3) carry[t] = 0;
    __syncthreads();
    for (int i0 = 0; i0 < n; i0 += 1024) {
        const int i = i0 + t;
        int c[3] = {0, 0, 0};
        if (i < n) {
            const MapDev m = maps[i];
            for (int p = 0; p < 3; ++p) c[p] = (int)phase_items(m, p, lrun);
        }
        int incl[3];
#pragma unroll
        for (int p = 0; p < 3; ++p) {
            incl[p] = c[p];
            for (int o = 1; o < 64; o <<= 1) {
                const int v = __shfl_up(incl[p], o);
                if (lane >= o) incl[p] += v;
            }
            if (lane == 63) wsum[w][p] = incl[p];
        }
        __syncthreads();
#pragma unroll
        for (int p = 0; p < 3; ++p) {
            int before = carry[p];
            for (int v = 0; v < w; ++v) before += wsum[v][p];
            if (i < n) pref[p * (n + 1) + i] = before + incl[p] - c[p];
            if (i == n - 1) pref[p * (n + 1) + n] = before + incl[p];
        }
        __syncthreads();
        if (t < 3) {
            int tot = 0;
            for (int v = 0; v < 16; ++v) tot += wsum[v][t];
            carry[t] += tot;
        }
        __syncthreads();
    }
}

// The map of every work item of every phase (one workgroup per map), so an
// item finds its map with one load.
__global__ void k_batch_itemmap(const int32_t* pref, int n, int32_t* itemmap, int64_t icap) {
    const int i = blockIdx.x;
    for (int p = 0; p < 3; ++p) {
        const int lo = pref[p * (n + 1) + i], hi = pref[p * (n + 1) + i + 1];
        for (int k = lo + threadIdx.x; k < hi; k += blockDim.x) itemmap[p * icap + k] = i;
    }
}

__global__ void k_fill_u32(uint32_t* p, int64_t n, uint32_t v) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

int64_t align256(int64_t v) { return (v + 255) & ~(int64_t)255; }

// Two sets of item tables, for the launches over all maps (FUSED, PHASED) and
// for those per map: each kind picks its own run length, and a captured run
// reads its set again at every replay, whatever the other kind has run since.
constexpr int TABLES = 2;

struct BLayout {
    int64_t off_maps, off_pref[TABLES], off_queues, off_itemmap[TABLES], off_g1, off_g2, total;
    int64_t icap;            // item-map entries per phase
};

// Device record of a map whose pairs start at pair_off and pair2_off.
MapDev map_dev(const edt_batch_map& s, int64_t pair_off, int64_t pair2_off) {
    MapDev m = {};
    m.nx = s.nx; m.ny = s.ny; m.nz = s.nz;
    m.nby = (s.ny + 7) / 8; m.nbz = (s.nz + 7) / 8;
    m.nw = (s.nx + 31) / 32;
    m.np = 2 * ((s.nx + 3) / 4);
    m.ps = (m.np * s.nz + 63) & ~63;
    m.occ_off = s.occ_offset;
    m.out_off = s.out_offset;
    m.pair_off = pair_off;
    m.pair2_off = pair2_off;
    return m;
}
int64_t map_pairs(const MapDev& m) { return (((int64_t)m.np * m.ny * m.nz) + 63) & ~(int64_t)63; }
int64_t map_pairs2(const MapDev& m) { return (int64_t)m.ps * m.ny; }

bool blayout(const edt_batch_map* maps, int n, int dmax, BLayout* L) {
    if (!maps || n < 1 || n > (1 << 16) || dmax < 1 || dmax > 64) return false;
    int64_t nb = 0, pairs = 0, pairs2 = 0, ic[3] = {0, 0, 0};
    for (int i = 0; i < n; ++i) {
        const edt_batch_map& m = maps[i];
        if (m.nx < 1 || m.ny < 1 || m.nz < 1 || m.nx > 4096 || m.ny > 4096 || m.nz > 4096)
            return false;
        if (m.occ_offset < 0 || m.out_offset < 0) return false;
        nb += (int64_t)((m.nx + 7) / 8) * ((m.ny + 7) / 8) * ((m.nz + 7) / 8);
        const MapDev d = map_dev(m, 0, 0);
        pairs += map_pairs(d);
        pairs2 += map_pairs2(d);
        for (int p = 0; p < 3; ++p) ic[p] += phase_items(d, p, 1);   // run length 1: the most
    }
    const int64_t icap = ic[0] > ic[1] ? (ic[0] > ic[2] ? ic[0] : ic[2])
                                       : (ic[1] > ic[2] ? ic[1] : ic[2]);
    if (nb > (1ll << 26)) return false;
    int64_t o = 0;
    L->off_maps = o; o += align256((int64_t)n * sizeof(MapDev));
    for (int t = 0; t < TABLES; ++t) {
        L->off_pref[t] = o; o += align256((int64_t)3 * (n + 1) * 4);
        L->off_itemmap[t] = o; o += align256(3 * icap * 4);
    }
    L->off_queues = o; o += align256((int64_t)3 * (n + 1) * 4);
    L->icap = icap;
    L->off_g1 = o; o += align256(pairs * 2);
    L->off_g2 = o; o += align256(pairs2 * 4);
    L->total = o;
    return true;
}

int grid_cap(int64_t work, int cap) {
    int64_t g = work < 1 ? 1 : work;
    return (int)(g > cap ? cap : g);
}

}  // namespace

struct edt_batch {
    int n;
    int dmax;
    BLayout L;
    char* ws;
    MapDev* host_maps;       // in processing order
    int last_lrun[TABLES];   // run length that each set of item tables is for
    int lrun[TABLES][65];    // run length taken for a caller's, per set
    int64_t items[65];       // most items of a phase, per run length
    int cus;
};

namespace {

// Run lengths: the caller's, halved while the items of a launch would leave
// most of the GPU without a wave: a run is walked in order, about 1.5 us per 8
// rows, and two maps of 64 voxels a side have 64 runs of 16 blocks, 512 of one
// (27.8 -> 15.3 us; 5 maps of up to 256: 82 -> 71 us).  A PER_MAP launch has
// one map's items (the mean map's here).  Told once, when the batch is made: a
// walk over 65,536 maps takes the host 79 us.
void run_lengths(edt_batch* b) {
    int64_t runs[65] = {}, zruns[65] = {}, words = 0;
    for (int i = 0; i < b->n; ++i) {
        words += phase_items(b->host_maps[i], 0, 1);
        for (int l = 1; l <= 64; ++l) {
            runs[l] += phase_items(b->host_maps[i], 1, l);
            zruns[l] += phase_items(b->host_maps[i], 2, l);
        }
    }
    for (int l = 1; l <= 64; ++l) {
        const int64_t most = runs[l] > zruns[l] ? runs[l] : zruns[l];
        b->items[l] = most > words ? most : words;
    }
    for (int t = 0; t < TABLES; ++t)
        for (int l = 1; l <= 64; ++l) {
            int e = l;
            while (e > 1 && runs[e] / (t == 0 ? 1 : b->n) < (int64_t)b->cus * 8) e = (e + 1) / 2;
            b->lrun[t][l] = e;
        }
}

// Waves per CU of the fused launch at most, in whole workgroups, and no more of
// them than items: a workgroup costs it two grid barriers.  24 maps of 32 to 256
// voxels a side at d_max 24, one obstacle in 50 voxels, 32 waves asked for in
// workgroups of 4: 20 a CU (what the registers allow) 600 us, 16 545, 12 513, 8
// 527; two maps of 32 a side 280 -> 38.  Workgroups of 8: two a CU are best (64
// maps 663 us; with one 784).
constexpr int FUSED_WAVES = 12;

template <bool F16>
edt_status launch_batch(edt_batch* b, const BArgs& a, int mode, int waves_per_cu, int wg_waves,
                        hipStream_t st) {
    const int bs = 64 * wg_waves;
    const size_t lds = (size_t)wg_waves * XSLICE;      // phases 0 and 2
    if (mode == EDT_BATCH_FUSED) {
        int per_cu = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_batch_fused<F16>, bs, lds) !=
            hipSuccess)
            return EDT_ERR_HIP;
        int wgs_per_cu =
            waves_per_cu > 0 ? (waves_per_cu + wg_waves - 1) / wg_waves : 8 / wg_waves;
        const int most = (FUSED_WAVES + wg_waves - 1) / wg_waves;
        if (wgs_per_cu > most) wgs_per_cu = most;
        if (wgs_per_cu < 1) wgs_per_cu = 1;
        int64_t g = (int64_t)b->cus * (wgs_per_cu < per_cu ? wgs_per_cu : per_cu);
        const int64_t need = (b->items[a.lrun] + wg_waves - 1) / wg_waves;
        if (g > need) g = need;
        if (g < 1) return EDT_ERR_HIP;
        void* args[] = {(void*)&a};
        if (hipLaunchCooperativeKernel((const void*)k_batch_fused<F16>, dim3((unsigned)g), dim3(bs), args,
                                       (unsigned)lds, st) != hipSuccess)
            return EDT_ERR_HIP;
        return EDT_OK;
    }
    const void* kern[3] = {(const void*)k_batch_phase<F16, 0>, (const void*)k_batch_phase<F16, 1>,
                           (const void*)k_batch_phase<F16, 2>};
    const int wpc = waves_per_cu > 0 ? waves_per_cu : 8;
    if (mode == EDT_BATCH_PHASED) {
        // as many waves as the fused launch would have, per phase
        for (int phase = 0; phase < 3; ++phase) {
            int per_cu = 0;
            if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern[phase], bs,
                                                             phase != 1 ? lds : 0) != hipSuccess)
                return EDT_ERR_HIP;
            const int wgs_per_cu = (wpc + wg_waves - 1) / wg_waves;
            const int g = b->cus * (wgs_per_cu < per_cu ? wgs_per_cu : per_cu);
            if (g < 1) return EDT_ERR_HIP;
            int map = -1;
            void* args[] = {(void*)&a, (void*)&map};
            if (hipLaunchKernel(kern[phase], dim3(g), dim3(bs), args, phase != 1 ? lds : 0,
                                st) != hipSuccess)
                return EDT_ERR_HIP;
        }
        return EDT_OK;
    }
    // PER_MAP: three launches per map, each sized to the map's items
    for (int mi = 0; mi < b->n; ++mi) {
        const MapDev& m = b->host_maps[mi];
        for (int phase = 0; phase < 3; ++phase) {
            const int waves = grid_cap(phase_items(m, phase, a.lrun), b->cus * wpc);
            int map = mi;
            void* args[] = {(void*)&a, (void*)&map};
            if (hipLaunchKernel(kern[phase], dim3((waves + wg_waves - 1) / wg_waves), dim3(bs),
                                args, phase != 1 ? lds : 0, st) != hipSuccess)
                return EDT_ERR_HIP;
        }
    }
    return hipGetLastError() == hipSuccess ? EDT_OK : EDT_ERR_HIP;
}

}  // namespace

extern "C" {

int64_t edt_batch_workspace_bytes(const edt_batch_map* maps, int32_t n_maps, int32_t d_max) {
    BLayout L;
    if (!blayout(maps, n_maps, d_max, &L)) return EDT_ERR_ARG;
    return L.total;
}

edt_status edt_batch_create(const edt_batch_map* maps, int32_t n_maps, int32_t d_max, void* d_ws,
                            int64_t ws_bytes, void* stream, edt_batch** out) {
    if (!out) return EDT_ERR_ARG;
    *out = nullptr;
    BLayout L;
    if (!blayout(maps, n_maps, d_max, &L) || !d_ws || ((uintptr_t)d_ws & 255)) return EDT_ERR_ARG;
    if (ws_bytes < L.total) return EDT_ERR_CAPACITY;
    edt_batch* b = (edt_batch*)calloc(1, sizeof(edt_batch));
    if (!b) return EDT_ERR_CAPACITY;
    b->host_maps = (MapDev*)calloc((size_t)n_maps, sizeof(MapDev));
    if (!b->host_maps) {
        free(b);
        return EDT_ERR_CAPACITY;
    }
    b->n = n_maps;
    b->dmax = d_max;
    b->L = L;
    b->ws = (char*)d_ws;
    // processing order: largest map first (longest-processing-time first)
    int* order = (int*)malloc(sizeof(int) * (size_t)n_maps);
    if (!order) {
        free(b->host_maps);
        free(b);
        return EDT_ERR_CAPACITY;
    }
    for (int i = 0; i < n_maps; ++i) order[i] = i;
    for (int i = 1; i < n_maps; ++i) {   // insertion sort by volume, descending
        const int v = order[i];
        const int64_t vol = (int64_t)maps[v].nx * maps[v].ny * maps[v].nz;
        int j = i - 1;
        while (j >= 0 && (int64_t)maps[order[j]].nx * maps[order[j]].ny * maps[order[j]].nz < vol) {
            order[j + 1] = order[j];
            --j;
        }
        order[j + 1] = v;
    }
    int64_t pairs = 0, pairs2 = 0;
    for (int k = 0; k < n_maps; ++k) {
        b->host_maps[k] = map_dev(maps[order[k]], pairs, pairs2);
        pairs += map_pairs(b->host_maps[k]);
        pairs2 += map_pairs2(b->host_maps[k]);
    }
    free(order);
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&b->cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) {
        free(b->host_maps);
        free(b);
        return EDT_ERR_HIP;
    }
    run_lengths(b);
    hipStream_t st = (hipStream_t)stream;
    if (hipMemcpyAsync(b->ws + L.off_maps, b->host_maps, sizeof(MapDev) * (size_t)n_maps,
                       hipMemcpyHostToDevice, st) != hipSuccess) {
        free(b->host_maps);
        free(b);
        return EDT_ERR_HIP;
    }
    if (hipStreamSynchronize(st) != hipSuccess) {   // the host map table may go away now
        free(b->host_maps);
        free(b);
        return EDT_ERR_HIP;
    }
    *out = b;
    return EDT_OK;
}

edt_status edt_batch_destroy(edt_batch* b) {
    if (!b) return EDT_ERR_ARG;
    free(b->host_maps);
    free(b);
    return EDT_OK;
}

edt_status edt_batch_run(edt_batch* b, const uint8_t* d_occ, int32_t* d_out, int32_t mode,
                         const edt_tune* tune, void* stream) {
    if (!b || !d_occ || !d_out) return EDT_ERR_ARG;
    if (mode != EDT_BATCH_FUSED && mode != EDT_BATCH_PER_MAP && mode != EDT_BATCH_PHASED)
        return EDT_ERR_ARG;
    edt_tune t = {8, 8, 4, 0, 4};
    if (tune) t = *tune;
    if (t.wg_waves == 0) t.wg_waves = 4;
    if (t.lrun < 1 || t.lrun > 64 || t.chunk < 1 || t.chunk > 1024 || t.waves_per_cu < 0 ||
        t.waves_per_cu > 64 || (t.schedule != 0 && t.schedule != 1) ||
        (t.wg_waves != 1 && t.wg_waves != 2 && t.wg_waves != 4 && t.wg_waves != 8))
        return EDT_ERR_ARG;
    hipStream_t st = (hipStream_t)stream;
    const BLayout& L = b->L;
    BArgs a;
    a.maps = (const MapDev*)(b->ws + L.off_maps);
    const int table = mode == EDT_BATCH_PER_MAP ? 1 : 0;
    a.pref = (const int32_t*)(b->ws + L.off_pref[table]);
    a.queues = (int32_t*)(b->ws + L.off_queues);
    a.occ = d_occ;
    a.out = d_out;
    a.g1 = (uint16_t*)(b->ws + L.off_g1);
    a.g2 = (uint32_t*)(b->ws + L.off_g2);
    a.n_maps = b->n;
    a.dmax = b->dmax;
    a.D = b->dmax * b->dmax;
    a.M = (b->dmax + 7) / 8;
    a.lrun = b->lrun[table][t.lrun];
    a.chunk = t.chunk;
    a.schedule = t.schedule;
    a.itemmap = (const int32_t*)(b->ws + L.off_itemmap[table]);
    a.icap = L.icap;
    // item offsets and the item -> map table depend on the run length only:
    // rebuilt when it changes for the mode's set; the dynamic schedule's grab counters start at
    // zero on every run
    if (a.lrun != b->last_lrun[table]) {
        hipLaunchKernelGGL(k_batch_prefix, dim3(1), dim3(1024), 0, st, a.maps, b->n, a.lrun,
                           (int32_t*)a.pref);
        hipLaunchKernelGGL(k_batch_itemmap, dim3(b->n), dim3(256), 0, st, a.pref, b->n,
                           (int32_t*)a.itemmap, a.icap);
        b->last_lrun[table] = a.lrun;
    }
    if (t.schedule == 0)
        hipLaunchKernelGGL(k_fill_u32, dim3(1), dim3(256), 0, st, (uint32_t*)a.queues,
                           (int64_t)3 * (b->n + 1), 0u);
    if (hipGetLastError() != hipSuccess) return EDT_ERR_HIP;
    return win_f16(a.M) ? launch_batch<true>(b, a, mode, t.waves_per_cu, t.wg_waves, st)
                        : launch_batch<false>(b, a, mode, t.waves_per_cu, t.wg_waves, st);
}

}  // extern "C"
