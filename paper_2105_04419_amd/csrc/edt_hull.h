// edt_hull.h -- lower envelopes of long columns, built by bands in LDS.
//
// out(i) = min over v of f(v) + (i - v)^2.  With F(v) = f(v) + v^2 the value
// is i^2 + min over v of F(v) - 2 i v, so the envelope is the lower convex
// hull of the points (v, F(v)), and the minimum at i is taken by the hull
// point whose two edges have slopes around 2 i.  A workgroup holds HC columns
// at a time; a column is split into bands of HB rows, one lane per band:
//
//   1  hull_scan    each lane builds the hull of its band's points (Graham's
//                   scan, left to right) from the rows HullMask lets through;
//   2  hull_merge   the hulls of two neighbouring groups of bands become one
//                   by dropping points at the seam until both sides agree
//                   (log2(bands) levels, one lane per column and pair);
//   3  hull_enter, hull_cover, hull_start: the point in charge of each
//                   band's first output;
//   4  HullCursor   each lane walks its band's outputs from that point on.
//
// A point is one entry, value << 5 | row of its band, kept in the place of
// the column's rows, so a band takes HB entries a column whatever its input.
// Entries of 32 bits hold f itself, entries of 16 bits a distance d <= 2047
// with f = d^2 (half the LDS: two workgroups of 1024 rows on a CU instead of
// one).  F(v) stays below 2^23 for sides up to HULL_NX x HULL_N x HULL_N, so
// the products of a band's scan (row distances below 32) fit 32 bits; those
// between bands are taken in 64 bits.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace edt {

constexpr int HB = 32;             // rows of a band
constexpr int HC = 32;             // columns of a group
constexpr int HULL_N = 1024;       // longest column (32 bands: one 32-bit mask)
constexpr int HULL_NX = 2048;      // longest row in front of the columns
constexpr int32_t HINF = 1 << 29;  // no finite value

// LDS of a group: hull points; per band and column the surviving range
// (first | end << 8), the output from which its points are in charge and the
// band in charge of its first output; per column the bands holding points.
template <class T>
struct HullLds {
    T* st;               // [bands][HB][HC]
    uint16_t* rng;       // [bands][HC]
    uint16_t* enter;     // [bands][HC]
    uint16_t* start;     // [bands][HC]
    uint32_t* nem;       // [HC]
};
__host__ __device__ inline int hull_bands(int n) { return (n + HB - 1) / HB; }
template <class T>
__host__ __device__ inline int hull_lds_bytes(int n) {
    const int nb = hull_bands(n);
    return nb * HB * HC * (int)sizeof(T) + 3 * nb * HC * 2 + HC * 4;
}
template <class T>
__host__ __device__ inline HullLds<T> hull_lds(unsigned char* p, int n) {
    const int nb = hull_bands(n);
    HullLds<T> h;
    h.st = (T*)p;
    h.nem = (uint32_t*)(h.st + nb * HB * HC);
    h.rng = (uint16_t*)(h.nem + HC);
    h.enter = h.rng + nb * HC;
    h.start = h.enter + nb * HC;
    return h;
}

// Lets a kernel take `bytes` of LDS for its envelopes.  The limit belongs to the
// kernel and the whole process: every caller sets the most the kernel can ever
// ask for, so that none lowers it for another.
inline bool hull_allow_lds(const void* kernel, int bytes) {
    return hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes) ==
           hipSuccess;
}

// Product of two signed 24-bit values (one full-rate instruction; the
// compiler falls back to the quarter-rate 32-bit product where it cannot
// prove the ranges).
__host__ __device__ inline int32_t hull_mul(int32_t a, int32_t b) {
#if defined(__HIP_DEVICE_COMPILE__)
    int32_t r;
    asm("v_mul_i32_i24 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
#else
    return a * b;
#endif
}
// a * b <= c * d for signed 24-bit values.
__host__ __device__ inline bool hull_le(int32_t a, int32_t b, int32_t c, int32_t d) {
#if defined(__HIP_DEVICE_COMPILE__)
    int32_t h0, h1;
    asm("v_mul_hi_i32_i24 %0, %1, %2" : "=v"(h0) : "v"(a), "v"(b));
    asm("v_mul_hi_i32_i24 %0, %1, %2" : "=v"(h1) : "v"(c), "v"(d));
    const uint32_t l0 = (uint32_t)hull_mul(a, b), l1 = (uint32_t)hull_mul(c, d);
    return (int64_t)(((uint64_t)(uint32_t)h0 << 32) | l0) <=
           (int64_t)(((uint64_t)(uint32_t)h1 << 32) | l1);
#else
    return (int64_t)a * b <= (int64_t)c * d;
#endif
}
__host__ __device__ inline int hull_top_bit(uint32_t m) { return 31 - __builtin_clz(m); }
__host__ __device__ inline int hull_low_bit(uint32_t m) { return __builtin_ctz(m); }

// f of an entry.
template <class T>
__host__ __device__ inline int32_t hull_f(uint32_t e) {
    const uint32_t x = e >> 5;
    return (int32_t)(sizeof(T) == 2 ? (x & 0x7ffu) * (x & 0x7ffu) : x);
}

// Rows of a band that can matter, taken in order: bit r of the mask is set
// unless row r has no value, lies on or above the segment between its two
// neighbours, is no lower than the next row already at the first output, or
// is still no lower than the row before at the last one.  With the slopes
// D(r) = F(r + 1) - F(r), a parabola is in charge from D(r - 1) / 2 to
// D(r) / 2, so all of it is one comparison of neighbouring slopes clamped to
// the outputs' range.  On the tunnel extent the z pass keeps 9.7 of 32 rows
// (24.5 by the segment rule alone).  F = f + r^2 with r the row of the band,
// HINF without a value and past the band's ends.
struct HullMask {
    int32_t lo, hi;              // slopes that are in charge before / after the outputs
    int32_t Fb = HINF, cp;       // the row before and the clamped slope up to it
    uint32_t bits = 0u;
    // base: the band's first row; outputs first .. last are wanted
    __host__ __device__ HullMask(int base, int first, int last)
        : lo(2 * (first - base)), hi(2 * (last - base) + 1), cp(clamped(0)) {}
    __host__ __device__ int32_t clamped(int32_t D) const {
#if defined(__HIP_DEVICE_COMPILE__)
        int32_t r;                                   // lo < hi: the median
        asm("v_med3_i32 %0, %1, %2, %3" : "=v"(r) : "v"(D), "v"(lo), "v"(hi));
        return r;
#else
        const int32_t d = D < lo ? lo : D;
        return d > hi ? hi : d;
#endif
    }
    // row r with F = Fc decides on row r - 1: bit `at` of bits
    __host__ __device__ void row(int32_t Fc, uint32_t at) {
        const int32_t c = clamped(Fc - Fb);
        bits |= cp < c ? at : 0u;
        cp = c;
        Fb = Fc;
    }
};

// Hull of one band.  Entry r * HC of s holds row r, bit r of m tells whether
// it is a point to look at; hull point k ends up in entry k * HC (never past
// the row that is being read).  Returns their number.  (v1, F1) is the newest
// hull point, (dv, dF) its difference to the one before it; dv = 0, dF = -1
// where there is none, which the test below never drops.
template <class T>
__host__ __device__ inline int hull_scan(T* s, uint32_t m) {
    if (!m) return 0;
    int v1 = hull_low_bit(m);
    m &= m - 1u;
    uint32_t e = s[v1 * HC];
    s[0] = (T)e;
    int32_t F1 = hull_f<T>(e) + hull_mul(v1, v1), dF = -1;
    int dv = 0, p = 0;
    if (m) e = s[hull_low_bit(m) * HC];
    while (m) {
        const int q = hull_low_bit(m);
        const uint32_t eq = e;
        m &= m - 1u;
        // the next point is on its way while this one is tested
        e = s[(m ? hull_low_bit(m) : 0) * HC];
        const int32_t Fq = hull_f<T>(eq) + hull_mul(q, q);
        int32_t A = Fq - F1;
        int b = q - v1;
        while (hull_mul(A, dv) <= hull_mul(dF, b)) {
            v1 -= dv;
            F1 -= dF;
            const bool bottom = p <= HC;             // the new top is the first point
            const uint32_t e0 = s[bottom ? 0 : p - 2 * HC];
            const int v0 = (int)(e0 & (HB - 1));
            const int32_t F0 = hull_f<T>(e0) + v0 * v0;
            p -= HC;
            dv = bottom ? 0 : v1 - v0;
            dF = bottom ? -1 : F1 - F0;
            A = Fq - F1;
            b = q - v1;
        }
        p += HC;
        s[p] = (T)eq;
        dv = b;
        dF = A;
        v1 = q;
        F1 = Fq;
    }
    return p / HC + 1;
}

// A hull point of a column: its row v of the whole column, F = f + v^2.
// `base` is the first row of the band that holds entry e.
struct HullPoint {
    int v;
    int32_t F;
};
template <class T>
__host__ __device__ inline HullPoint hull_decode(uint32_t e, int base) {
    HullPoint p;
    p.v = base + (int)(e & (HB - 1));
    p.F = hull_f<T>(e) + hull_mul(p.v, p.v);
    return p;
}
template <class T>
__host__ __device__ inline HullPoint hull_point(const HullLds<T>& h, int col, int band, int k) {
    return hull_decode<T>(h.st[(band * HB + k) * HC + col], band * HB);
}
// Place of entry k of a band.
__host__ __device__ inline int hull_at(int col, int band, int k) {
    return (band * HB + k) * HC + col;
}
// b lies on or above the segment a - c (a.v < b.v < c.v).
__host__ __device__ inline bool hull_above(const HullPoint& a, const HullPoint& b,
                                           const HullPoint& c) {
    return hull_le(c.F - b.F, b.v - a.v, b.F - a.F, c.v - b.v);
}

// Joins the hulls of the bands in ml (all before those in mr) of one column;
// returns the bands that no longer hold a point (the caller clears them in
// h.nem).  m: the bands of the column that hold points.  l and r are the
// points at the seam, p the one before l, q the one after r; entries are
// walked by their place in h.st, and only a band that runs out looks for the
// next one.
template <class T>
__host__ __device__ inline uint32_t hull_merge(const HullLds<T>& h, int col, uint32_t m, uint32_t ml,
                                               uint32_t mr) {
    ml &= m;
    mr &= m;
    if (!ml || !mr) return 0u;
    int bl = hull_top_bit(ml), br = hull_low_bit(mr);
    const int xl = h.rng[bl * HC + col], xr = h.rng[br * HC + col];
    // places of l and of its band's first point; of r and of its band's last
    int pl = hull_at(col, bl, (xl >> 8) - 1), ll = hull_at(col, bl, xl & 255);
    int pr = hull_at(col, br, xr & 255), lr = hull_at(col, br, (xr >> 8) - 1);
    HullPoint l = hull_decode<T>(h.st[pl], bl * HB), r = hull_decode<T>(h.st[pr], br * HB);
    HullPoint p = l, q = r;
    int pp = 0, pb = 0, lp = 0, pq = 0, qb = 0, lq = 0;
    bool newp = true, newq = true;
    for (;;) {
        if (newp) {
            bool none = false;
            pp = pl - HC;
            pb = bl;
            lp = ll;
            if (pl == ll) {
                const uint32_t rest = ml & ((1u << bl) - 1u);
                none = rest == 0u;
                pp = pl;
                if (!none) {
                    pb = hull_top_bit(rest);
                    const int x = h.rng[pb * HC + col];
                    pp = hull_at(col, pb, (x >> 8) - 1);
                    lp = hull_at(col, pb, x & 255);
                }
            }
            p = hull_decode<T>(h.st[pp], pb * HB);
            p.F += none;                     // p = l, just above it: never drops l
        }
        if (newq) {
            bool none = false;
            pq = pr + HC;
            qb = br;
            lq = lr;
            if (pr == lr) {
                const uint32_t rest = mr & ~((2u << br) - 1u);
                none = rest == 0u;
                pq = pr;
                if (!none) {
                    qb = hull_low_bit(rest);
                    const int x = h.rng[qb * HC + col];
                    pq = hull_at(col, qb, x & 255);
                    lq = hull_at(col, qb, (x >> 8) - 1);
                }
            }
            q = hull_decode<T>(h.st[pq], qb * HB);
            q.F += none;
        }
        newp = hull_above(p, l, r);
        newq = hull_above(l, r, q);
        if (!newp && !newq) break;
        if (newp) {
            pl = pp;
            bl = pb;
            ll = lp;
            l = p;
        }
        if (newq) {
            pr = pq;
            br = qb;
            lr = lq;
            r = q;
        }
    }
    const int b0 = hull_at(col, bl, 0), b1 = hull_at(col, br, 0);
    h.rng[bl * HC + col] = (uint16_t)((ll - b0) / HC | (((pl - b0) / HC + 1) << 8));
    h.rng[br * HC + col] = (uint16_t)((pr - b1) / HC | (((lr - b1) / HC + 1) << 8));
    return (ml & ~((2u << bl) - 1u)) | (mr & ((1u << br) - 1u));
}

// e is no higher than p (p.v < e.v) at output i.
__host__ __device__ inline bool hull_beats(const HullPoint& p, const HullPoint& e, int i) {
    return e.F - p.F <= 2 * hull_mul(i, e.v - p.v);
}

// The output from which the points of `band` are in charge: the least i >= 0
// at which its first point beats the last one before it.  m: the bands of the
// column holding points (this one among them).
template <class T>
__host__ __device__ inline void hull_enter(const HullLds<T>& h, int col, int band, uint32_t m) {
    const uint32_t before = m & ((1u << band) - 1u);
    int i = 0;
    if (before) {
        const int b = hull_top_bit(before);
        const HullPoint p = hull_point(h, col, b, (h.rng[b * HC + col] >> 8) - 1);
        const HullPoint e = hull_point(h, col, band, h.rng[band * HC + col] & 255);
        const int32_t num = e.F - p.F, den = 2 * (e.v - p.v);
        if (num > 0) {
            // the quotient, rounded up; the float one is off by one at most
            i = (int)((float)num / (float)den);
            i += hull_mul(i, den) < num;
            i += hull_mul(i, den) < num;
            i -= hull_mul(i - 1, den) >= num;
        }
    }
    h.enter[band * HC + col] = (uint16_t)(i < 0x7fff ? i : 0x7fff);
}

// Writes `band` down for the bands whose first output its points are in
// charge of.
template <class T>
__host__ __device__ inline void hull_cover(const HullLds<T>& h, int col, int band, int nb,
                                           uint32_t m) {
    const uint32_t after = m & ~((2u << band) - 1u);
    const int s0 = h.enter[band * HC + col];
    const int s1 = after ? (int)h.enter[hull_low_bit(after) * HC + col] : nb * HB;
    const int b1 = (s1 + HB - 1) / HB < nb ? (s1 + HB - 1) / HB : nb;
    for (int b = (s0 + HB - 1) / HB; b < b1; ++b) h.start[b * HC + col] = (uint16_t)band;
}

// Index of the point of `band` in charge of output i, given that one is.
template <class T>
__host__ __device__ inline int hull_start(const HullLds<T>& h, int col, int band, int i) {
    const int x = h.rng[band * HC + col];
    int l = x & 255, r = x >> 8;
    while (r - l > 1) {
        const int k = (l + r) >> 1;
        if (hull_beats(hull_point(h, col, band, k - 1), hull_point(h, col, band, k), i)) l = k;
        else r = k;
    }
    return l;
}

// The points of one column from point k of `band` on, for outputs taken HO at
// a time.  Every point in charge of one of the HO outputs is offered to all of
// them: the lanes of a wave then advance together once or twice per HO rows
// instead of some lane at nearly every row (on the tunnel extent 439 -> 397 us
// in pass y, 463 -> 417 us in pass z).
constexpr int HO = 8;
template <class T>
struct HullCursor {
    int band, at, last;          // place of the next point, and of its band's last one
    uint32_t after;              // bands holding points after `band`
    HullPoint cur, nxt;
    int32_t lead;                // F_nxt - F_cur, kept positive after the last point
    // makes nxt the current point and fetches the one after it
    __host__ __device__ void step(const HullLds<T>& h, int col) {
        cur = nxt;
        bool none = false;
        if (at == last) {
            none = after == 0u;
            if (!none) {
                band = hull_low_bit(after);
                after &= after - 1u;
                const int x = h.rng[band * HC + col];
                at = hull_at(col, band, x & 255);
                last = hull_at(col, band, (x >> 8) - 1);
            }
        } else {
            at += HC;
        }
        nxt = hull_decode<T>(h.st[at], band * HB);
        lead = nxt.F - cur.F + none;
    }
    __host__ __device__ void init(const HullLds<T>& h, int col, uint32_t m, int band0, int k0) {
        band = band0;
        at = hull_at(col, band, k0);
        last = hull_at(col, band, (h.rng[band * HC + col] >> 8) - 1);
        after = m & ~((2u << band) - 1u);
        nxt = hull_decode<T>(h.st[at], band * HB);
        step(h, col);
    }
    // res[u] = min(res[u], value at output i + u)
    __host__ __device__ void take(const HullLds<T>& h, int col, int i, int32_t (&res)[HO]) {
        for (;;) {
            // F + (i + u)(i + u - 2 v) = [F + i (i - 2 v)] + u [2 (i - v)] + u^2
            const int d = i - cur.v;
            int32_t val = cur.F + hull_mul(i, d - cur.v);
#pragma unroll
            for (int u = 0; u < HO; ++u) {
                const int32_t x = val + u * u;
                res[u] = x < res[u] ? x : res[u];
                val += 2 * d;
            }
            // the next point takes over at i + HO or later: done
            if (lead > 2 * hull_mul(i + HO - 1, nxt.v - cur.v)) break;
            step(h, col);
        }
    }
};

// Distance along a row from its record: word = occupancy of 32 consecutive
// voxels, ends = distance at the first | distance at the last << 16 (0xffff:
// the row holds no obstacle).  Any distance of the word follows from the bits
// around it and the two end distances.  >= 0xffff where there is none.
__host__ __device__ inline uint32_t row_distance(uint32_t word, uint32_t ends, int c) {
    const uint32_t lo = word << (31 - c), hi = word >> c;
    const uint32_t dl = lo ? (uint32_t)__builtin_clz(lo) : ~0u;       // one instruction each:
    const uint32_t dr = hi ? (uint32_t)__builtin_ctz(hi) : ~0u;       // all ones without a bit
    const uint32_t e0 = (ends & 0xffffu) + (uint32_t)c, e1 = (ends >> 16) + (uint32_t)(31 - c);
    const uint32_t d = dl < dr ? dl : dr, e = e0 < e1 ? e0 : e1;
    return d < e ? d : e;
}

}  // namespace edt
