// edt_kernels.hip -- HIP kernels of the exact truncated EDT for gfx950.
//
// Global transform (the field of Eq. 1, section III, limited to d_max):
//   ingest          dense grid or leaf-block list -> occupancy bits + hash
//   tile dilation   region = obstacle blocks grown by R blocks (per tile)
//   items (y,z)     runs of consecutive region blocks, at most LRUN long
//   pass_x          g1 = squared distance along x, from the occupancy bits
//   pass_y          g2(y) = min_j g1(y+j) + j^2
//   pass_z          s(z)  = min(D, min_k g2(z+k) + k^2)
// The squared Euclidean distance splits into per-axis terms, so the three
// passes give exactly Eq. 1; terms with an axis offset beyond d_max exceed D
// and never change the clamped result.  For d_max <= 64 the y and z passes
// take the windowed minimum directly, branch-free on packed 16-bit pairs;
// for larger radii they follow the lower envelope of parabolas (Felzenszwalb
// & Huttenlocher, cited by the paper as the global transform), built by bands
// of 32 rows in LDS (edt_hull.h).
//
// Incremental transform (Algorithm 1's raise and lower waves, at block
// granularity): changed voxels are the wave centres; a block is on the lower
// front if some added voxel is closer to the block than its largest value,
// and on the raise front if some removed voxel is no farther than its largest
// value (only such blocks can change); the g1/g2 intermediates are kept
// current for every block and the marked blocks are recomputed exactly.
#include "edt_dev.h"
#include "edt_hull.h"
#include "edt_row.h"
#include "edt_win.h"

namespace edt {

// ---------------------------------------------------------------------------
// small utility kernels
// ---------------------------------------------------------------------------
__global__ void k_fill_u64(unsigned long long* p, int64_t n, unsigned long long v) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}
__global__ void k_fill_i32(int32_t* p, int64_t n, int32_t v) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

// Global transform start: empty block table, counters reset (the error word
// is kept until it is read).
__global__ void k_begin_global(Grid g, int64_t tcap) {
    const int64_t tid = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = tid; i < tcap; i += stride) g.tkeys[i] = KEY_EMPTY;
    int4* ts = (int4*)g.tslots;
    for (int64_t i = tid; i < tcap * 128; i += stride) ts[i] = make_int4(-1, -1, -1, -1);
    for (int64_t i = tid; i < tcap * 16; i += stride) g.tobst[i] = 0u;
    for (int64_t i = tid; i < tcap; i += stride) g.tflag[i] = 0;
    if (tid < C_N && tid != C_ERR) g.cnt[tid] = 0;
}

// Every tile within ceil(R / 8) tiles of an obstacle tile must exist before
// the dilation.  Called by a whole wave: for each lane whose block is the
// first obstacle block of its tile (tile coordinates tx, ty, tz), the wave
// inserts the tile's neighbours, one neighbour per lane.  The trigger is the
// tile's first obstacle, not the tile's creation: a tile may already exist
// as the neighbour of another obstacle tile.
__device__ inline void grow_tiles(const Grid& g, bool first, int tx, int ty, int tz) {
    unsigned long long m = __ballot(first);
    if (m == 0ull) return;
    const int TR = (g.R + 7) >> 3, w = 2 * TR + 1, w3 = w * w * w;
    const int ntx = (g.nbx + 7) >> 3, nty = (g.nby + 7) >> 3, ntz = (g.nbz + 7) >> 3;
    const int lane = __lane_id();
    while (m) {
        const int src = __ffsll((long long)m) - 1;
        m &= m - 1ull;
        const int cx = __shfl(tx, src), cy = __shfl(ty, src), cz = __shfl(tz, src);
        for (int o0 = 0; o0 < w3; o0 += 64) {
            const int o = o0 + lane;
            bool tnew = false;
            int32_t t = -1;
            if (o < w3 && o != w3 / 2) {
                const int ax = cx + o % w - TR, ay = cy + (o / w) % w - TR, az = cz + o / (w * w) - TR;
                if (ax >= 0 && ay >= 0 && az >= 0 && ax < ntx && ay < nty && az < ntz) {
                    t = hinsert(g.tkeys, g.tmask, pack_key(ax, ay, az), &tnew);
                    if (t < 0) set_error(g, -3 /* EDT_ERR_CAPACITY */);
                }
            }
            const int j = wave_append(tnew, &g.cnt[C_NTILE]);
            if (tnew) g.tlist[j] = t;
        }
    }
}

// Pool slots for the lanes that just created a block at tile entry e: one
// counter atomic per wave.  Returns the slot, or -1 (not created / pool full).
__device__ inline int32_t claim_slots(const Grid& g, bool created, int64_t e,
                                      unsigned long long key, uint32_t flags) {
    const int idx = wave_append(created, &g.cnt[C_NBLK]);
    if (!created) return -1;
    if (idx >= g.max_blocks) {
        g.tslots[e] = -1;
        set_error(g, -3 /* EDT_ERR_CAPACITY */);
        g.cnt[C_ABORT] = 1;
        return -1;
    }
    g.bkey[idx] = key;
    g.flags[idx] = flags;
    g.tslots[e] = idx;
    return idx;
}

// ---------------------------------------------------------------------------
// ingest
// ---------------------------------------------------------------------------
// Workgroup b of a one-dimensional grid over an (nxb, nyb, nzb) box of
// blocks (a 3-D grid would cap y and z at 65535 workgroups).
__device__ inline void block_of(int nxb, int nyb, int& bx, int& by, int& bz) {
    const int64_t b = blockIdx.x;
    bx = (int)(b % nxb);
    const int64_t r = b / nxb;
    by = (int)(r % nyb);
    bz = (int)(r / nyb);
}

// Dense grid.  One wave per strip of 8 blocks along x; lane = row (y + 8z).
// Each lane reads 64 contiguous bytes of its row, packs 8 bits per block and
// the wave ballot decides whether a block holds any obstacle.  A workgroup
// takes four strips next to each other along y: they lie in one tile, where
// their 32 blocks are one word of the obstacle mask, and no other workgroup
// holds them; so it finds or creates the tile once, stores the word, and takes
// the slots with one atomic.  (One atomic per lane and address kept 600 strips
// of 203 x 117 x 75 waiting: 24 us, now 8.)
__global__ void __launch_bounds__(256) k_ingest_dense(Grid g, const uint8_t* __restrict__ occ) {
    __shared__ uint32_t word;                 // blocks holding an obstacle, byte = strip
    __shared__ int32_t tile, first_slot;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int sx, byq, bz;
    block_of((g.nbx + 7) / 8, (g.nby + 3) / 4, sx, byq, bz);
    const int by = 4 * byq + w;
    const int bx0 = sx * 8;
    if (threadIdx.x == 0) word = 0u;
    __syncthreads();
    const int y = 8 * by + (lane & 7), z = 8 * bz + (lane >> 3);
    const int x0 = 8 * bx0;
    uint32_t bytes[8];
    const bool row_ok = (y < g.ny) && (z < g.nz);
    const uint8_t* row = occ + ((int64_t)z * g.ny + y) * (int64_t)g.nx;
    // 64 voxels in two words (16-byte loads at any alignment)
    uint32_t w0 = 0u, w1 = 0u;
    if (row_ok) {
        w0 = row_word(row, g.nx, 2 * sx);
        if (x0 + 32 < g.nx) w1 = row_word(row, g.nx, 2 * sx + 1);
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) bytes[j] = ((j < 4 ? w0 : w1) >> (8 * (j & 3))) & 0xffu;
    // bit j: block bx0 + j holds an obstacle
    uint32_t m8 = 0u;
#pragma unroll
    for (int j = 0; j < 8; ++j)
        if (__ballot(bytes[j] != 0) != 0 && bx0 + j < g.nbx) m8 |= 1u << j;
    if (lane == 0 && m8) atomicOr(&word, m8 << (8 * w));
    __syncthreads();
    const uint32_t all = word;
    if (all == 0u) return;
    if (w == 0) {
        bool first = false;
        if (lane == 0) {
            static_assert(C_NDIL == C_NBLK + 1 && C_NBLK == 0, "adjacent counters");
            bool tnew = false;
            const int32_t t = hinsert(g.tkeys, g.tmask, pack_key(sx, by >> 3, bz >> 3), &tnew);
            tile = t;
            if (t < 0) {
                set_error(g, -3 /* EDT_ERR_CAPACITY */);
            } else {
                const unsigned long long nb = (unsigned long long)__popc(all);
                first_slot = (int32_t)(uint32_t)atomicAdd((unsigned long long*)&g.cnt[C_NBLK],
                                                          nb | (nb << 32));
                g.tobst[(int64_t)t * 16 + (((by & 7) + 8 * (bz & 7)) >> 2)] = all;
                first = atomicOr(&g.tflag[t], 1) == 0;
                if (tnew) g.tlist[atomicAdd(&g.cnt[C_NTILE], 1)] = t;
            }
        }
        grow_tiles(g, first, sx, by >> 3, bz >> 3);
    }
    __syncthreads();
    const int32_t t = tile;
    const int base = first_slot + __popc(all & ((1u << (8 * w)) - 1u));
    // lane j < 8: the slot of block bx0 + j (-1: none, or the pool is full)
    int32_t slot = -1;
    if (lane < 8 && ((m8 >> lane) & 1u) && t >= 0) {
        const int idx = base + __popc(m8 & ((1u << lane) - 1u));
        if (idx < g.max_blocks) {
            slot = idx;
            g.bkey[slot] = pack_key(bx0 + lane, by, bz);
            g.flags[slot] = F_DILATED;
            g.tslots[(int64_t)t * 512 + block_local(lane, by, bz)] = slot;
        } else {
            set_error(g, -3 /* EDT_ERR_CAPACITY */);
            g.cnt[C_ABORT] = 1;
        }
    }
    uint8_t* occ8 = (uint8_t*)g.occ;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int32_t sj = __shfl(slot, j);
        if (sj >= 0) {
            occ8[(int64_t)sj * 64 + lane] = (uint8_t)bytes[j];
            uint32_t* chg = lane < 16 ? g.chg_add : g.chg_rem;
            if (lane < 32) chg[(int64_t)sj * 16 + (lane & 15)] = 0u;
        }
    }
}

// Block list: eight input blocks per wave, eight lanes per block.  Lane q of
// a block reads rows 8q .. 8q + 7 (64 bytes: z = q, y = 0..7) and returns
// their bit rows as one 64-bit word, which is word q of the block's
// occupancy; voxels beyond the extent are dropped.
__device__ inline unsigned long long block_rows8(const Grid& g, const int32_t* xyz,
                                                 const uint8_t* data, int64_t i, int q,
                                                 int& bx, int& by, int& bz, bool& in_range) {
    bx = xyz[3 * i];
    by = xyz[3 * i + 1];
    bz = xyz[3 * i + 2];
    in_range = bx >= 0 && by >= 0 && bz >= 0 && bx < g.nbx && by < g.nby && bz < g.nbz;
    const uint4* p = (const uint4*)(data + i * 512 + 64 * q);
    uint4 v[4];
#pragma unroll
    for (int w = 0; w < 4; ++w) v[w] = p[w];
    const int xr = g.nx - 8 * bx;
    const uint32_t xm = xr >= 8 ? 0xffu : (xr <= 0 ? 0u : (1u << xr) - 1u);
    const bool zok = 8 * bz + q < g.nz;
    unsigned long long rows = 0ull;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        const uint32_t d[4] = {v[w].x, v[w].y, v[w].z, v[w].w};
#pragma unroll
        for (int h = 0; h < 2; ++h) {              // row y = 2w + h
            uint32_t b = 0u;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                b |= (((d[2 * h] >> (8 * k)) & 0xffu) != 0u) << k;
                b |= (((d[2 * h + 1] >> (8 * k)) & 0xffu) != 0u) << (k + 4);
            }
            const bool ok = zok && 8 * by + 2 * w + h < g.ny;
            rows |= (unsigned long long)(ok ? (b & xm) : 0u) << (8 * (2 * w + h));
        }
    }
    return rows;
}

// Word q of input block i's occupancy.  BITS: the input already holds the
// pool's bit layout (64 bytes per block, as the compaction gathers it);
// otherwise one byte per voxel (block_rows8).
template <bool BITS>
__device__ inline unsigned long long input_rows(const Grid& g, const int32_t* xyz,
                                                const uint8_t* data, int64_t i, int q, int& bx,
                                                int& by, int& bz, bool& in_range) {
    if (!BITS) return block_rows8(g, xyz, data, i, q, bx, by, bz, in_range);
    bx = xyz[3 * i];
    by = xyz[3 * i + 1];
    bz = xyz[3 * i + 2];
    in_range = bx >= 0 && by >= 0 && bz >= 0 && bx < g.nbx && by < g.nby && bz < g.nbz;
    return ((const unsigned long long*)data)[i * 8 + q];
}

// Block list, phase 1: record every block holding an obstacle in its tile's
// obstacle mask (creating the tile and its neighbourhood).  Pool slots are
// assigned by the dilation.  The block count is n, or *n_dev when given.
template <bool BITS>
__global__ void __launch_bounds__(64) k_ingest_blocks_mark(Grid g, const int32_t* xyz,
                                                          const uint8_t* data, int64_t n0,
                                                          const int32_t* n_dev) {
    const int lane = threadIdx.x, sub = lane >> 3, q = lane & 7;
    const int64_t n = n_dev ? (int64_t)*n_dev : n0;
    for (int64_t i0 = (int64_t)blockIdx.x * 8; i0 < n; i0 += (int64_t)gridDim.x * 8) {
        const int64_t i = i0 + sub;
        int bx = 0, by = 0, bz = 0;
        bool ok = false;
        unsigned long long rows = 0ull;
        if (i < n) rows = input_rows<BITS>(g, xyz, data, i, q, bx, by, bz, ok);
        const bool any = ((__ballot(rows != 0ull) >> (8 * sub)) & 0xffull) != 0ull;
        // lane q = 0 of each obstacle block finds or creates the block's tile
        bool act = false, tnew = false;
        int32_t t = -1;
        if (q == 0 && i < n) {
            if (!ok) {
                set_error(g, -2 /* EDT_ERR_RANGE */);
            } else if (any) {
                t = hinsert(g.tkeys, g.tmask, pack_key(bx >> 3, by >> 3, bz >> 3), &tnew);
                if (t < 0) set_error(g, -3 /* EDT_ERR_CAPACITY */);
                else act = true;
            }
        }
        const int j = wave_append(tnew, &g.cnt[C_NTILE]);
        if (tnew) g.tlist[j] = t;
        // the wave's blocks of one tile merge their mask bits into one atomic
        // per mask word, and only the first of them sets the tile's flag
        const int local = block_local(bx, by, bz);
        const int word = act ? local >> 5 : -1;
        const uint32_t bit = act ? 1u << (local & 31) : 0u;
        const int32_t tk = act ? t : -1;
        uint32_t bits = 0u;
        bool wlead = act, tlead = act;
#pragma unroll
        for (int s2 = 0; s2 < 8; ++s2) {
            const int32_t ot = __shfl(tk, 8 * s2);
            const int ow = __shfl(word, 8 * s2);
            const uint32_t ob = __shfl(bit, 8 * s2);
            if (act && ot == t) {
                if (8 * s2 < lane) tlead = false;
                if (ow == word) {
                    bits |= ob;
                    if (8 * s2 < lane) wlead = false;
                }
            }
        }
        if (wlead) atomicOr(&g.tobst[(int64_t)t * 16 + word], bits);
        bool first = false;
        if (tlead) first = atomicOr(&g.tflag[t], 1) == 0;
        grow_tiles(g, first, bx >> 3, by >> 3, bz >> 3);
    }
}

// Block list, phase 2 (after the dilation created and zeroed every slot): OR
// the bits in (repeated listings merge), one 64-bit word per lane.
template <bool BITS>
__global__ void __launch_bounds__(64) k_ingest_blocks_write(Grid g, const int32_t* xyz,
                                                           const uint8_t* data, int64_t n0,
                                                           const int32_t* n_dev) {
    const int lane = threadIdx.x, sub = lane >> 3, q = lane & 7;
    const int64_t n = n_dev ? (int64_t)*n_dev : n0;
    for (int64_t i0 = (int64_t)blockIdx.x * 8; i0 < n; i0 += (int64_t)gridDim.x * 8) {
        const int64_t i = i0 + sub;
        if (i >= n) continue;
        int bx, by, bz;
        bool ok;
        const unsigned long long rows = input_rows<BITS>(g, xyz, data, i, q, bx, by, bz, ok);
        if (!ok || rows == 0ull) continue;
        const int32_t slot = find_block(g, bx, by, bz);
        if (slot < 0) continue;
        atomicOr((unsigned long long*)g.occ + (int64_t)slot * 8 + q, rows);
    }
}

// ---------------------------------------------------------------------------
// region growth on tiles: every block within R blocks (Chebyshev) of an
// obstacle block joins the pool.  TR = ceil(R / 8) tiles of neighbourhood.
// ---------------------------------------------------------------------------
// One workgroup per tile: OR the obstacle masks of the tile neighbourhood
// shifted by -R..R along x, then y, then z (separable Chebyshev dilation on
// bit rows in LDS) and create the missing blocks of the dilated mask.  RT:
// the block radius R as a constant (1 .. 8, one tile of neighbourhood, loops
// unrolled, one wave), or 0 for any R read from the grid: up to 9^3 tiles of
// neighbourhood and 72^2 rows, which NT = 256 lanes share (33 -> 18 us at
// R = 13, where the 128 tiles of a 512 x 512 x 128 extent leave half the CUs
// without a workgroup).
template <int RT, int NT>
__global__ void __launch_bounds__(NT) k_tile_dilate(Grid g) {
    extern __shared__ __align__(16) uint32_t sm[];
    const int R = RT > 0 ? RT : g.R, TR = RT > 0 ? 1 : (R + 7) >> 3, w = 2 * TR + 1,
              NN = w * w * w;
    const int E = 8 + 2 * R;                 // rows of the dilation window per axis
    uint32_t* nmask = sm;                    // [NN][16] neighbour obstacle masks
    uint8_t* s1 = (uint8_t*)(sm + NN * 16);  // [E][E]  x-dilated rows (y', z')
    uint8_t* s2 = s1 + E * E;                // [E][8]  y-dilated rows (z', y)
    uint8_t* dil = s2 + E * 8;               // [64]    result rows (y, z)
    const int tid = threadIdx.x, lane = tid & 63;
    const int64_t ntiles = g.cnt[C_NTILE];
    for (int64_t it = blockIdx.x; it < ntiles; it += gridDim.x) {
        const int t = g.tlist[it];
        int tx, ty, tz;
        unpack_key(g.tkeys[t], tx, ty, tz);
        // this lane's 8 table entries (row y + 8z), read now so the load
        // overlaps the dilation; only this workgroup writes them
        const int64_t e0 = (int64_t)t * 512 + 8 * lane;
        const int4 ta = *(const int4*)(g.tslots + e0), tb = *(const int4*)(g.tslots + e0 + 4);
        for (int n = tid; n < NN; n += NT) {
            const int dx = n % w - TR, dy = (n / w) % w - TR, dz = n / (w * w) - TR;
            const int nt = (tx + dx < 0 || ty + dy < 0 || tz + dz < 0)
                               ? -1
                               : hpos(g.tkeys, g.tmask, pack_key(tx + dx, ty + dy, tz + dz));
            const uint4* from = (const uint4*)(g.tobst + (int64_t)(nt >= 0 ? nt : 0) * 16);
#pragma unroll
            for (int k = 0; k < 4; ++k)
                ((uint4*)nmask)[n * 4 + k] = nt >= 0 ? from[k] : make_uint4(0u, 0u, 0u, 0u);
            // the tile and its face neighbours for the tile passes
            // (n = dx + 1 + 3 (dy + 1) + 9 (dz + 1) when TR = 1)
            if (TR == 1) {
                const int k = n == 13 ? 0 : n == 12 ? 1 : n == 14 ? 2 : n == 10 ? 3
                            : n == 16 ? 4 : n == 4 ? 5 : n == 22 ? 6 : -1;
                if (k >= 0) g.tinfo[it * 8 + k] = nt;
            }
        }
        __syncthreads();
        for (int r = tid; r < E * E; r += NT) {            // x dilation
            const int Y = r % E - R, Z = r / E - R;
            // the row across the w tiles along x: one mask byte per tile, bit
            // position X + 8 TR for X = -8 TR .. 8 + 8 TR - 1 (<= 72 bits)
            const int ny = ((Y >> 3) + TR), nz = ((Z >> 3) + TR);
            const int byte = (Y & 7) + 8 * (Z & 7);
            if (RT > 0) {
                // the row over the three tiles in 24 bits (bit 8 + X for
                // X = -8 .. 15); bit x of the result ORs bits 8 + x - R ..
                // 8 + x + R
                uint32_t row = 0u;
#pragma unroll
                for (int tx2 = 0; tx2 < 3; ++tx2) {
                    const int n = tx2 + 3 * (ny + 3 * nz);
                    row |= ((nmask[n * 16 + (byte >> 2)] >> (8 * (byte & 3))) & 0xffu) << (8 * tx2);
                }
                uint32_t d = 0u;
#pragma unroll
                for (int sh = 8 - RT; sh <= 8 + RT; ++sh) d |= row >> sh;
                s1[r] = (uint8_t)d;
                continue;
            }
            unsigned long long lo = 0ull, hi = 0ull;
            for (int tx2 = 0; tx2 < w; ++tx2) {
                const int n = tx2 + w * (ny + w * nz);
                const unsigned long long b =
                    (nmask[n * 16 + (byte >> 2)] >> (8 * (byte & 3))) & 0xffu;
                const int pos = 8 * tx2;
                if (pos < 64) lo |= b << pos;
                else hi |= b << (pos - 64);
            }
            uint32_t d = 0u;
            for (int x = 0; x < 8; ++x) {       // any bit in [x - R, x + R] + 8 TR
                const int a0 = x - R + 8 * TR, end = x + R + 8 * TR;
                const unsigned long long mlo =
                    (end >= 63 ? ~0ull : ((1ull << (end + 1)) - 1ull)) & (~0ull << a0);
                bool any = a0 < 64 && (lo & mlo) != 0ull;
                if (end >= 64) {
                    const int hs = a0 > 64 ? a0 - 64 : 0, he = end - 64;
                    const unsigned long long mhi =
                        (he >= 63 ? ~0ull : ((1ull << (he + 1)) - 1ull)) & (~0ull << hs);
                    any = any || (hi & mhi) != 0ull;
                }
                d |= (any ? 1u : 0u) << x;
            }
            s1[r] = (uint8_t)d;
        }
        __syncthreads();
        for (int r = tid; r < E * 8; r += NT) {            // y dilation
            const int y = r & 7, zp = r >> 3;
            uint32_t d = 0u;
#pragma unroll
            for (int dy = 0; dy <= 2 * (RT > 0 ? RT : 8); ++dy)
                if (RT > 0 || dy <= 2 * R) d |= s1[(y + dy) + E * zp];
            if (RT == 0)
                for (int dy = 17; dy <= 2 * R; ++dy) d |= s1[(y + dy) + E * zp];
            s2[r] = (uint8_t)d;
        }
        __syncthreads();
        if (tid < 64) {                                     // z dilation, lane = y + 8z
            const int y = lane & 7, z = lane >> 3;
            uint32_t d = 0u;
#pragma unroll
            for (int dz = 0; dz <= 2 * (RT > 0 ? RT : 8); ++dz)
                if (RT > 0 || dz <= 2 * R) d |= s2[y + 8 * (z + dz)];
            if (RT == 0)
                for (int dz = 17; dz <= 2 * R; ++dz) d |= s2[y + 8 * (z + dz)];
            dil[lane] = (uint8_t)d;
        }
        __syncthreads();
        // create the dilated blocks that are missing; lane = row (y, z), its
        // 8 table entries are 8 lane .. 8 lane + 7.  One counter atomic per
        // tile; the new slots are contiguous.
        if (tid < 64) {
            const int y = lane & 7, z = lane >> 3;
            const int by = 8 * ty + y, bz = 8 * tz + z;
            const uint32_t d = dil[lane];
            const int32_t ex[8] = {ta.x, ta.y, ta.z, ta.w, tb.x, tb.y, tb.z, tb.w};
            const int nc = TR + w * (TR + w * TR);            // centre tile in nmask
            const uint32_t ob = (nmask[nc * 16 + (lane >> 2)] >> (8 * (lane & 3))) & 0xffu;
            uint32_t want = 0u;
#pragma unroll
            for (int x = 0; x < 8; ++x)
                if (((d >> x) & 1u) && 8 * tx + x < g.nbx && by < g.nby && bz < g.nbz && ex[x] == -1)
                    want |= 1u << x;
            const int c = __popc(want);
            int incl = c;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const int v = __shfl_up(incl, o);
                if (lane >= o) incl += v;
            }
            const int total = __shfl(incl, 63);
            // obstacle blocks created here (block-list input) are counted as
            // obstacle blocks; one 64-bit atomic advances both the block count
            // (low word) and that count (high word)
            const int nobst = wave_sum(__popc(want & ob));
            if (total > 0) {
                int base = 0;
                if (lane == 0) {
                    static_assert(C_NDIL == C_NBLK + 1 && C_NBLK == 0, "adjacent counters");
                    const unsigned long long old = atomicAdd(
                        (unsigned long long*)&g.cnt[C_NBLK],
                        (unsigned long long)total | ((unsigned long long)nobst << 32));
                    base = (int)(uint32_t)old;
                }
                base = __shfl(base, 0);
                int slot = base + incl - c;
#pragma unroll
                for (int x = 0; x < 8; ++x) {
                    if (!((want >> x) & 1u)) continue;
                    const bool o = (ob >> x) & 1u;
                    if (slot < g.max_blocks) {
                        g.tslots[e0 + x] = slot;
                        g.bkey[slot] = pack_key(8 * tx + x, by, bz);
                        g.flags[slot] = o ? F_DILATED : 0u;
                    } else {
                        g.tslots[e0 + x] = -1;
                        set_error(g, -3 /* EDT_ERR_CAPACITY */);
                        g.cnt[C_ABORT] = 1;
                    }
                    ++slot;
                }
                // zero the occupancy and change masks of the new slots
                // [base, base + total), 16-byte stores (4 per mask of 64 bytes)
                const int64_t lo = base, hi = min((int64_t)base + total, (int64_t)g.max_blocks);
                const uint4 zero = make_uint4(0u, 0u, 0u, 0u);
                for (int64_t k = lo * 4 + lane; k < hi * 4; k += 64) {
                    ((uint4*)g.occ)[k] = zero;
                    ((uint4*)g.chg_add)[k] = zero;
                    ((uint4*)g.chg_rem)[k] = zero;
                }
            }
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// work items: run starts along `axis` (1 = y, 2 = z)
// ---------------------------------------------------------------------------
__device__ inline bool run_member(const Grid& g, int32_t slot, uint32_t runflag) {
    return slot >= 0 && (runflag == 0u || (g.flags[slot] & runflag));
}

// A block starts a work item along `axis` when it is the first member of a
// run (the previous block is absent or not a member) or sits on an LRUN
// boundary.  axes: 1 = y only, 2 = z only, 3 = both (global transform).
__device__ inline bool run_start(const Grid& g, int bx, int by, int bz, int axis,
                                 uint32_t runflag) {
    const int c = axis == 1 ? by : bz;
    if (c % g.lrun == 0) return true;
    return !run_member(g, axis == 1 ? find_block(g, bx, by - 1, bz) : find_block(g, bx, by, bz - 1),
                       runflag);
}

// y items from the ys list and z items from the dirty list in one launch
// (incremental transform).
// Workgroups vb of vgrid (of blockDim.x threads) share the lists.
__device__ inline void items_update_body(const Grid& g, int64_t vb, int64_t vgrid) {
    const int64_t ny = min((int64_t)g.cnt[C_NYS], (int64_t)g.max_blocks);
    const int64_t nd = min((int64_t)g.cnt[C_NDIRTY], (int64_t)g.max_blocks);
    // a wave takes entries of one list only (the y part is padded to 64)
    const int64_t nyp = (ny + 63) & ~(int64_t)63;
    for (int64_t i = vb * blockDim.x + threadIdx.x; i - __lane_id() < nyp + nd;
         i += vgrid * blockDim.x) {
        const bool zpart = i - __lane_id() >= nyp;
        const int64_t k = zpart ? i - nyp : i;
        const bool ok = zpart ? k < nd : k < ny;
        bool st = false;
        int32_t slot = -1;
        if (ok) {
            slot = zpart ? g.list_dirty[k] : g.list_ys[k];
            int bx, by, bz;
            unpack_key(g.bkey[slot], bx, by, bz);
            st = run_start(g, bx, by, bz, zpart ? 2 : 1, zpart ? F_DIRTY : F_YS);
        }
        const int idx = wave_append(st, &g.cnt[zpart ? C_NZI : C_NYI]);
        if (st) (zpart ? g.list_zi : g.list_yi)[idx] = slot;
    }
}

// ---------------------------------------------------------------------------
// per-tile variants for the global transform
// ---------------------------------------------------------------------------
// Slot of the block at position a in [-8, 16) along one axis of a tile row
// or column (other coordinates inside the tile; `local` is the in-tile
// index with that axis' coordinate zero, `stride` its step): the tile below,
// the tile itself or the tile above, from the face neighbours recorded by
// the dilation.
__device__ inline int32_t axis_slot(const Grid& g, int lo, int self, int hi, int a, int local,
                                    int stride) {
    const int t = a < 0 ? lo : (a >= 8 ? hi : self);
    return t < 0 ? -1 : g.tslots[(int64_t)t * 512 + local + stride * (a & 7)];
}

// Slot of the block at tile-relative position (x, y, z) (each coordinate in
// [-8, 16)) of the tile at `tpos`, whose tile coordinates are (tx, ty, tz);
// neighbouring tiles are looked up in the tile hash.
__device__ inline int32_t tile_rel_slot(const Grid& g, int tpos, int tx, int ty, int tz, int x,
                                        int y, int z) {
    const int dx = x >> 3, dy = y >> 3, dz = z >> 3;
    int t = tpos;
    if (dx | dy | dz) {
        const int ax = tx + dx, ay = ty + dy, az = tz + dz;
        if (ax < 0 || ay < 0 || az < 0) return -1;
        t = hpos(g.tkeys, g.tmask, pack_key(ax, ay, az));
        if (t < 0) return -1;
    }
    return g.tslots[(int64_t)t * 512 + (x & 7) + 8 * (y & 7) + 64 * (z & 7)];
}

// Work items of the global transform, one workgroup per tile: a block starts
// a y (z) item when it sits on an LRUN boundary or the block before it along
// y (z) is absent.
__global__ void __launch_bounds__(64) k_items_tiles(Grid g) {
    __shared__ int32_t own[512];
    __shared__ int32_t below[64];     // (x, 7, z) of the tile at ty - 1
    __shared__ int32_t behind[64];    // (x, y, 7) of the tile at tz - 1
    const int lane = threadIdx.x;
    const int64_t ntiles = g.cnt[C_NTILE];
    for (int64_t it = blockIdx.x; it < ntiles; it += gridDim.x) {
        const int t = g.tlist[it];
        int tx, ty, tz;
        unpack_key(g.tkeys[t], tx, ty, tz);
        for (int i = lane; i < 512; i += 64) own[i] = g.tslots[(int64_t)t * 512 + i];
        below[lane] = tile_rel_slot(g, t, tx, ty, tz, lane & 7, -1, lane >> 3);
        behind[lane] = tile_rel_slot(g, t, tx, ty, tz, lane & 7, lane >> 3, -1);
        __syncthreads();
        for (int i = lane; i < 512; i += 64) {
            const int x = i & 7, y = (i >> 3) & 7, z = i >> 6;
            const int32_t slot = own[i];
            const int by = 8 * ty + y, bz = 8 * tz + z;
            const bool ex = slot >= 0;
            const int32_t py = y > 0 ? own[i - 8] : below[x + 8 * z];
            const int32_t pz = z > 0 ? own[i - 64] : behind[x + 8 * y];
            const bool sy = ex && ((by % g.lrun) == 0 || py < 0);
            const bool sz = ex && ((bz % g.lrun) == 0 || pz < 0);
            const int jy = wave_append(sy, &g.cnt[C_NYI]);
            if (sy) g.list_yi[jy] = slot;
            const int jz = wave_append(sz, &g.cnt[C_NZI]);
            if (sz) g.list_zi[jz] = slot;
        }
        __syncthreads();
    }
}

// g1 of a strip of 8 blocks along x (slots sl, -1 absent), one wave, lane =
// row (y + 8z) of the blocks.  b: the rows' bytes; L: distance from the voxel
// before the strip back to the nearest obstacle at or before it, R: from the
// voxel after the strip to the nearest one at or after it.  Each lane sweeps
// its row twice with a carried distance (left to right, then right to left
// inside each block); a voxel's distance to the nearest obstacle along x is
// the smaller of the two, capped at d_max.  The squared values are transposed
// through LDS so that every lane stores 16 contiguous bytes of the y-major g1
// block.
template <bool F16>
__device__ inline void x_strip(const Grid& g, const int32_t* sl, const uint32_t (&b)[8], uint32_t L,
                               uint32_t R, uint4 (*tr)[72], int lane) {
    const uint32_t dmax = (uint32_t)g.dmax;
    // rc[j]: distance from the first voxel after central block j to
    // the nearest obstacle at or after it
    uint32_t rc[8];
#pragma unroll
    for (int j = 7; j >= 0; --j) {
        rc[j] = R;
        const uint32_t bj = b[j];
        R = bj ? (uint32_t)(__ffs(bj) - 1) : R + 8u;
    }
    // least g1 of each block: 0 on a row holding an obstacle, else set
    // by the end voxels (voxel 0 is nearest the left obstacle, voxel 7
    // the right one).  lc: distance from the voxel before block j to
    // the nearest obstacle at or before it.  The squares (<= 255^2) are
    // reduced over the wave two blocks at a time, packed.
    uint32_t bmins[4];
    {
        uint32_t lc = L, nsq[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const uint32_t bj = b[j];
            const uint32_t near = bj ? 0u : min(min(lc + 1u, rc[j] + 1u), dmax);
            nsq[j] = near * near;
            lc = bj ? (uint32_t)__clz(bj) - 24u : lc + 8u;
        }
#pragma unroll
        for (int h = 0; h < 4; ++h)
            bmins[h] = wave_reduce_pk_u16<false>(nsq[2 * h] | (nsq[2 * h + 1] << 16));
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const uint32_t bj = b[j];
        const int bmin = (int)((bmins[j >> 1] >> (16 * (j & 1))) & 0xffffu);
        uint32_t m[8], d[8];
#pragma unroll
        for (int x = 0; x < 8; ++x) m[x] = (uint32_t)((int32_t)(bj << (31 - x)) >> 31);
#pragma unroll
        for (int x = 0; x < 8; ++x) { L = (L + 1u) & ~m[x]; d[x] = L; }
        uint32_t r = rc[j];
#pragma unroll
        for (int x = 7; x >= 0; --x) {
            r = (r + 1u) & ~m[x];
            const uint32_t v = min(min(d[x], r), dmax);
            d[x] = F16 ? (uint32_t)__builtin_bit_cast(unsigned short,
                                                             (_Float16)(v * v))
                              : v * v;
        }
        const int32_t slot = sl[j];
        if (lane == 0 && slot >= 0) g.bmin1[slot] = (uint16_t)bmin;
        // a block that is D everywhere is not stored: its readers see
        // the block minimum D and take the shared D block instead
        if (slot >= 0 && bmin < g.D) {
            uint4* buf = tr[j & 1];
            buf[lane + (lane >> 3)] = make_uint4(d[0] | (d[1] << 16), d[2] | (d[3] << 16),
                                                 d[4] | (d[5] << 16), d[6] | (d[7] << 16));
            __syncthreads();
            // lane = x + 8z gathers column x of rows y + 8z, y = 0..7
            const uint16_t* t16 = (const uint16_t*)buf + 72 * (lane >> 3) + (lane & 7);
            uint32_t w[4];
#pragma unroll
            for (int q = 0; q < 4; ++q)
                w[q] = (uint32_t)t16[16 * q] | ((uint32_t)t16[16 * q + 8] << 16);
            *reinterpret_cast<uint4*>(g.g1 + (int64_t)slot * 512 + 8 * lane) =
                make_uint4(w[0], w[1], w[2], w[3]);
        }
    }
}

// pass X for the global transform: one wave per row of 8 blocks along x
// inside a tile (64 per tile), with M = R <= 8 blocks of context on each side
// (d_max <= 64).
template <int M>
__global__ void __launch_bounds__(64) k_pass_x_rows(Grid g) {
    constexpr int NB = 8 + 2 * M;
    constexpr uint32_t FAR = 1u << 20;
    __shared__ int32_t sl[NB];
    __shared__ uint4 tr[2][72];       // row r at r + r / 8: conflict-free reads
    const int lane = threadIdx.x;
    const int64_t nrows = (int64_t)g.cnt[C_NTILE] * 64;
    const uint8_t* occ8 = (const uint8_t*)g.occ;
    for (int64_t it = blockIdx.x; it < nrows; it += gridDim.x) {
        const int32_t* ti = g.tinfo + (it >> 6) * 8;
        const int jy = (int)(it & 7), jz = (int)((it >> 3) & 7);
        // raised priority for the chain of lookups and loads, as in the
        // window passes
        __builtin_amdgcn_s_setprio(2);
        if (lane < NB) sl[lane] = axis_slot(g, ti[1], ti[0], ti[2], lane - M, 8 * jy + 64 * jz, 1);
        __syncthreads();
        bool any = false;
#pragma unroll
        for (int j = 0; j < 8; ++j) any = any || sl[M + j] >= 0;
        if (any) {
            uint32_t b[NB];
            uint32_t orb = 0u;
#pragma unroll
            for (int k = 0; k < NB; ++k) {
                const int32_t s2 = sl[k];
                b[k] = s2 >= 0 ? (uint32_t)occ8[(int64_t)s2 * 64 + lane] : 0u;
                orb |= b[k];
            }
            __builtin_amdgcn_s_setprio(0);
            if (!__any(orb != 0u)) {
                // no obstacle in the strip or its context: every g1 is D,
                // and a block that is D everywhere needs only its minimum
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const int32_t slot = sl[M + j];
                    if (lane == 0 && slot >= 0) g.bmin1[slot] = (uint16_t)g.D;
                }
                __syncthreads();
                continue;
            }
            // distance from the last voxel before the central blocks back to
            // the nearest obstacle at or before it
            uint32_t L = FAR;
#pragma unroll
            for (int k = 0; k < M; ++k) L = b[k] ? (uint32_t)__clz(b[k]) - 24u : L + 8u;
            uint32_t R = FAR;
#pragma unroll
            for (int k = NB - 1; k >= M + 8; --k) R = b[k] ? (uint32_t)(__ffs(b[k]) - 1) : R + 8u;
            uint32_t bc[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) bc[j] = b[M + j];
            x_strip<win_f16(M)>(g, sl + M, bc, L, R, tr, lane);
        }
        __syncthreads();
    }
}

// The same for larger radii (R = 9 .. 32 blocks of context): the context is
// walked outwards four blocks at a time until every row has met an obstacle.
// One wave per strip of 8 blocks instead of one per block looks its 2 R + 8
// slots up once per strip (125 -> 19 us at d_max 100 on 512 x 512 x 128).
__global__ void __launch_bounds__(64) k_pass_x_rows_wide(Grid g) {
    constexpr uint32_t FAR = 1u << 20;
    __shared__ int32_t sl[8 + 2 * 32];
    __shared__ uint4 tr[2][72];
    const int lane = threadIdx.x, R = g.R;
    const int64_t nrows = (int64_t)g.cnt[C_NTILE] * 64;
    const uint8_t* occ8 = (const uint8_t*)g.occ;
    for (int64_t it = blockIdx.x; it < nrows; it += gridDim.x) {
        const int t = g.tlist[it >> 6];
        int tx, ty, tz;
        unpack_key(g.tkeys[t], tx, ty, tz);
        const int jy = (int)(it & 7), jz = (int)((it >> 3) & 7);
        for (int i = lane; i < 8 + 2 * R; i += 64)
            sl[i] = tile_rel_slot(g, t, tx, ty, tz, i - R, jy, jz);
        __syncthreads();
        bool any = false;
#pragma unroll
        for (int j = 0; j < 8; ++j) any = any || sl[R + j] >= 0;
        if (any) {
            auto byte = [&](int i) -> uint32_t {
                const int32_t s2 = sl[i];
                return s2 >= 0 ? (uint32_t)occ8[(int64_t)s2 * 64 + lane] : 0u;
            };
            uint32_t b[8], orb = 0u;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                b[j] = byte(R + j);
                orb |= b[j];
            }
            uint32_t L = FAR, Rr = FAR;
            for (int k = 0; k < R; k += 4) {
                uint32_t l[4], r[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    l[u] = k + u < R ? byte(R - 1 - k - u) : 0u;
                    r[u] = k + u < R ? byte(R + 8 + k + u) : 0u;
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    if (L == FAR && l[u]) L = 8u * (k + u) + (uint32_t)__clz(l[u]) - 24u;
                    if (Rr == FAR && r[u]) Rr = 8u * (k + u) + (uint32_t)(__ffs(r[u]) - 1);
                }
                if (__all(L != FAR && Rr != FAR)) break;
            }
            if (!__any(orb != 0u || L != FAR || Rr != FAR)) {
                // no obstacle in the strip or its context
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const int32_t slot = sl[R + j];
                    if (lane == 0 && slot >= 0) g.bmin1[slot] = (uint16_t)g.D;
                }
            } else {
                x_strip<false>(g, sl + R, b, L, Rr, tr, lane);
            }
        }
        __syncthreads();
    }
}

// The first list entry of workgroup vb, read alongside the list's length and
// not behind it: the update's kernels are chains of dependent loads.  (With
// this, and the block minima read beside the flags in resolve_run, an update of
// 30 voxels takes 44.1 us for 44.7.)  Used only if vb is below the length; the
// lists hold max_blocks entries.
__device__ inline int32_t first_entry(const Grid& g, const int32_t* list, int64_t vb) {
    return list[vb < g.max_blocks ? vb : g.max_blocks - 1];
}

// ---------------------------------------------------------------------------
// pass X over a list of blocks (incremental transform): squared 1-D distance
// along x from the bits, clamped to D.  One wave per block, lane = row (y + 8z).
// ---------------------------------------------------------------------------
__device__ inline void pass_x_body(const Grid& g, const int32_t* list, int list_counter,
                                   int64_t vb, int64_t vgrid, int32_t* nb) {
    const int lane = threadIdx.x;
    int32_t entry = first_entry(g, list, vb);
    const int64_t n0 = g.cnt[list_counter];
    const int64_t n = n0 < g.max_blocks ? n0 : g.max_blocks;
    const int R = g.R;
    const uint8_t* occ8 = (const uint8_t*)g.occ;
    for (int64_t w = vb; w < n; w += vgrid) {
        const int32_t slot = entry;
        if (w + vgrid < n) entry = list[w + vgrid];
        int bx, by, bz;
        unpack_key(g.bkey[slot], bx, by, bz);
        for (int i = lane; i < 2 * R + 1; i += 64)
            nb[i] = (i == R) ? slot : find_block(g, bx - R + i, by, bz);
        __syncthreads();
        const uint32_t c = occ8[(int64_t)slot * 64 + lane];
        int prev = -100000, next = 100000;
        if (R <= 8) {
            // issue all neighbour loads at once, then scan in registers
            uint32_t lb[8], rb[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const int32_t sl = k < R ? nb[R - 1 - k] : -1;
                const int32_t sr = k < R ? nb[R + 1 + k] : -1;
                lb[k] = sl >= 0 ? (uint32_t)occ8[(int64_t)sl * 64 + lane] : 0u;
                rb[k] = sr >= 0 ? (uint32_t)occ8[(int64_t)sr * 64 + lane] : 0u;
            }
#pragma unroll
            for (int k = 7; k >= 0; --k) {
                if (lb[k]) prev = -8 * (k + 1) + (31 - __clz(lb[k]));
                if (rb[k]) next = 8 * (k + 1) + (__ffs(rb[k]) - 1);
            }
        } else {
            for (int k = 1; k <= R; ++k) {
                const int32_t s2 = nb[R - k];
                if (s2 < 0) continue;
                const uint32_t b = occ8[(int64_t)s2 * 64 + lane];
                if (b) { prev = -8 * k + (31 - __clz(b)); break; }
            }
            for (int k = 1; k <= R; ++k) {
                const int32_t s2 = nb[R + k];
                if (s2 < 0) continue;
                const uint32_t b = occ8[(int64_t)s2 * 64 + lane];
                if (b) { next = 8 * k + (__ffs(b) - 1); break; }
            }
        }
        int dl[8];
        int p = prev;
#pragma unroll
        for (int x = 0; x < 8; ++x) {
            if ((c >> x) & 1u) p = x;
            dl[x] = x - p;
        }
        int q = next;
        const int y = lane & 7, z = lane >> 3;
        const int dmax = g.dmax;
        uint16_t* dst = g.g1 + (int64_t)slot * 512 + 64 * z + y;
        int mn = dmax;
        const bool f16 = win_f16(R);
#pragma unroll
        for (int x = 7; x >= 0; --x) {
            if ((c >> x) & 1u) q = x;
            const int d = min(min(dl[x], q - x), dmax);
            dst[8 * x] = f16 ? __builtin_bit_cast(uint16_t, (_Float16)(d * d)) : (uint16_t)(d * d);
            mn = min(mn, d);
        }
        mn = (int)(wave_reduce_pk_u16<false>((uint32_t)(mn * mn)) & 0xffffu);
        if (lane == 0) g.bmin1[slot] = (uint16_t)mn;
        __syncthreads();
    }
}

// Incremental transform: pass x over the xs list and the y / z work items
// are independent, so they share one launch; the first nxw workgroups take
// pass x.
__global__ void __launch_bounds__(64) k_upd_x_items(Grid g, int nxw, int32_t* nfree) {
    __shared__ int32_t nb[72];
    // no kernel from here on reads the cancel mark or the scan's list length:
    // clear them for the next call
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        g.cnt[C_UABORT] = 0;
        if (nfree) *nfree = 0;
    }
    if ((int)blockIdx.x < nxw) pass_x_body(g, g.list_xs, C_NXS, blockIdx.x, nxw, nb);
    else items_update_body(g, (int64_t)blockIdx.x - nxw, (int64_t)gridDim.x - nxw);
}

// ---------------------------------------------------------------------------
// work items of the list-driven passes
// ---------------------------------------------------------------------------
// Resolve the run of a y/z work item into LDS: sl[0 .. LRUN + 2R) holds the
// slots of blocks start-R .. start+LRUN+R-1 along `axis` (-1 = absent).
// Returns (hb, len, ha): halo blocks before, run length, halo blocks after.
// With bmin given, `least` receives its value for the block of sl[lane], read
// alongside the block's flags (unchanged if the block is absent).
__device__ inline void resolve_run(const Grid& g, int32_t* sl, uint8_t* mem, int bx, int by,
                                   int bz, int axis, uint32_t runflag, int& hb, int& len,
                                   int& ha, const uint16_t* bmin, int& least) {
    const int R = g.R;
    const int nl = g.lrun + 2 * R;
    const int lane = threadIdx.x;
    for (int i = lane; i < nl; i += (int)blockDim.x) {
        const int o = i - R;
        const int32_t s = axis == 1 ? find_block(g, bx, by + o, bz) : find_block(g, bx, by, bz + o);
        sl[i] = s;
        if (bmin && i == lane && s >= 0) least = bmin[s];
        mem[i] = run_member(g, s, runflag) ? 1 : 0;
    }
    __syncthreads();
    const int start = axis == 1 ? by : bz;
    hb = 0;
    while (hb < R && sl[R - 1 - hb] >= 0) ++hb;
    len = 1;
    while (len < g.lrun && ((start + len) % g.lrun) != 0 && mem[R + len]) ++len;
    ha = 0;
    while (ha < R && sl[R + len + ha] >= 0) ++ha;
}

// An incremental pass is done with the run's own blocks (sl[R .. R + len))
// once its outputs are stored: pass Y clears their g1 / g2 marks and the seed
// mark, pass Z the front marks, so the next update starts with clean flags.
// Runs of one pass never share a block, and a run only reads the membership
// of its own blocks, so clearing cannot change another run.
__device__ inline void finish_run(const Grid& g, const int32_t* sl, int len, int axis,
                                  uint32_t runflag) {
    if (runflag == 0u) return;                  // global transform: no marks
    const uint32_t clear =
        axis == 1 ? (F_YS | F_XS | F_SEED | F_DILNEW) : (F_DIRTY | F_RAISE | F_LOWER);
    const int lane = threadIdx.x;
    if (lane < len) atomicAnd(&g.flags[sl[g.R + lane]], ~clear);
}

// ---------------------------------------------------------------------------
// lower envelope along y or z for d_max > 64 (core in edt_hull.h)
// ---------------------------------------------------------------------------
// LDS of a work item of `blocks` blocks (run and halo): the envelope of 32
// columns, then the slots, the block extrema and the membership bytes.
template <class T>
__host__ __device__ inline int hull_item_lds(int blocks) {
    return hull_lds_bytes<T>(8 * blocks) + 128 * 4 + 128 * 4 + 128;
}

// Pass Y (AXIS 1: g1 -> g2 and the least g2 of each block) and pass Z (AXIS 2:
// g2 -> s and the largest s of each block) over the work items: one workgroup
// per item (a run of up to g.lrun output blocks and the blocks within R of
// them), one lane per column and band of 32 rows, the item's 64 columns in two
// halves of 32 (x = 4 h .. 4 h + 3 in pass Y, y = 4 h .. 4 h + 3 in pass Z, so
// each half reads runs of 64 and writes runs of 64 bytes).  Values >= D are no
// points.  g1 holds squares, so pass Y keeps 16-bit entries.  blocks: the most
// blocks an item can have (LDS and workgroup are sized for it).
//
// At d_max 100 on 512 x 512 x 128 the passes take 109 and 84 us; with one lane
// per column walking its rows in order they took 631 and 510 us (the ring of
// live parabolas in LDS, two or three waves a SIMD waiting on it).  Runs of up
// to 64 blocks: 32 repeat more of the halo (pass Y 140 us).  80 registers, for
// six waves a SIMD; with 114 pass Y ran 174 us at runs of 32.
template <int AXIS>
__global__ void __launch_bounds__(1024, 6) k_pass_hull(Grid g, const int32_t* items, int item_counter,
                                                   uint32_t runflag, int blocks) {
    using T = typename std::conditional<AXIS == 1, uint16_t, uint32_t>::type;
    extern __shared__ __align__(16) unsigned char lds[];
    const HullLds<T> h = hull_lds<T>(lds, 8 * blocks);
    int32_t* sl = (int32_t*)(lds + hull_lds_bytes<T>(8 * blocks));
    int32_t* ext = sl + 128;
    uint8_t* mem = (uint8_t*)(ext + 128);
    const int t = threadIdx.x, col = t & (HC - 1), band = t / HC;
    const int R = g.R, D = g.D;
    const int64_t nit = g.cnt[item_counter];
    const uint16_t* src = AXIS == 1 ? g.g1 : g.g2;
    const uint16_t* bmin = AXIS == 1 ? g.bmin1 : g.bmin2;
    uint16_t* dst = AXIS == 1 ? g.g2 : g.s;
    for (int64_t it = blockIdx.x; it < nit; it += gridDim.x) {
        const int32_t s0 = items[it];
        int bx, by, bz;
        unpack_key(g.bkey[s0], bx, by, bz);
        int hb, len, ha, none = 0;
        resolve_run(g, sl, mem, bx, by, bz, AXIS, runflag, hb, len, ha, nullptr, none);
        const int base = R - hb;                  // sl index of item block 0
        const int n = hb + len + ha, nb = hull_bands(8 * n);
        const int i0 = band * HB;
        for (int half = 0; half < 2; ++half) {
            // this lane's column of the source block (16 bytes each)
            const int sc = AXIS == 1 ? 4 * half + (col >> 3) + 8 * (col & 7) : 32 * half + col;
            if (t < HC) h.nem[t] = 0u;
            uint32_t acc = 0u;
            T* own = h.st + i0 * HC + col;
            if (band < nb) {
                HullMask mask(i0, 8 * hb, 8 * (hb + len) - 1);
                uint4 v[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int j = 4 * band + u;
                    const int32_t slot = j < n ? sl[base + j] : -1;
                    const bool full = slot >= 0 && (int)bmin[slot] < D;   // else D everywhere
                    const uint32_t dd = (uint32_t)D | ((uint32_t)D << 16);
                    v[u] = make_uint4(dd, dd, dd, dd);
                    if (full) v[u] = ((const uint4*)src)[(int64_t)slot * 64 + sc];
                }
#pragma unroll
                for (int r = 0; r < HB; ++r) {
                    const uint32_t w = word_of(v[r >> 3], (r & 7) >> 1);
                    const int f = (int)((r & 1) ? w >> 16 : w & 0xffffu);
                    const uint32_t e = AXIS == 1
                                           ? (uint32_t)(__builtin_amdgcn_sqrtf((float)f) + 0.5f)
                                           : (uint32_t)f;
                    mask.row(f >= D ? HINF : f + r * r, r == 0 ? 0u : 1u << (r - 1));
                    own[r * HC] = (T)((e << 5) | (uint32_t)r);
                }
                mask.row(HINF, 1u << (HB - 1));
                acc = mask.bits;
            }
            __syncthreads();
            if (band < nb) {
                const int k = hull_scan(own, acc);
                h.rng[band * HC + col] = (uint16_t)(k << 8);
                if (k) atomicOr(&h.nem[col], 1u << band);
            }
            __syncthreads();
            for (int s = 1; s < nb; s <<= 1) {
                const int lb = 2 * band * s;
                if (lb + s < nb) {
                    const uint32_t m = (1u << s) - 1u;
                    const uint32_t dead = hull_merge(h, col, h.nem[col], m << lb, m << (lb + s));
                    if (dead) atomicAnd(&h.nem[col], ~dead);
                }
                __syncthreads();
            }
            const uint32_t m = band < nb ? h.nem[col] : 0u;
            if ((m >> band) & 1u) hull_enter(h, col, band, m);
            __syncthreads();
            if ((m >> band) & 1u) hull_cover(h, col, band, nb, m);
            __syncthreads();
            if (4 * band < hb + len && 4 * band + 4 > hb) {
                HullCursor<T> c;
                if (m) {
                    const int b = h.start[band * HC + col];
                    c.init(h, col, m, b, hull_start(h, col, b, i0));
                }
#pragma unroll 1
                for (int j = max(4 * band, hb); j < min(4 * band + 4, hb + len); ++j) {
                    int32_t res[HO];
#pragma unroll
                    for (int u = 0; u < HO; ++u) res[u] = D;
                    if (m) c.take(h, col, 8 * j, res);
                    const int32_t slot = sl[base + j];
                    uint16_t* o = dst + (int64_t)slot * 512 + 32 * half + col;
                    int x = res[0];
#pragma unroll
                    for (int u = 0; u < HO; ++u) {
                        o[64 * u] = (uint16_t)res[u];
                        x = AXIS == 1 ? min(x, res[u]) : max(x, res[u]);
                    }
                    // extremum of the block: the half's, then both
#pragma unroll
                    for (int d = 16; d > 0; d >>= 1) {
                        const int y = __shfl_xor(x, d, 32);
                        x = AXIS == 1 ? min(x, y) : max(x, y);
                    }
                    if (col == 0) {
                        if (half == 0) {
                            ext[j] = x;
                        } else if (AXIS == 1) {
                            g.bmin2[slot] = (uint16_t)min(x, ext[j]);
                        } else {
                            g.bmax[slot] = max(x, ext[j]);
                        }
                    }
                }
            }
            __syncthreads();
        }
        finish_run(g, sl, len, AXIS, runflag);
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// windowed minimum along y or z for d_max <= 64 (core in edt_win.h)
// ---------------------------------------------------------------------------
// The stored field s holds integers (uint16), or for radii whose window runs
// in binary16 (win_f16) the binary16 bit patterns of those integers, as the
// window computes them; readers take the integer with s_int / s_pair_int.
__device__ inline int s_int(const Grid& g, uint32_t bits) {
    return win_f16(g.R) ? f16_int(bits) : (int)bits;
}
__device__ inline uint32_t s_pair_int(const Grid& g, uint32_t w) {
    return win_f16(g.R) ? ((uint32_t)f16_int(w & 0xffffu) | ((uint32_t)f16_int(w >> 16) << 16))
                        : w;
}

__device__ inline void store_through(uint16_t* p, uint16_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Stores the results of one step of the windowed minimum: acc[o] holds output
// row o of two consecutive blocks (low half: slot0, high half: slot1; a
// negative slot has no storage and its half is dropped).  Pass Y writes g2
// (z-major rows) and the block minima; pass Z writes s and the block maxima.
// The slots are wave-uniform, so the branches are scalar and each store
// takes its block's base from scalar registers and the row from an
// immediate offset.  The block extrema are reduced on the packed values,
// both blocks at once (binary16 patterns of non-negative values order like
// the values).
template <int AXIS, bool F16>
__device__ inline void win_store(const Grid& g, int32_t slot0, int32_t slot1, const u16x2* acc,
                                 int lane) {
    if (AXIS == 1) {
        const int out_lane = (lane & 7) * 8 + (lane >> 3);
        if (slot0 >= 0) {
            uint16_t* d0 = g.g2 + (int64_t)slot0 * 512 + out_lane;
#pragma unroll
            for (int o = 0; o < 8; ++o) d0[64 * o] = acc[o].x;
        }
        if (slot1 >= 0) {
            uint16_t* d1 = g.g2 + (int64_t)slot1 * 512 + out_lane;
#pragma unroll
            for (int o = 0; o < 8; ++o) d1[64 * o] = acc[o].y;
        }
        // least output of each block, for the skip bounds of pass Z
        const uint32_t m = wave_reduce_pk_u16<false>(as_u32(min8<F16>(acc)));
        if (lane == 0) {
            if (slot0 >= 0) g.bmin2[slot0] = F16 ? (uint16_t)f16_int(m & 0xffffu) : (uint16_t)m;
            if (slot1 >= 0) g.bmin2[slot1] = F16 ? (uint16_t)f16_int(m >> 16) : (uint16_t)(m >> 16);
        }
    } else {
        // s goes through the caches: what follows a transform reads it, and
        // finds it in the last-level cache (tunnel extent at d_max 32: dense
        // readback 131 -> 102 us; non-temporal stores, which pass that cache by,
        // made the transform alone 159.3 us).  It is written through the L2
        // (system scope), which leaves that to the g2 still to be read: 160.8 us
        // for 161.9 with plain stores.
        const uint32_t m = wave_reduce_pk_u16<true>(as_u32(max8<F16>(acc)));
        if (slot0 >= 0) {
            uint16_t* d0 = g.s + (int64_t)slot0 * 512 + lane;
#pragma unroll
            for (int o = 0; o < 8; ++o) store_through(&d0[64 * o], acc[o].x);
            if (lane == 0) g.bmax[slot0] = F16 ? f16_int(m & 0xffffu) : (int)(m & 0xffffu);
        }
        if (slot1 >= 0) {
            uint16_t* d1 = g.s + (int64_t)slot1 * 512 + lane;
#pragma unroll
            for (int o = 0; o < 8; ++o) store_through(&d1[64 * o], acc[o].y);
            if (lane == 0) g.bmax[slot1] = F16 ? f16_int(m >> 16) : (int)(m >> 16);
        }
    }
}

// List-driven form: one wave per work item (a run of up to LRUN blocks,
// extended by the halo of resolve_run).
template <int M, int AXIS>
__global__ void __launch_bounds__(64) k_pass_win(Grid g, const int32_t* items, int item_counter,
                                                 uint32_t runflag) {
    __shared__ int32_t sl[96];
    __shared__ uint8_t mem[96];
    const int lane = threadIdx.x;
    int32_t entry = first_entry(g, items, blockIdx.x);
    const int64_t nit = g.cnt[item_counter];
    const uint16_t* src = AXIS == 1 ? g.g1 : g.g2;
    constexpr bool F16 = win_f16(M);
    const uint32_t Dw = F16 ? f16_bits((uint32_t)g.D) : (uint32_t)g.D;
    const uint32_t Dp = Dw | (Dw << 16);      // D in the window's representation
    for (int64_t it = blockIdx.x; it < nit; it += gridDim.x) {
        const int32_t s0 = entry;
        if (it + gridDim.x < nit) entry = items[it + gridDim.x];
        int bx, by, bz;
        unpack_key(g.bkey[s0], bx, by, bz);
        // the lane's block of the run, j = lane of the window below
        int hb, len, ha, least = g.D;
        resolve_run(g, sl, mem, bx, by, bz, AXIS, runflag, hb, len, ha,
                    AXIS == 1 ? g.bmin1 : g.bmin2, least);
        const int base = M - hb;          // sl index of item block 0
        const int nb = hb + len + ha;
        // skip masks over window positions j (block hb - M + j of the run,
        // the window of output block hb): least input of the block, D for
        // absent blocks and past the run
        const int bm = hb - M + lane >= 0 && hb - M + lane < nb ? least : g.D;
        WinSkip sk;
        sk.d = __ballot(bm >= g.D);
#pragma unroll
        for (int G = 0; G < M; ++G) {
            const int kg = G == 0 ? 1 : 8 * G;
            sk.g[G] = __ballot(bm + kg * kg >= g.D);
        }
        auto blk = [&](int b) -> uint4 {
            const int j = b - hb + M;
            const bool own = b >= 0 && b < nb && !((sk.d >> j) & 1ull);
            const int32_t s2 = own ? sl[base + b] : -1;
            const uint4* p = s2 >= 0 ? (const uint4*)src + (int64_t)s2 * 64 + lane
                                     : (const uint4*)g.dblock + lane;
            return *p;
        };
        auto emit = [&](int ob, const u16x2* acc, bool has1) {
            const int32_t slot0 = __builtin_amdgcn_readfirstlane(sl[base + ob]);
            const int32_t slot1 = __builtin_amdgcn_readfirstlane(has1 ? sl[base + ob + 1] : -1);
            win_store<AXIS, F16>(g, slot0, slot1, acc, lane);
        };
        window_min<M, F16>(hb, len, Dp, blk, emit, [](int) { return true; }, sk);
        finish_run(g, sl, len, AXIS, runflag);
        __syncthreads();
    }
}

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

// Tile form for the global transform: one wave per column of 8 blocks along
// the pass axis inside a tile (64 columns per tile), with M blocks of context
// on each side taken from the neighbouring tiles.  Absent blocks hold no
// obstacle within d_max, so they read as the constant D block.
// SPLIT (extents of at most 64 tiles, where whole columns are too few waves
// for the GPU's 1,024 SIMDs): a column goes to four or two waves, of two or
// four blocks each, that repeat its context (pass Y of one tile at d_max 20 7.5
// -> 5.0 us in four, 6.0 in two; of 16 tiles at d_max 50 24 -> 18 us in two,
// while pass Z takes 10 us in two and 13 in four).
template <int M, int AXIS, bool SPLIT>
__global__ void __launch_bounds__(64) k_pass_win_tiles(Grid g) {
    constexpr int NB = 8 + 2 * M;
    __shared__ int32_t sl[NB];
    const int lane = threadIdx.x;
    const int64_t ncol = (int64_t)g.cnt[C_NTILE] * 64;
    const uint16_t* src = AXIS == 1 ? g.g1 : g.g2;
    constexpr bool F16 = win_f16(M);
    const uint32_t Dw = F16 ? f16_bits((uint32_t)g.D) : (uint32_t)g.D;
    const uint32_t Dpw = Dw | (Dw << 16);     // D in the window's representation
    const int sp = !SPLIT ? 0 : ncol <= 512 ? 2 : ncol <= 4096 ? 1 : 0;
    const int count = 8 >> sp;                // output blocks of a wave
    for (int64_t iw = blockIdx.x; iw < ncol << sp; iw += gridDim.x) {
        const int64_t it = iw >> sp;
        const int j0 = SPLIT ? (int)(iw & ((1 << sp) - 1)) * count : 0;
        const int32_t* ti = g.tinfo + (it >> 6) * 8;
        const int ca = (int)(it & 7), cb = (int)((it >> 3) & 7);
        // the lookups and the window's first loads form a chain of
        // dependent loads; a raised wave priority issues its links ahead of
        // the other waves' window arithmetic (back to normal once the first
        // window blocks are requested)
        __builtin_amdgcn_s_setprio(2);
        if (lane < NB)
            sl[lane] = AXIS == 1 ? axis_slot(g, ti[3], ti[0], ti[4], lane - M, ca + 64 * cb, 8)
                                 : axis_slot(g, ti[5], ti[0], ti[6], lane - M, ca + 8 * cb, 64);
        __syncthreads();
        bool any = false;
#pragma unroll
        for (int j = 0; j < 8; ++j)
            any = any || (sl[M + j] >= 0 && (!SPLIT || (j >= j0 && j < j0 + count)));
        if (any) {
            // skip masks over window positions j (block j - M): least input
            // of the block, D for absent blocks and past the context
            const uint16_t* bmin = AXIS == 1 ? g.bmin1 : g.bmin2;
            int bm = g.D;
            if (lane < NB) {
                const int32_t s2 = sl[lane];
                if (s2 >= 0) bm = bmin[s2];
            }
            // (bit 0 is the first block of the wave's own window, block j0 - M)
            WinSkip sk;
            const uint64_t flat = __ballot(bm >= g.D);
            sk.d = flat >> j0;
#pragma unroll
            for (int G = 0; G < M; ++G) {
                const int kg = G == 0 ? 1 : 8 * G;
                sk.g[G] = __ballot(bm + kg * kg >= g.D) >> j0;
            }
            const uint64_t window = SPLIT ? (1ull << (count + 2 * M)) - 1ull : ~0ull;
            if ((sk.d & window) == window) {
                // every block of the window is D everywhere, so is every
                // output: pass Y records the block minimum D and stores no
                // g2 (its readers take the shared D block); pass Z stores s
                // as whole D blocks, 16 bytes per lane, and the maximum D
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    if (SPLIT && (j < j0 || j >= j0 + count)) continue;
                    const int32_t slot = __builtin_amdgcn_readfirstlane(sl[M + j]);
                    if (slot < 0) continue;
                    if (AXIS == 1) {
                        if (lane == 0) g.bmin2[slot] = (uint16_t)g.D;
                    } else {
                        ((u32x4*)(g.s + (int64_t)slot * 512))[lane] = (u32x4){Dpw, Dpw, Dpw, Dpw};
                        if (lane == 0) g.bmax[slot] = g.D;
                    }
                }
                __syncthreads();
                continue;
            }
            // a block that is D everywhere reads the shared D block (cache
            // resident) instead of its own copy
            auto blk = [&](int b) -> uint4 {
                const int j = b + M;
                const int32_t s2 = (j < NB && !((flat >> j) & 1ull)) ? sl[j] : -1;
                const uint4* p = s2 >= 0 ? (const uint4*)src + (int64_t)s2 * 64 + lane
                                         : (const uint4*)g.dblock + lane;
                return *p;
            };
            auto emit = [&](int ob, const u16x2* acc, bool) {
                const int32_t slot0 = __builtin_amdgcn_readfirstlane(sl[M + ob]);
                const int32_t slot1 = __builtin_amdgcn_readfirstlane(sl[M + ob + 1]);
                win_store<AXIS, F16>(g, slot0, slot1, acc, lane);
            };
            auto need = [&](int ob) { return sl[M + ob] >= 0 || sl[M + ob + 1] >= 0; };
            window_min<M, F16>(j0, SPLIT ? count : 8, Dpw, blk, emit, need, sk);
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// readback and query
// ---------------------------------------------------------------------------
// Dense readbacks: one workgroup of four waves per strip of RB_BLOCKS blocks
// along x (256 voxels) at one block row (by, bz).  The strip's blocks are
// first staged in LDS with coalesced loads (a block's 1 KiB of s as one
// 16-byte load per lane), then each wave writes whole rows of the strip, four
// consecutive voxels per lane: one store instruction covers 1 KiB of int32
// output (256 bytes of occupancy), so every row of the output is written
// contiguously, with non-temporal stores (the output is not read back by the
// library; streaming it past the caches took the int32 readback of the
// tunnel field from 4.6 to 6.7 TB/s).  Absent blocks read D (free for the
// occupancy).
constexpr int RB_BLOCKS = 32;
typedef int i32x4 __attribute__((ext_vector_type(4)));
enum { RB_FIELD = 0, RB_SIGNED = 1, RB_OCC = 2 };

template <int KIND>
__global__ void __launch_bounds__(256) k_read_strip(Grid g, void* __restrict__ out) {
    constexpr int NV = KIND == RB_OCC ? 1 : RB_BLOCKS * 65;
    __shared__ int32_t sl[RB_BLOCKS];
    __shared__ uint4 val[NV];                  // block b, row r at b * 65 + r (8 values of s)
    __shared__ uint8_t bits[RB_BLOCKS * 64];   // occupancy byte of block b, row r
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int nsx = (g.nbx + RB_BLOCKS - 1) / RB_BLOCKS;
    const int64_t wg = blockIdx.x;
    const int bx0 = (int)(wg % nsx) * RB_BLOCKS;
    const int by = (int)((wg / nsx) % g.nby), bz = (int)((wg / nsx) / g.nby);
    const uint8_t* occ8 = (const uint8_t*)g.occ;
    if (t < RB_BLOCKS) sl[t] = bx0 + t < g.nbx ? find_block(g, bx0 + t, by, bz) : -1;
    __syncthreads();
    // stage: wave w takes blocks w, w + 4, ...; lane = row (y + 8z)
    for (int bb = w; bb < RB_BLOCKS; bb += 4) {
        const int32_t slot = sl[bb];
        if (slot < 0) continue;
        const uint8_t ob = occ8[(int64_t)slot * 64 + lane];
        if (KIND != RB_FIELD) bits[bb * 64 + lane] = ob;
        if (KIND == RB_OCC) continue;
        uint4 v = ((const uint4*)(g.s + (int64_t)slot * 512))[lane];
        v = make_uint4(s_pair_int(g, v.x), s_pair_int(g, v.y), s_pair_int(g, v.z),
                       s_pair_int(g, v.w));
        if (KIND == RB_SIGNED && __any(ob != 0u)) {
            // occupied voxels take their interior value (D without storage)
            const int32_t ii = g.iidx[slot];
            const uint32_t dd = (uint32_t)g.D | ((uint32_t)g.D << 16);
            const uint4 iv = ii >= 0 ? ((const uint4*)(g.ic1 + (int64_t)ii * 512))[lane]
                                     : make_uint4(dd, dd, dd, dd);
            uint32_t* vw = &v.x;
            const uint32_t* iw = &iv.x;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint32_t lo = (ob >> (2 * q)) & 1u ? 0x0000ffffu : 0u;
                const uint32_t hi = (ob >> (2 * q + 1)) & 1u ? 0xffff0000u : 0u;
                vw[q] = (vw[q] & ~(lo | hi)) | (iw[q] & (lo | hi));
            }
        }
        val[bb * 65 + lane] = v;
    }
    __syncthreads();
    // write: wave w takes rows w, w + 4, ...
    const int x = 8 * bx0 + 4 * lane;
    const int bb = lane >> 1;
    const int32_t slot = sl[bb];
    if (x >= g.nx) return;
    for (int r = w; r < 64; r += 4) {
        const int y = 8 * by + (r & 7), z = 8 * bz + (r >> 3);
        if (y >= g.ny || z >= g.nz) continue;
        const int64_t off = ((int64_t)z * g.ny + y) * (int64_t)g.nx + x;
        const uint32_t ob = slot >= 0 && KIND != RB_FIELD ? (bits[bb * 64 + r] >> (4 * (lane & 1))) & 15u
                                                          : 0u;
        if (KIND == RB_OCC) {
            const uint32_t v = (ob & 1u) | ((ob & 2u) << 7) | ((ob & 4u) << 14) | ((ob & 8u) << 21);
            uint8_t* o = (uint8_t*)out + off;
            if (x + 4 <= g.nx && ((uintptr_t)o & 3) == 0) {
                __builtin_nontemporal_store(v, (uint32_t*)o);
            } else {
                for (int k = 0; k < 4 && x + k < g.nx; ++k) o[k] = (uint8_t)(v >> (8 * k));
            }
        } else {
            int32_t v[4];
            if (slot < 0) {
                v[0] = v[1] = v[2] = v[3] = g.D;
            } else {
                const uint2 h = ((const uint2*)&val[bb * 65 + r])[lane & 1];
                v[0] = (int32_t)(h.x & 0xffffu);
                v[1] = (int32_t)(h.x >> 16);
                v[2] = (int32_t)(h.y & 0xffffu);
                v[3] = (int32_t)(h.y >> 16);
                if (KIND == RB_SIGNED) {
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        if ((ob >> k) & 1u) v[k] = -v[k];
                }
            }
            int32_t* o = (int32_t*)out + off;
            if (x + 4 <= g.nx && ((uintptr_t)o & 15) == 0) {
                __builtin_nontemporal_store((i32x4){v[0], v[1], v[2], v[3]}, (i32x4*)o);
            } else {
                for (int k = 0; k < 4 && x + k < g.nx; ++k) o[k] = v[k];
            }
        }
    }
}

// g1, g2 and s of voxel (x, y, z) inside the extent (absent block: D).  The
// global passes X and Y do not always store a block that is D everywhere, so
// g1 and g2 are D wherever their block minimum is.
__device__ inline int field_g1(const Grid& g, int x, int y, int z) {
    const int32_t slot = find_block(g, x >> 3, y >> 3, z >> 3);
    if (slot < 0 || (int)g.bmin1[slot] >= g.D) return g.D;
    const uint16_t v = g.g1[(int64_t)slot * 512 + (y & 7) + 8 * (x & 7) + 64 * (z & 7)];
    return win_f16(g.R) ? f16_int(v) : (int)v;
}
__device__ inline int field_g2(const Grid& g, int x, int y, int z) {
    const int32_t slot = find_block(g, x >> 3, y >> 3, z >> 3);
    if (slot < 0 || (int)g.bmin2[slot] >= g.D) return g.D;
    const uint16_t v = g.g2[(int64_t)slot * 512 + (z & 7) + 8 * (x & 7) + 64 * (y & 7)];
    return win_f16(g.R) ? f16_int(v) : (int)v;
}
__device__ inline bool field_occ(const Grid& g, int x, int y, int z) {
    const int32_t slot = find_block(g, x >> 3, y >> 3, z >> 3);
    if (slot < 0) return false;
    const int v = (x & 7) + 8 * (y & 7) + 64 * (z & 7);
    return (g.occ[(int64_t)slot * 16 + (v >> 5)] >> (v & 31)) & 1u;
}

// One thread per query.  s = min over k of g2(z + k) + k^2 and
// g2 = min over j of g1(y + j) + j^2, g1 = (x - x')^2 for the nearest
// obstacle x' of the row: the offsets are found again by equality, nearest
// first (uncapped values: s < D), then the obstacle sits at x +- sqrt(g1).
__global__ void k_query_nearest(Grid g, const int32_t* __restrict__ xyz, int64_t n,
                                int32_t* __restrict__ out) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int x = xyz[3 * i], y = xyz[3 * i + 1], z = xyz[3 * i + 2];
        int ox = -1, oy = -1, oz = -1;
        if (x >= 0 && y >= 0 && z >= 0 && x < g.nx && y < g.ny && z < g.nz) {
            const int32_t slot = find_block(g, x >> 3, y >> 3, z >> 3);
            const int sv = slot < 0 ? g.D
                                    : s_int(g, g.s[(int64_t)slot * 512 + (x & 7) + 8 * (y & 7) + 64 * (z & 7)]);
            if (sv < g.D) {
                // z offset
                int kz = 0, t2 = -1;
                for (int a = 0; a * a <= sv && t2 < 0; ++a) {
                    for (int sg = 0; sg < 2 && t2 < 0; ++sg) {
                        const int zz = sg ? z + a : z - a;
                        if ((sg && a == 0) || zz < 0 || zz >= g.nz) continue;
                        const int v = field_g2(g, x, y, zz);
                        if (v + a * a == sv) { kz = zz; t2 = v; }
                    }
                }
                // y offset
                int ky = 0, t1 = -1;
                for (int a = 0; t2 >= 0 && a * a <= t2 && t1 < 0; ++a) {
                    for (int sg = 0; sg < 2 && t1 < 0; ++sg) {
                        const int yy = sg ? y + a : y - a;
                        if ((sg && a == 0) || yy < 0 || yy >= g.ny) continue;
                        const int v = field_g1(g, x, yy, kz);
                        if (v + a * a == t2) { ky = yy; t1 = v; }
                    }
                }
                // x offset: g1 is a perfect square d^2
                if (t1 >= 0) {
                    int d = (int)sqrtf((float)t1);
                    while (d * d > t1) --d;
                    while ((d + 1) * (d + 1) <= t1) ++d;
                    if (x - d >= 0 && field_occ(g, x - d, ky, kz)) ox = x - d;
                    else if (x + d < g.nx && field_occ(g, x + d, ky, kz)) ox = x + d;
                    if (ox >= 0) { oy = ky; oz = kz; }
                }
            }
        }
        out[3 * i] = ox;
        out[3 * i + 1] = oy;
        out[3 * i + 2] = oz;
    }
}

__global__ void k_query(Grid g, const int32_t* __restrict__ xyz, int64_t n, int32_t* __restrict__ out) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int x = xyz[3 * i], y = xyz[3 * i + 1], z = xyz[3 * i + 2];
        int32_t v = g.D;
        if (x >= 0 && y >= 0 && z >= 0 && x < g.nx && y < g.ny && z < g.nz) {
            const int32_t slot = find_block(g, x >> 3, y >> 3, z >> 3);
            if (slot >= 0) v = s_int(g, g.s[(int64_t)slot * 512 + (x & 7) + 8 * (y & 7) + 64 * (z & 7)]);
        }
        out[i] = v;
    }
}

// ---------------------------------------------------------------------------
// incremental update
// ---------------------------------------------------------------------------

// The change entries of an update: n explicit ones (voxel, new state), or,
// with `nfree` set, those of a range scan: the first min(*nfree, n) entries of
// the list set a voxel free, and entry min(*nfree, n) + r is ray r of the
// scan, which sets its end voxel occupied if the ray has a return and both
// its ends lie in the extent (the last entry of a voxel counts, so hits win).
struct Changes {
    const int32_t* xyz;
    const uint8_t* state;
    int64_t n;
    int32_t* nfree;
    const int32_t* origin;
    const int32_t* ends;
    const uint8_t* hits;
    int64_t nray;
};

__device__ inline bool in_extent(const Grid& g, const int v[3]) {
    return v[0] >= 0 && v[1] >= 0 && v[2] >= 0 && v[0] < g.nx && v[1] < g.ny && v[2] < g.nz;
}

__device__ inline int64_t list_entries(const Changes& c) {
    if (!c.nfree) return c.n;
    const int64_t f = *c.nfree;
    return f < c.n ? f : c.n;
}

// Voxel of entry i (nl: list_entries); returns its new state.
__device__ inline bool change_voxel(const Changes& c, int64_t i, int64_t nl, int v[3]) {
    const int32_t* p = i < nl ? c.xyz + 3 * i : c.ends + 3 * (i - nl);
    v[0] = p[0];
    v[1] = p[1];
    v[2] = p[2];
    return i < nl ? !c.nfree && c.state[i] != 0 : true;
}

__device__ inline bool upd_winner(const Grid& g, int64_t i) {
    const int32_t h = g.upos[i];
    return h >= 0 && g.uvals[h] == (int32_t)i;
}

// Fresh pool slots claimed by lanes of this wave: an empty block with
// background values.  Called by the whole wave (each slot's 1 KiB arrays are
// written as one 16-byte store per lane).
__device__ inline void init_slots(const Grid& g, int32_t slot) {
    unsigned long long m = __ballot(slot >= 0);
    const int lane = __lane_id();
    // g1, g2 and s hold D in their own representation (binary16 for small radii)
    const uint32_t dw = win_f16(g.R) ? f16_bits((uint32_t)g.D) : (uint32_t)g.D;
    const uint4 dg = make_uint4(dw | (dw << 16), dw | (dw << 16), dw | (dw << 16), dw | (dw << 16));
    while (m) {
        const int src = __ffsll((long long)m) - 1;
        m &= m - 1ull;
        const int64_t s = __shfl(slot, src);
        if (lane < 16) {
            g.occ[s * 16 + lane] = 0u;
            g.chg_add[s * 16 + lane] = 0u;
            g.chg_rem[s * 16 + lane] = 0u;
        }
        ((uint4*)(g.g1 + s * 512))[lane] = dg;
        ((uint4*)(g.g2 + s * 512))[lane] = dg;
        ((uint4*)(g.s + s * 512))[lane] = dg;    // s holds D like g1, g2
        if (lane == 0) {
            g.bmax[s] = g.D;
            g.bmin1[s] = (uint16_t)g.D;
            g.bmin2[s] = (uint16_t)g.D;
        }
    }
}

// First kernel of an update: range check (any entry outside the extent
// cancels the whole call), last-entry-wins dedupe through a voxel-keyed hash
// (value = max entry index), and the blocks the call needs.  Every entry that
// sets a voxel gets its block (fresh slots hold background values), not only
// the winning ones: a block made for an entry that loses to a later one is
// harmless (background values are its field, and the region may be larger
// than needed), and the allocation need not wait for the dedupe.  A block
// that holds no obstacle yet and is not listed is listed for dilation (its
// creator appends it; for an existing block the listing flag decides).  The
// update's counters are zeroed here by the first workgroup, except the
// dilation list's (zeroed by the previous call's fronts kernel), to which
// every workgroup of this kernel appends.  A cancelled update sets
// C_UABORT, which the x-items kernel clears after its last reader.
__global__ void k_upd_dedupe_alloc(Grid g, Changes c) {
    const int64_t nl = list_entries(c), n = nl + c.nray;
    bool o_in = true;
    if (c.nray) {
        const int o[3] = {c.origin[0], c.origin[1], c.origin[2]};
        o_in = in_extent(g, o);
    }
    if (blockIdx.x == 0 && threadIdx.x >= C_NYI && threadIdx.x < C_N &&
        threadIdx.x != C_NNEWDIL)
        g.cnt[threadIdx.x] = 0;
    const int lane = __lane_id();
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i - lane < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        bool want = false;
        int bx = 0, by = 0, bz = 0;
        if (i < n) {
            int v[3];
            const bool st = change_voxel(c, i, nl, v);
            const bool inside = in_extent(g, v);
            int32_t h = -1;
            if (i >= nl && !(c.hits[i - nl] && o_in && inside)) {
                // a ray that sets no voxel
            } else if (!inside) {
                set_error(g, -2);
                g.cnt[C_UABORT] = 1;
            } else {
                const unsigned long long key = (unsigned long long)v[0] +
                    (unsigned long long)g.nx * ((unsigned long long)v[1] + (unsigned long long)g.ny * v[2]);
                bool created;
                h = hinsert(g.ukeys, g.umask, key, &created);
                if (h < 0) {
                    set_error(g, -3);
                    g.cnt[C_UABORT] = 1;
                } else {
                    atomicMax(&g.uvals[h], (int32_t)i);
                    want = st;
                    bx = v[0] >> 3; by = v[1] >> 3; bz = v[2] >> 3;
                }
            }
            g.upos[i] = h;
        }
        bool created = false;
        int64_t e = -1;
        unsigned long long key = 0;
        if (want) {
            key = pack_key(bx, by, bz);
            e = insert_block(g, bx, by, bz, &created);
            if (e < 0) {
                set_error(g, -3);
                g.cnt[C_UABORT] = 1;
            }
        }
        const int32_t sl = claim_slots(g, created, e, key, 0u);
        if (created && sl < 0) g.cnt[C_UABORT] = 1;   // pool full
        init_slots(g, sl);
        bool newdil = created && sl >= 0;
        int32_t dslot = sl;
        if (!created && e >= 0) {
            const int32_t s2 = __hip_atomic_load(&g.tslots[e], __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT);
            if (s2 >= 0 && !(g.flags[s2] & (F_DILATED | F_NEWDIL))) {
                const uint32_t o = atomicOr(&g.flags[s2], F_NEWDIL);
                newdil = !(o & (F_DILATED | F_NEWDIL));
                dslot = s2;
            }
        }
        const int j = wave_append(newdil, &g.cnt[C_NNEWDIL]);
        if (newdil) g.list_newdil[j] = dslot;
    }
}

// Apply the winning entries: flip occupancy bits, record the changed voxels
// per block (the wave centres) and list the blocks that hold them.  The
// voxel-keyed dedupe table is emptied here for the next call: each winner
// clears its entry once it has read it (the entries that lose to it only
// ever compare the stored index with their own), and a call cancelled before
// this kernel clears the entry of every input.  Workgroups vb of vgrid.
__device__ inline void upd_apply_body(const Grid& g, const Changes& c, int64_t vb, int64_t vgrid) {
    const int64_t nl = list_entries(c), n = nl + c.nray;
    const int64_t t0 = vb * blockDim.x + threadIdx.x, stride = vgrid * blockDim.x;
    {
        // the blocks listed for dilation are being dilated by the other
        // workgroups of this launch (or the call is cancelled): their
        // listing mark goes
        const int64_t nd = g.cnt[C_NNEWDIL];
        for (int64_t i = t0; i < nd; i += stride) atomicAnd(&g.flags[g.list_newdil[i]], ~F_NEWDIL);
    }
    if (g.cnt[C_UABORT] != 0) {
        for (int64_t i = t0; i < n; i += stride) {
            const int32_t h = g.upos[i];
            if (h >= 0) {
                g.ukeys[h] = KEY_EMPTY;
                g.uvals[h] = -1;
            }
        }
        return;
    }
    for (int64_t i = t0; i - __lane_id() < n; i += stride) {
        bool add = false, rem = false, first_seed = false, new_dil = false;
        int32_t slot = -1;
        if (i < n && upd_winner(g, i)) {
            const int32_t h = g.upos[i];
            g.ukeys[h] = KEY_EMPTY;
            g.uvals[h] = -1;
            int p[3];
            const bool tgt = change_voxel(c, i, nl, p);
            slot = find_block(g, p[0] >> 3, p[1] >> 3, p[2] >> 3);
            if (slot >= 0) {
                const int v = (p[0] & 7) + 8 * (p[1] & 7) + 64 * (p[2] & 7);
                const uint32_t bit = 1u << (v & 31);
                const int64_t w = (int64_t)slot * 16 + (v >> 5);
                const bool cur = (g.occ[w] & bit) != 0;
                if (tgt != cur) {
                    if (tgt) {
                        atomicOr(&g.occ[w], bit);
                        atomicOr(&g.chg_add[w], bit);
                        add = true;
                        const uint32_t o = atomicOr(&g.flags[slot], F_DILATED | F_SEED);
                        new_dil = !(o & F_DILATED);
                        first_seed = !(o & F_SEED);
                        if (new_dil) atomicOr(&g.flags[slot], F_DILNEW);
                    } else {
                        atomicAnd(&g.occ[w], ~bit);
                        atomicOr(&g.chg_rem[w], bit);
                        rem = true;
                        const uint32_t o = atomicOr(&g.flags[slot], F_SEED);
                        first_seed = !(o & F_SEED);
                    }
                }
            }
        }
        const unsigned long long ma = __ballot(add), mr = __ballot(rem);
        if (__lane_id() == (int)(__ffsll((long long)(ma | mr | 1ull)) - 1) && (ma | mr)) {
            atomicAdd(&g.cnt[C_NADD], __popcll(ma));
            atomicAdd(&g.cnt[C_NREM], __popcll(mr));
        }
        const int j = wave_append(first_seed, &g.cnt[C_NSEED]);
        if (first_seed) g.list_seed[j] = slot;
        if (new_dil) atomicAdd(&g.cnt[C_NDIL], 1);   // obstacle blocks (statistics)
    }
}

// Blocks that gain their first obstacle bring their R-neighbourhood in, one
// thread per neighbour.  Workgroups vb of vgrid.
__device__ inline void upd_dilate_body(const Grid& g, int64_t vb, int64_t vgrid) {
    if (g.cnt[C_UABORT] != 0) return;
    const int R = g.R, w = 2 * R + 1, w3 = w * w * w;
    const int64_t total = (int64_t)g.cnt[C_NNEWDIL] * w3;
    const int lane = __lane_id();
    for (int64_t i = vb * blockDim.x + threadIdx.x; i - lane < total; i += vgrid * blockDim.x) {
        bool created = false;
        int64_t e = -1;
        unsigned long long key = 0;
        if (i < total) {
            const int32_t slot = g.list_newdil[i / w3];
            const int o = (int)(i % w3);
            int bx, by, bz;
            unpack_key(g.bkey[slot], bx, by, bz);
            bx += o % w - R;
            by += (o / w) % w - R;
            bz += o / (w * w) - R;
            key = pack_key(bx, by, bz);
            if (bx >= 0 && by >= 0 && bz >= 0 && bx < g.nbx && by < g.nby && bz < g.nbz) {
                e = insert_block(g, bx, by, bz, &created);
                if (e < 0) {
                    set_error(g, -3);
                    g.cnt[C_UABORT] = 1;
                }
            }
        }
        const int32_t sl = claim_slots(g, created, e, key, 0u);
        if (created && sl < 0) g.cnt[C_UABORT] = 1;   // pool full
        init_slots(g, sl);
    }
}

// The occupancy changes and the dilation of the listed blocks share a
// launch: the first napply workgroups apply the entries, the others dilate.
// The two never touch the same block (dilation only creates absent blocks;
// every block an entry changes exists since the first kernel), so they need
// no order.  A full pool found by the dilation cancels the call after the
// bits may have changed: the fronts kernel then restores them from the
// change masks (and undoes the call's F_DILATED marks), so a cancelled call
// still leaves the map as it was.
__global__ void k_upd_apply_dilate(Grid g, Changes c, int napply) {
    if ((int)blockIdx.x < napply) upd_apply_body(g, c, blockIdx.x, napply);
    else upd_dilate_body(g, (int64_t)blockIdx.x - napply, (int64_t)gridDim.x - napply);
}

// Bounding boxes (block-local) of the added and removed voxels of each seed.
// Packed as xmin | xmax<<4 | ymin<<8 | ymax<<12 | zmin<<16 | zmax<<20 | 1<<24.
// byte = the wave's row (y, z) = lane of the voxel set; x from one ballot per
// bit, y and z from the ballot of nonempty rows (bit y + 8z).
__device__ inline int32_t row_box(uint32_t byte) {
    const unsigned long long rows = __ballot(byte != 0u);
    if (rows == 0ull) return 0;
    uint32_t xo = 0u;
#pragma unroll
    for (int x = 0; x < 8; ++x) xo |= (__ballot((byte >> x) & 1u) != 0ull ? 1u : 0u) << x;
    unsigned long long f = rows | (rows >> 32);
    f |= f >> 16;
    f |= f >> 8;
    const uint32_t yo = (uint32_t)f & 0xffu;
    uint32_t zo = 0u;
#pragma unroll
    for (int z = 0; z < 8; ++z) zo |= (((rows >> (8 * z)) & 0xffull) != 0ull ? 1u : 0u) << z;
    const int xmn = __ffs(xo) - 1, xmx = 31 - __clz(xo);
    const int ymn = __ffs(yo) - 1, ymx = 31 - __clz(yo);
    const int zmn = __ffs(zo) - 1, zmx = 31 - __clz(zo);
    return xmn | (xmx << 4) | (ymn << 8) | (ymx << 12) | (zmn << 16) | (zmx << 20) | (1 << 24);
}

// squared distance between voxel boxes [a0,a1] and [b0,b1] per axis
__device__ inline int box_gap2(int a0, int a1, int b0, int b1) {
    const int d = max(0, max(b0 - a1, a0 - b1));
    return d * d;
}
__device__ inline int box_dist2(int32_t pk, int sx, int sy, int sz, int bx, int by, int bz) {
    const int xmn = 8 * sx + (pk & 15), xmx = 8 * sx + ((pk >> 4) & 15);
    const int ymn = 8 * sy + ((pk >> 8) & 15), ymx = 8 * sy + ((pk >> 12) & 15);
    const int zmn = 8 * sz + ((pk >> 16) & 15), zmx = 8 * sz + ((pk >> 20) & 15);
    return box_gap2(xmn, xmx, 8 * bx, 8 * bx + 7) + box_gap2(ymn, ymx, 8 * by, 8 * by + 7) +
           box_gap2(zmn, zmx, 8 * bz, 8 * bz + 7);
}

// Raise / lower fronts around every seed and the g1/g2 recompute sets.  One
// workgroup (up to 1024 threads: every block within R of the seed at once for
// d_max <= 32) per seed block: its first wave takes the bounding boxes of the
// seed's added and removed voxels (and, for d_max <= 64, the positions of the
// 27 tiles around its tile, since the fronts reach at most one tile beyond
// it), then every thread marks blocks within R of the seed:
//   lower: some added voxel a has |box(B) - a|^2 < bmax(B)   (a value can drop)
//   raise: some removed voxel r has |box(B) - r|^2 <= bmax(B) and < D
//   xs:    blocks within R along x of a seed (their g1 can change)
//   ys:    blocks within R in x and y of a seed (their g2 can change)
// The seed's change masks are emptied for the next call once read, and the
// dilation-list count is cleared (no later kernel of the update reads it;
// the next call's first kernel appends to that list).  In a call cancelled
// after the occupancy changed (the pool filled during the dilation) the
// workgroup instead restores the seed's bits from its change masks, drops
// its marks and the F_DILATED it gained, and builds no fronts.
__global__ void __launch_bounds__(1024) k_upd_fronts(Grid g) {
    __shared__ int32_t rec[32];     // boxes, block coordinates, 27 tile positions
    __shared__ int wcnt[16][5];     // per wave: dirty, ys, xs, raise, lower
    __shared__ int bbase[3];        // the workgroup's list positions
    const int R = g.R, w = 2 * R + 1, w3 = w * w * w;
    int32_t entry = first_entry(g, g.list_seed, blockIdx.x);
    const int64_t ns = g.cnt[C_NSEED];
    const int lane = __lane_id(), wid = threadIdx.x >> 6;
    const bool cancel = g.cnt[C_UABORT] != 0;
    if (blockIdx.x == 0 && threadIdx.x == 0) g.cnt[C_NNEWDIL] = 0;
    for (int64_t si = blockIdx.x; si < ns; si += gridDim.x) {
        const int32_t seed = entry;
        if (si + gridDim.x < ns) entry = g.list_seed[si + gridDim.x];
        if (cancel) {
            if (wid == 0) {
                if (lane < 16) {
                    const int64_t w = (int64_t)seed * 16 + lane;
                    const uint32_t a = g.chg_add[w], r = g.chg_rem[w];
                    g.occ[w] = (g.occ[w] & ~a) | r;
                    g.chg_add[w] = 0u;
                    g.chg_rem[w] = 0u;
                }
                if (lane == 0) {
                    const uint32_t f = atomicAnd(&g.flags[seed], ~(F_SEED | F_DILNEW));
                    if (f & F_DILNEW) {
                        atomicAnd(&g.flags[seed], ~F_DILATED);
                        atomicSub(&g.cnt[C_NDIL], 1);
                    }
                }
            }
            continue;
        }
        if (wid == 0) {
            const uint32_t a = ((const uint8_t*)g.chg_add)[(int64_t)seed * 64 + lane];
            const uint32_t r = ((const uint8_t*)g.chg_rem)[(int64_t)seed * 64 + lane];
            int sx, sy, sz;
            unpack_key(g.bkey[seed], sx, sy, sz);
            const int32_t ba = row_box(a);
            const int32_t br = row_box(r);
            if (lane < 16) {
                g.chg_add[(int64_t)seed * 16 + lane] = 0u;
                g.chg_rem[(int64_t)seed * 16 + lane] = 0u;
            }
            if (lane == 0) {
                rec[0] = ba;
                rec[1] = br;
                rec[2] = sx;
                rec[3] = sy;
                rec[4] = sz;
            }
            if (R <= 8 && lane < 27) {
                const int tx = (sx >> 3) + lane % 3 - 1, ty = (sy >> 3) + (lane / 3) % 3 - 1,
                          tz = (sz >> 3) + lane / 9 - 1;
                rec[5 + lane] = (tx < 0 || ty < 0 || tz < 0)
                                    ? -1
                                    : hpos(g.tkeys, g.tmask, pack_key(tx, ty, tz));
            }
        }
        __syncthreads();
        const int32_t pa = rec[0], pr = rec[1], sx = rec[2], sy = rec[3], sz = rec[4];
        for (int o0 = 0; o0 < w3; o0 += blockDim.x) {
            const int o = o0 + (int)threadIdx.x;
            bool new_dirty = false, new_xs = false, new_ys = false, raise = false, lower = false;
            int32_t slot = -1;
            if (o < w3) {
                const int ox = o % w - R, oy = (o / w) % w - R, oz = o / (w * w) - R;
                const int bx = sx + ox, by = sy + oy, bz = sz + oz;
                // box distances need no loads: a block beyond D of both boxes
                // can only join the g1 / g2 sets (its own x row or xy plane of
                // the seed)
                const int da = pa != 0 ? box_dist2(pa, sx, sy, sz, bx, by, bz) : 0x7fffffff;
                const int dr = pr != 0 ? box_dist2(pr, sx, sy, sz, bx, by, bz) : 0x7fffffff;
                const bool maybe = da < g.D || dr < g.D || oz == 0;
                if (!maybe) {
                } else if (R <= 8) {
                    // the block's tile among the 27 recorded around the seed's tile
                    if (bx >= 0 && by >= 0 && bz >= 0) {
                        const int k = ((bx >> 3) - (sx >> 3) + 1) + 3 * ((by >> 3) - (sy >> 3) + 1) +
                                      9 * ((bz >> 3) - (sz >> 3) + 1);
                        const int32_t t = rec[5 + k];
                        if (t >= 0) slot = g.tslots[(int64_t)t * 512 + block_local(bx, by, bz)];
                    }
                } else {
                    slot = find_block(g, bx, by, bz);
                }
                if (slot >= 0) {
                    const int bm = g.bmax[slot];
                    const uint32_t seen = g.flags[slot];   // bits only get set in this kernel
                    lower = da < bm;
                    raise = dr <= bm && dr < g.D;
                    uint32_t want = 0;
                    if (lower) want |= F_LOWER | F_DIRTY;
                    if (raise) want |= F_RAISE | F_DIRTY;
                    if (oz == 0) want |= F_YS;
                    if (oz == 0 && oy == 0) want |= F_XS;
                    if (!(want & ~seen)) {
                        raise = lower = false;              // already marked by another seed
                    } else {
                        const uint32_t old = atomicOr(&g.flags[slot], want);
                        new_dirty = (want & F_DIRTY) && !(old & F_DIRTY);
                        new_ys = (want & F_YS) && !(old & F_YS);
                        new_xs = (want & F_XS) && !(old & F_XS);
                        raise = raise && !(old & F_RAISE);
                        lower = lower && !(old & F_LOWER);
                    }
                }
            }
            // list appends and statistics: one counter atomic per list and
            // workgroup, positions from the waves' ballots
            const unsigned long long md = __ballot(new_dirty), my = __ballot(new_ys),
                                     mx = __ballot(new_xs), mr = __ballot(raise),
                                     ml = __ballot(lower);
            if (lane == 0) {
                wcnt[wid][0] = __popcll(md);
                wcnt[wid][1] = __popcll(my);
                wcnt[wid][2] = __popcll(mx);
                wcnt[wid][3] = __popcll(mr);
                wcnt[wid][4] = __popcll(ml);
            }
            __syncthreads();
            const int nw = (int)(blockDim.x >> 6);
            if (threadIdx.x < 5) {
                const int c = threadIdx.x;
                int sum = 0;
                for (int v = 0; v < nw; ++v) sum += wcnt[v][c];
                const int ctr = c == 0 ? C_NDIRTY : c == 1 ? C_NYS : c == 2 ? C_NXS
                              : c == 3 ? C_NRAISE : C_NLOWER;
                const int base = sum ? atomicAdd(&g.cnt[ctr], sum) : 0;
                if (c < 3) bbase[c] = base;
            }
            __syncthreads();
            int bd = bbase[0], by_ = bbase[1], bx_ = bbase[2];
            for (int v = 0; v < wid; ++v) {
                bd += wcnt[v][0];
                by_ += wcnt[v][1];
                bx_ += wcnt[v][2];
            }
            const unsigned long long below = (1ull << lane) - 1ull;
            if (new_dirty) g.list_dirty[bd + __popcll(md & below)] = slot;
            if (new_ys) g.list_ys[by_ + __popcll(my & below)] = slot;
            if (new_xs) g.list_xs[bx_ + __popcll(mx & below)] = slot;
            __syncthreads();
        }
    }
}

// ---------------------------------------------------------------------------
// Occupancy integration of a range scan: rays from the sensor voxel o to end
// voxels e.  A ray visits o and every voxel the segment between the two voxel
// centres enters through a face; the i-th face crossing on axis a lies at
// segment parameter (2i + 1) / (2 |d_a|), d = e - o, and crossings at equal
// parameters are taken in the order x, y, z.  Visited voxels become free, the
// end voxel of a ray with a return becomes occupied, and hits win.
// ---------------------------------------------------------------------------

// Voxel entered at crossing j of axis a of the ray.  On every other axis b the
// voxel has moved by the number of b-crossings up to it: crossing i' of axis b
// is strictly earlier iff (2i' + 1) |d_a| < (2j + 1) |d_b|, and one at the
// same parameter counts when b comes before a.  The products stay below 2^42,
// exact in binary64, and the quotients below 2^21, so the product with the
// reciprocal in binary32 is off by less than a half and one step up or down
// makes the floor exact.
__device__ inline void ray_crossing_voxel(const int o[3], const int d[3], const int ad[3], int a,
                                          int j, int v[3]) {
    const int Q = a == 0 ? ad[0] : a == 1 ? ad[1] : ad[2];
    const double q = (double)Q, rq = (double)__builtin_amdgcn_rcpf((float)Q);
    int c[3];
#pragma unroll
    for (int b = 0; b < 3; ++b) {
        const double P = (double)(2 * j + 1) * (double)ad[b];
        int fl = (int)(P * rq);
        const double rem = fma(-(double)fl, q, P);
        int more = rem > 0.0 ? 1 : 0;
        if (rem < 0.0) { --fl; more = 1; }
        else if (rem >= q) { ++fl; more = rem > q ? 1 : 0; }
        // earlier and equal: (2i' + 1) Q <= P; earlier only: (2i' + 1) Q < P
        c[b] = b == a ? j + 1 : (fl + (b < a ? 1 : more)) >> 1;
        v[b] = o[b] + (d[b] < 0 ? -c[b] : c[b]);
    }
}

// The voxels that a scan's rays visit and that are occupied now (the end voxel
// of a ray with a return excepted) go to `list` as entries to set free, through
// the counter *c.nfree and up to the capacity c.n.  Rays with an endpoint
// outside the extent visit nothing and set EDT_ERR_RANGE.
//
// A ray's path is taken block by block: a lane takes one block that a ray
// enters, the sensor's or the one behind a crossing into a new block (every
// eighth crossing of an axis), and if the block has held an obstacle walks the
// ray's few voxels in it over the block's bits in LDS.  What bounds it is the
// chain of loads (ray, tile, slot, flags, bits) and the walk.  16,384 rays of
// 28 voxels on the mean in the 1024 x 1024 x 128 tunnels take 11.1 us.  A lane
// per visited voxel took 15.1, and 6.3 more for the prefix sums over all rays
// that gave each lane its voxel; on 200,000 rays through an open map its
// arithmetic (a hash and two divisions for each voxel) made a whole call 969 us
// and is 90 now.  Half a wave per block, testing the seven crossings of each
// axis, took 25.7: two in three lie in another block.
// A workgroup takes 64 rays, dealt out because neighbours have much the same
// length: 8 neighbours to a workgroup took 22, most waves without a block and
// a few with four times the mean.  The grid's second dimension deals out the
// blocks of one group, so that a few long rays fill the chip as well.
constexpr int SCAN_RAYS = 64, SCAN_T = 512;
__global__ void __launch_bounds__(SCAN_T) k_scan_clear(Grid g, Changes c, int32_t* __restrict__ list) {
    __shared__ int32_t first[SCAN_RAYS + 1];      // first block of each ray, and their number
    __shared__ int32_t end[SCAN_RAYS][4];         // end voxel and return of each ray
    __shared__ uint32_t bits[SCAN_T][17];         // occupancy of each lane's block
    __shared__ uint16_t at[SCAN_T][22];           // its voxels to set free
    __shared__ int wcnt[SCAN_T / 64], wgbase;
    const int t = threadIdx.x, lane = t & 63, wid = t >> 6;
    const int o[3] = {c.origin[0], c.origin[1], c.origin[2]};
    const bool o_in = in_extent(g, o);
    const int64_t groups = (c.nray + SCAN_RAYS - 1) / SCAN_RAYS;
    for (int64_t gr = blockIdx.x; gr < groups; gr += gridDim.x) {
        if (wid == 0) {
            // neighbouring rays have much the same length: deal them out
            const int64_t r = gr + lane * groups;
            int n = 0;
            if (r < c.nray) {
                const int e[3] = {c.ends[3 * r], c.ends[3 * r + 1], c.ends[3 * r + 2]};
                if (o_in && in_extent(g, e))
                    n = 1 + abs((e[0] >> 3) - (o[0] >> 3)) + abs((e[1] >> 3) - (o[1] >> 3)) +
                        abs((e[2] >> 3) - (o[2] >> 3));
                else
                    set_error(g, -2 /* EDT_ERR_RANGE */);
                end[lane][0] = e[0];
                end[lane][1] = e[1];
                end[lane][2] = e[2];
                end[lane][3] = c.hits[r];
            }
            int incl = n;
#pragma unroll
            for (int s = 1; s < SCAN_RAYS; s <<= 1) {
                const int v = __shfl_up(incl, s);
                if (lane >= s) incl += v;
            }
            first[lane] = incl - n;
            if (lane == SCAN_RAYS - 1) first[SCAN_RAYS] = incl;
        }
        __syncthreads();
        const int total = first[SCAN_RAYS];
        for (int c0 = SCAN_T * (int)blockIdx.y; c0 < total; c0 += SCAN_T * (int)gridDim.y) {
            const int f = c0 + t;
            int r = 0;                             // the last ray with first[r] <= f
#pragma unroll
            for (int k = SCAN_RAYS / 2; k > 0; k >>= 1) r += first[r + k] <= f ? k : 0;
            const int e[3] = {end[r][0], end[r][1], end[r][2]};
            const bool ret = end[r][3] != 0;
            int v[3] = {o[0], o[1], o[2]};
            int32_t slot = -1;
            const int d[3] = {e[0] - o[0], e[1] - o[1], e[2] - o[2]};
            const int ad[3] = {abs(d[0]), abs(d[1]), abs(d[2])};
            if (f < total) {
                int m = f - first[r] - 1;          // -1: the sensor's block
                if (m >= 0) {
                    const int m0 = abs((e[0] >> 3) - (o[0] >> 3));
                    const int m1 = abs((e[1] >> 3) - (o[1] >> 3));
                    int a = 0;
                    if (m >= m0) {
                        m -= m0;
                        a = 1;
                        if (m >= m1) { m -= m1; a = 2; }
                    }
                    const int oa = a == 0 ? o[0] : a == 1 ? o[1] : o[2];
                    const int da = a == 0 ? d[0] : a == 1 ? d[1] : d[2];
                    // the m-th crossing of axis a into a new block
                    ray_crossing_voxel(o, d, ad, a, 8 * m + (da < 0 ? oa & 7 : 7 - (oa & 7)), v);
                }
                slot = find_block(g, v[0] >> 3, v[1] >> 3, v[2] >> 3);
                if (slot >= 0 && !(g.flags[slot] & F_DILATED)) slot = -1;
            }
            if (slot >= 0) {
                const uint4* p = (const uint4*)(g.occ + (int64_t)slot * 16);
                const uint4 q[4] = {p[0], p[1], p[2], p[3]};
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    bits[t][4 * k] = q[k].x;
                    bits[t][4 * k + 1] = q[k].y;
                    bits[t][4 * k + 2] = q[k].z;
                    bits[t][4 * k + 3] = q[k].w;
                }
            }
            // the walk: at most 22 voxels, as a ray never turns back
            int n = 0;
            if (slot >= 0) {
                // e.. compares the parameters of the next crossings of two axes
                // a before b, (2 i_a + 1) |d_b| - (2 i_b + 1) |d_a|: the one on
                // a comes first iff it is <= 0.  Both lie within one period, so
                // the difference stays within 2 max |d| and is exact although
                // the products may wrap.
                const int mv[3] = {abs(v[0] - o[0]), abs(v[1] - o[1]), abs(v[2] - o[2])};
                const uint32_t n0 = 2 * mv[0] + 1, n1 = 2 * mv[1] + 1, n2 = 2 * mv[2] + 1;
                const int a0 = 2 * ad[0], a1 = 2 * ad[1], a2 = 2 * ad[2];
                int e01 = (int)(n0 * (uint32_t)ad[1] - n1 * (uint32_t)ad[0]);
                int e02 = (int)(n0 * (uint32_t)ad[2] - n2 * (uint32_t)ad[0]);
                int e12 = (int)(n1 * (uint32_t)ad[2] - n2 * (uint32_t)ad[1]);
                int left = ad[0] + ad[1] + ad[2] - mv[0] - mv[1] - mv[2];
                const int s0 = d[0] < 0 ? -1 : 1, s1 = d[1] < 0 ? -16 : 16,
                          s2 = d[2] < 0 ? -256 : 256;
                // position in the block, one hex digit per axis: leaving it
                // sets bit 3 of the digit that steps to 8 or to -1
                int p = (v[0] & 7) | (v[1] & 7) << 4 | (v[2] & 7) << 8;
#pragma unroll 1
                for (int k = 0; k < 22; ++k) {
                    const uint32_t word = bits[t][(p >> 7 & 14) | (p >> 6 & 1)];
                    const bool set = (word >> ((p & 7) | (p >> 1 & 24))) & 1u;
                    if (set && !(ret && left == 0)) at[t][n++] = (uint16_t)p;
                    if (--left < 0) break;
                    const bool x = max(e01, e02) <= 0, y = e12 <= 0;
                    e01 += x ? a1 : y ? -a0 : 0;
                    e02 += x ? a2 : y ? 0 : -a0;
                    e12 += x ? 0 : y ? a2 : -a1;
                    p += x ? s0 : y ? s1 : s2;
                    if (p & 0x888) break;
                }
            }
            // list positions: one counter atomic per workgroup
            int incl = n;
#pragma unroll
            for (int s = 1; s < 64; s <<= 1) {
                const int u = __shfl_up(incl, s);
                if (lane >= s) incl += u;
            }
            if (lane == 63) wcnt[wid] = incl;
            __syncthreads();
            int before = 0, all = 0;
#pragma unroll
            for (int k = 0; k < SCAN_T / 64; ++k) {
                before += k < wid ? wcnt[k] : 0;
                all += wcnt[k];
            }
            if (all != 0) {
                if (t == 0) wgbase = atomicAdd(c.nfree, all);
                __syncthreads();
                const int64_t q = (int64_t)wgbase + before + incl - n;
                for (int k = 0; k < n; ++k) {
                    if (q + k >= c.n) {
                        set_error(g, -3 /* EDT_ERR_CAPACITY */);
                        break;
                    }
                    const int p = at[t][k];
                    int32_t* out = list + 3 * (q + k);
                    out[0] = (v[0] & ~7) | (p & 7);
                    out[1] = (v[1] & ~7) | (p >> 4 & 7);
                    out[2] = (v[2] & ~7) | (p >> 8 & 7);
                }
            }
            __syncthreads();
        }
        __syncthreads();
    }
}

// Pool slots holding an obstacle, in chunks of 256 slots per wave: lane l
// reads slots 4l .. 4l + 3 of the chunk whole (four 16-byte loads each, all
// in flight together), the wave takes an exclusive prefix sum of the lanes'
// counts, and one counter atomic per chunk reserves the list positions.
// The occupancy words stay in w[t][0..3] for the caller.
struct SlotChunk {
    uint4 w[4][4];
    uint32_t has;     // bit t: slot 4 lane + t holds an obstacle
    int pos;          // first list position of this lane's slots
    int total;        // obstacle slots in the chunk
};

__device__ inline void scan_chunk(const Grid& g, int64_t c0, int64_t n, int32_t* counter,
                                  SlotChunk& c) {
    const int lane = __lane_id();
    c.has = 0u;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const int64_t slot = c0 + 4 * lane + t;
        const uint4* p = (const uint4*)(g.occ + (slot < n ? slot : 0) * 16);
#pragma unroll
        for (int q = 0; q < 4; ++q) c.w[t][q] = slot < n ? p[q] : make_uint4(0u, 0u, 0u, 0u);
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        uint32_t a = 0u;
#pragma unroll
        for (int q = 0; q < 4; ++q) a |= c.w[t][q].x | c.w[t][q].y | c.w[t][q].z | c.w[t][q].w;
        c.has |= (a != 0u ? 1u : 0u) << t;
    }
    const int mine = __popc(c.has);
    int incl = mine;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int v = __shfl_up(incl, o);
        if (lane >= o) incl += v;
    }
    c.total = __shfl(incl, 63);
    int base = 0;
    if (lane == 63 && c.total > 0) base = atomicAdd(counter, c.total);
    base = __shfl(base, 63);
    c.pos = base + incl - mine;
}

// ---------------------------------------------------------------------------
// Compaction: the blocks holding an obstacle (coordinates and occupancy
// words) are copied into a list, from which a global transform rebuilds the
// pool; blocks that no longer hold an obstacle and lie beyond R blocks of
// every obstacle block drop out.
// ---------------------------------------------------------------------------
// Pool growth (the context moves onto a larger workspace; the blocks and
// their field are copied, nothing is recomputed).  Tile positions depend on
// the hash capacity, so the tile tables are rebuilt: k_tile_rehash, one wave
// per old table position, inserts the tile's key into the new hash, records
// the new position in map[old position] (-1 for an empty position) and
// copies the tile's slot table, obstacle mask and flag.
__global__ void __launch_bounds__(64) k_tile_rehash(Grid o, Grid n, int32_t* map) {
    const int lane = threadIdx.x;
    for (int64_t p = blockIdx.x; p <= (int64_t)o.tmask; p += gridDim.x) {
        const unsigned long long key = o.tkeys[p];
        int32_t q = -1;
        if (key != KEY_EMPTY && lane == 0) {
            bool created;
            q = hinsert(n.tkeys, n.tmask, key, &created);
            if (q < 0) set_error(n, -3 /* EDT_ERR_CAPACITY */);
        }
        q = __shfl(q, 0);
        if (lane == 0) map[p] = q;
        if (q < 0) continue;
        const int4* src = (const int4*)(o.tslots + p * 512);
        int4* dst = (int4*)(n.tslots + (int64_t)q * 512);
        dst[lane] = src[lane];
        dst[lane + 64] = src[lane + 64];
        if (lane < 16) n.tobst[(int64_t)q * 16 + lane] = o.tobst[p * 16 + lane];
        if (lane == 0) n.tflag[q] = o.tflag[p];
    }
}

// Second step of the growth: the tile list and the face-neighbour records
// hold table positions; translate them through map.  Entries that do not
// name a position of the old table (face records are only written for
// d_max <= 64) become -1.
__global__ void k_tile_remap(Grid o, Grid n, const int32_t* map) {
    const int64_t nt = o.cnt[C_NTILE];
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < nt;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int32_t t = o.tlist[i];
        n.tlist[i] = (t >= 0 && t <= (int64_t)o.tmask) ? map[t] : -1;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int32_t v = o.tinfo[i * 8 + k];
            n.tinfo[i * 8 + k] = (v >= 0 && v <= (int64_t)o.tmask) ? map[v] : -1;
        }
    }
}

// Last step of the growth: a call that ran out of pool advanced the block
// counter past the old capacity without writing those slots; only the slots
// below it were claimed.  The pool abort flag no longer applies.
__global__ void k_grow_counts(Grid n, int32_t old_max_blocks) {
    if (n.cnt[C_NBLK] > old_max_blocks) n.cnt[C_NBLK] = old_max_blocks;
    n.cnt[C_ABORT] = 0;
}

__global__ void __launch_bounds__(64) k_compact_gather(Grid g, int32_t* count, int32_t* xyz,
                                                       uint32_t* bits) {
    const int lane = threadIdx.x;
    const int64_t n0 = g.cnt[C_NBLK];
    const int64_t n = n0 < g.max_blocks ? n0 : g.max_blocks;
    for (int64_t c0 = 256 * (int64_t)blockIdx.x; c0 < n; c0 += 256 * (int64_t)gridDim.x) {
        SlotChunk c;
        scan_chunk(g, c0, n, count, c);
        int idx = c.pos;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            if (!((c.has >> t) & 1u)) continue;
            uint4* dst = (uint4*)(bits + (int64_t)idx * 16);
#pragma unroll
            for (int q = 0; q < 4; ++q) dst[q] = c.w[t][q];
            int bx, by, bz;
            unpack_key(g.bkey[c0 + 4 * lane + t], bx, by, bz);
            xyz[3 * (int64_t)idx] = bx;
            xyz[3 * (int64_t)idx + 1] = by;
            xyz[3 * (int64_t)idx + 2] = bz;
            ++idx;
        }
    }
}

// ---------------------------------------------------------------------------
// Interior distances: for an occupied voxel, the squared distance to the
// nearest free voxel of the extent, clamped to D (the definition of the field
// with occupied and free exchanged: the inside half of a signed distance
// field).  Only blocks holding an obstacle carry interior values.  Every other
// block of the extent, in the pool or not, is all free, so both intermediate
// passes are 0 on it; the passes below take such blocks as 0 without storage.
// ---------------------------------------------------------------------------

// Lists the pool blocks holding an obstacle and writes every slot's interior
// index (-1 for the others).  C_NINT is zero before: pass x hands the count on
// in C_INTN and pass y clears C_NINT for the next call (with a kernel of its
// own for that, the signed field of 512 x 512 x 128 took 52.4 us, now 51.0).
__global__ void __launch_bounds__(64) k_int_list(Grid g) {
    const int lane = threadIdx.x;
    const int64_t n0 = g.cnt[C_NBLK];
    const int64_t n = n0 < g.max_blocks ? n0 : g.max_blocks;
    for (int64_t c0 = 256 * (int64_t)blockIdx.x; c0 < n; c0 += 256 * (int64_t)gridDim.x) {
        SlotChunk c;
        scan_chunk(g, c0, n, &g.cnt[C_NINT], c);
        int idx = c.pos;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int64_t slot = c0 + 4 * lane + t;
            if (slot >= n) continue;
            int32_t v = -1;
            if ((c.has >> t) & 1u) {
                if (idx < g.max_int) {
                    g.ilist[idx] = (int32_t)slot;
                    v = idx;
                } else {
                    set_error(g, -3 /* EDT_ERR_CAPACITY */);
                }
                ++idx;
            }
            g.iidx[slot] = v;
        }
    }
}

// Interior pass x: per row of a listed block, the distance along x to the
// nearest free voxel of the extent, squared and clamped to D.  One wave per
// block, lane = row y + 8z.  Neighbour blocks are read outwards until every
// lane has met a free voxel on both sides, at most R blocks each way (a voxel
// farther than that is beyond d_max).  Rows outside the extent get D.
__global__ void __launch_bounds__(64) k_int_x(Grid g) {
    __shared__ int32_t nb[72];
    const int lane = threadIdx.x;
    const int64_t n0 = g.cnt[C_NINT];
    if (blockIdx.x == 0 && lane == 0) g.cnt[C_INTN] = (int32_t)n0;
    const int64_t n = n0 < g.max_int ? n0 : g.max_int;
    const int R = g.R;
    const uint8_t* occ8 = (const uint8_t*)g.occ;
    const int y = lane & 7, z = lane >> 3;
    for (int64_t i = blockIdx.x; i < n; i += gridDim.x) {
        const int32_t slot = g.ilist[i];
        int bx, by, bz;
        unpack_key(g.bkey[slot], bx, by, bz);
        for (int k = lane; k < 2 * R + 1; k += 64)
            nb[k] = k == R ? slot : find_block(g, bx - R + k, by, bz);
        __syncthreads();
        const bool in = 8 * by + y < g.ny && 8 * bz + z < g.nz;
        // free voxels of row (y, z) in block bx + k (extent voxels only)
        auto freebits = [&](int k) -> uint32_t {
            const int w = g.nx - 8 * (bx + k);
            const uint32_t ext = w >= 8 ? 0xffu : (1u << w) - 1u;
            const int32_t s2 = nb[R + k];
            return s2 < 0 ? ext : ~(uint32_t)occ8[(int64_t)s2 * 64 + lane] & ext;
        };
        const uint32_t own = freebits(0);
        // nearest free voxel left of the block (offset from voxel 0 of the
        // block, negative) and right of it (offset, >= 8)
        int left = -(1 << 16), right = 1 << 16;
        bool dl = !in, dr = !in;
        for (int k = 1; k <= R; ++k) {
            if (!dl) {
                if (bx - k < 0) {
                    dl = true;
                } else {
                    const uint32_t f = freebits(-k);
                    if (f) { left = -8 * k + (31 - __clz(f)); dl = true; }
                }
            }
            if (!dr) {
                if (bx + k >= g.nbx) {
                    dr = true;
                } else {
                    const uint32_t f = freebits(k);
                    if (f) { right = 8 * k + (__ffs(f) - 1); dr = true; }
                }
            }
            if (__ballot(!(dl && dr)) == 0ull) break;
        }
        uint16_t* dst = g.ic1 + i * 512 + y + 64 * z;
#pragma unroll
        for (int x = 0; x < 8; ++x) {
            int d = min(x - left, right - x);
#pragma unroll
            for (int xx = 0; xx < 8; ++xx)
                if ((own >> xx) & 1u) d = min(d, abs(x - xx));
            d = min(d, g.dmax);
            dst[8 * x] = (uint16_t)(in ? d * d : g.D);
        }
        __syncthreads();
    }
}

// Interior pass along y (AXIS 1: ic1 -> ic2) or z (AXIS 2: ic2 -> ic1, the
// interior field): out(t) = min(D, min over t' of in(t') + (t - t')^2) along
// the axis, where `in` is the previous interior pass on listed blocks and 0
// on every other voxel of the extent.  One wave per listed block, lane = one
// column of 8 outputs.  Neighbour blocks are visited outwards and the walk
// stops once no lane can improve: every voxel of block offset k is at least
// 8(k - 1) + 1 away.  Columns outside the extent get D.
template <int AXIS>
__global__ void __launch_bounds__(64) k_int_yz(Grid g) {
    __shared__ int32_t nb[72];   // interior index of block offset k - R; -1 all free; -2 outside
    const int lane = threadIdx.x;
    const int64_t n0 = g.cnt[C_INTN];
    if (AXIS == 1 && blockIdx.x == 0 && lane == 0) g.cnt[C_NINT] = 0;
    const int64_t n = n0 < g.max_int ? n0 : g.max_int;
    const int R = g.R;
    const int D = g.D;
    const uint16_t* src = AXIS == 1 ? g.ic1 : g.ic2;
    uint16_t* dst = AXIS == 1 ? g.ic2 : g.ic1;
    const int ca = lane & 7, cb = lane >> 3;   // column (x, z) for y, (x, y) for z
    for (int64_t i = blockIdx.x; i < n; i += gridDim.x) {
        int bx, by, bz;
        unpack_key(g.bkey[g.ilist[i]], bx, by, bz);
        const int bc = AXIS == 1 ? by : bz;
        const int nbc = AXIS == 1 ? g.nby : g.nbz;
        for (int k = lane; k < 2 * R + 1; k += 64) {
            const int b = bc - R + k;
            int32_t e = -2;
            if (k == R) {
                e = (int32_t)i;
            } else if (b >= 0 && b < nbc) {
                const int32_t s2 = AXIS == 1 ? find_block(g, bx, b, bz) : find_block(g, bx, by, b);
                e = s2 < 0 ? -1 : g.iidx[s2];
            }
            nb[k] = e;
        }
        __syncthreads();
        const bool in = 8 * bx + ca < g.nx &&
                        (AXIS == 1 ? 8 * bz + cb < g.nz : 8 * by + cb < g.ny);
        int best[8];
        {
            const uint4 q = *reinterpret_cast<const uint4*>(src + i * 512 + 8 * lane);
            const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                int b = D;
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int v = (int)((w[u >> 1] >> (16 * (u & 1))) & 0xffffu);
                    b = min(b, v + (t - u) * (t - u));
                }
                best[t] = b;
            }
        }
        for (int k = 1; k <= R; ++k) {
            int worst = 0;
#pragma unroll
            for (int t = 0; t < 8; ++t) worst = max(worst, best[t]);
            const int lb = 8 * (k - 1) + 1;
            if (__ballot(in && lb * lb < worst) == 0ull) break;
#pragma unroll
            for (int side = -1; side <= 1; side += 2) {
                const int32_t e = nb[R + side * k];
                if (e == -2) continue;
                if (e == -1) {
                    // all free: the block's voxel nearest to the column
#pragma unroll
                    for (int t = 0; t < 8; ++t) {
                        const int d = side < 0 ? t + 8 * (k - 1) + 1 : 8 * k - t;
                        best[t] = min(best[t], d * d);
                    }
                } else {
                    const uint4 q = *reinterpret_cast<const uint4*>(src + (int64_t)e * 512 + 8 * lane);
                    const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const int v = (int)((w[u >> 1] >> (16 * (u & 1))) & 0xffffu);
                        const int tu = side * 8 * k + u;
#pragma unroll
                        for (int t = 0; t < 8; ++t) best[t] = min(best[t], v + (t - tu) * (t - tu));
                    }
                }
            }
        }
        uint16_t* o = dst + i * 512;
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const uint16_t v = (uint16_t)(in ? min(best[t], D) : D);
            if (AXIS == 1) o[cb + 8 * ca + 64 * t] = v;     // layout z + 8x + 64y
            else o[lane + 64 * t] = v;                      // layout x + 8y + 64z
        }
        __syncthreads();
    }
}

// Signed squared distance of voxel (x, y, z) inside the extent: s for a free
// voxel, minus the interior value for an occupied one.
__device__ inline int32_t signed_at(const Grid& g, int x, int y, int z) {
    const int32_t slot = find_block(g, x >> 3, y >> 3, z >> 3);
    if (slot < 0) return g.D;
    const int v = (x & 7) + 8 * (y & 7) + 64 * (z & 7);
    if ((g.occ[(int64_t)slot * 16 + (v >> 5)] >> (v & 31)) & 1u) {
        const int32_t ii = g.iidx[slot];
        return -(ii >= 0 ? (int32_t)g.ic1[(int64_t)ii * 512 + v] : g.D);
    }
    return s_int(g, g.s[(int64_t)slot * 512 + v]);
}

__global__ void k_query_signed(Grid g, const int32_t* __restrict__ xyz, int64_t n,
                               int32_t* __restrict__ out) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int x = xyz[3 * i], y = xyz[3 * i + 1], z = xyz[3 * i + 2];
        const bool in = x >= 0 && y >= 0 && z >= 0 && x < g.nx && y < g.ny && z < g.nz;
        out[i] = in ? signed_at(g, x, y, z) : g.D;
    }
}

__global__ void k_clear_error(Grid g) { g.cnt[C_ERR] = 0; }

}  // namespace edt
