// dr_tile.h -- the tile kernel: rasterises the + and - renders of one tile,
// shades both, forms the per-pixel difference and scatters it.  Included by
// one source file per tile size, each instantiating its size's kernels.
#pragma once

#include <type_traits>

#include "dr_launch.h"
#include "dr_wave.h"

// Map consecutive workgroups (which the dispatcher spreads round-robin over
// the 8 XCDs) to contiguous runs of tiles per XCD, so neighbouring tiles --
// sharing triangles, texels and accumulators -- meet in the same L2.
__device__ __forceinline__ int xcd_tile(int bid, int nb) {
    int x = bid & 7, k = bid >> 3;
    int q = nb >> 3, rem = nb & 7;
    return x * q + min(x, rem) + k;
}

// Rasterise triangle t over the tile: one lane per covered pixel.  Opaque
// (DEEP false): key[pixel] keeps the least depth|id (64-bit atomic min).
// Deep: key[pixel * DRD_MAX_LAYERS + l] keeps the L least keys in order,
// by an atomic-min cascade -- the key is offered to layer 0, and whichever
// of the offered and the resident key is larger moves on to the next layer
// (an empty slot ends the cascade).  Every layer thus ends with the least
// key that reached it, i.e. the l-th least key of the pixel, whatever the
// interleaving of the lanes and waves.
// Offer depth|id key k to pixel li of the tile.
template <bool DEEP>
__device__ __forceinline__ void insert_key(unsigned long long* key, int li, unsigned long long k, int L) {
    if constexpr (DEEP) {
        unsigned long long* list = key + li * DRD_MAX_LAYERS;
        for (int l = 0; l < L; ++l) {
            unsigned long long old = atomicMin(&list[l], k);
            if (old == ~0ull) break;
            k = old > k ? old : k;
        }
    } else {
        atomicMin(&key[li], k);
    }
}

// Keys per row of a tile: three more than its pixels for opaque tiles, since
// a raster slot that starts at the row's last pixel runs past it.
template <int TILE, bool DEEP>
struct KeyRow {
    static constexpr int N = DEEP ? TILE : TILE + 4;
};

// Rasterise triangle t over its box in the tile, one lane per covered pixel:
// triangles too large for the staged raster.  (cx1, cy1): the tile's last
// pixel inside the view.
template <int TILE, bool DEEP>
__device__ __forceinline__ void raster_tri(const TriR& r, unsigned t, int px0, int py0, int cx1, int cy1,
                                           int lane, unsigned long long* key, int L) {
    int x0, x1, y0, y1;
    tri_box(r, px0, py0, cx1, cy1, x0, x1, y0, y1);
    int bw = x1 - x0 + 1;
    int n = bw * (y1 - y0 + 1);
    unsigned m = ((1u << 20) + (unsigned)bw - 1u) / (unsigned)bw;     // exact for bw <= 32, idx < 1024
    for (int base = 0; base < n; base += 64) {
        int idx = base + lane;
        if (idx < n) {
            int dy = (int)(((unsigned)idx * m) >> 20);
            int x = x0 + idx - dy * bw, y = y0 + dy;
            int px = 256 * x + 128, py = 256 * y + 128;
            long long e0, e1, e2;
            if (!inside(r, px, py, e0, e1, e2)) continue;
            float z = depth_at(r, px, py);
            insert_key<DEEP>(key, (y - py0) * KeyRow<TILE, DEEP>::N + (x - px0),
                             ((unsigned long long)__float_as_uint(z) << 32) | t, L);
        }
    }
}

// Per-wave LDS staging of a batch of small triangles for the packed raster
// (48 B each, three 16-byte reads): edge k over the triangle's clipped
// bounding box is e_k(dx, dy) = 256 dX_k dy - 256 dY_k dx + c_k at pixel
// (x0 + dx, y0 + dy).  16-bit fields hold differences of snapped corners,
// which a TRI_SMALL triangle keeps within +-2^15.
struct __align__(16) PTri {
    int c[3];            // edge k at the box's corner pixel, plus 1 on a top-left edge
    unsigned t;
    int d[3];            // dX_k (low half), dY_k (high half)
    unsigned pk;         // bits 0..4 box width - 1, 5..15 key index of the corner pixel, 16.. first slot
    float z0, zx, zy;    // depth plane
    int dz;              // corner pixel centre minus vertex 0, in subpixels: x low, y high
};

struct RasterStage {
    PTri tri[64];
    int mark[64];
};

// Lanes of one wave exchange data through the wave's stage: a release fence
// before the wave barrier and an acquire fence after it make each lane's LDS
// stores visible to the other lanes' later loads (the barrier itself
// declares no memory effects, so without the fences the compiler could
// forward a lane's own store to its load past the other lanes' writes).
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

static_assert(sizeof(PTri) == 48, "PTri layout");

// Packed raster of a batch of TRI_SMALL triangles (one per lane; bh = 0:
// none), through the wave's LDS stage.  Each triangle's clipped box is cut
// into slots of RASTER_SLOT horizontally adjacent pixels (a row of w pixels
// gives ceil(w / RASTER_SLOT) slots), the batch's slots are laid end to end,
// and each pass gives one slot to every lane: one read of the staged record,
// one index computation and one pass marking then serve all the slot's
// pixels.  The non-empty triangles are stored by rank; each pass marks the
// slots where a triangle begins, and a lane's triangle is then the number of
// triangles begun up to its slot (a ballot and a lane-masked bit count) --
// one LDS read of the staged record instead of a binary search and a shuffle
// per field.  Edge values are exact: a TRI_SMALL triangle spans less than
// 32000 subpixels, so at every pixel of the box and up to three to its right
// both products of an edge function stay below 2^30 + 2^25 in magnitude and
// the edge value (plus 1) fits in 32 bits; the wrapped 32-bit sums equal it,
// as do the slot's further pixels' values, each its left neighbour's minus
// 256 dY.  e > 0 || (e == 0 && top-left) is e + [top-left] > 0.  A slot's
// pixels beyond the box are not covered, unless the box was clipped at the
// tile's or the view's edge: those keys fall on the row's spare columns, or
// on pixels that are not in the view and are not read (opaque; deep tiles
// test the box).
// Bound by vector issue.  The record's 48 B (80 B before) set the block's LDS
// (25.6 -> 18.5 KB for 16-pixel tiles, 6 -> 8 waves per SIMD) and a pass's LDS
// reads; with the raster compiled in once for bins, spill lists and scans
// (52 -> 34 KB of code) the GGX paper step went 1739 -> 1578 us, the
// full-image soup 1325 -> 1160 us.  Slots of 4 pixels: measured on the paper-scale step
// against 2, 3, 6 and 8 (2 -> 4: tile kernel -2 % at the start of an
// optimisation run, -9 % after 50 Adam steps, when the triangles have grown;
// 6 and 8 within 2 % of 4).
#define RASTER_SLOT 4
#define PK_SLOT 16               // first bit of PTri::pk's first slot
template <int TILE, bool DEEP>
__device__ __forceinline__ void raster_staged(RasterStage* st, const TriR& r, unsigned t, int x0, int y0, int bw,
                                              int bh, int px0, int py0, int lane, unsigned long long* key, int L) {
    constexpr int SL = RASTER_SLOT;                     // pixels per slot
    constexpr int KS = KeyRow<TILE, DEEP>::N;
    static_assert(TILE * KS <= 2048 && 64 * TILE * (TILE / SL) <= 65536 && SL == 4, "PTri::pk fields");
    const int sw = (bw + SL - 1) / SL;                  // slots per row
    const int c = sw * bh;                              // slots of this lane's triangle (0: none)
    const int P = wave_inclusive_sum(c);
    const int N = __builtin_amdgcn_readlane(P, 63);
    const int pex = P - c;
    unsigned long long nz = __ballot(c > 0);
    if (c > 0) {
        int rank = __builtin_amdgcn_mbcnt_hi((unsigned)(nz >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)nz, 0u));
        PTri q;
        int cx = 256 * x0 + 128, cy = 256 * y0 + 128;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            int ia = (k + 1) % 3, ib = (k + 2) % 3;
            int dX = r.X[ib] - r.X[ia], dY = r.Y[ib] - r.Y[ia];
            q.d[k] = (dX & 0xFFFF) | (dY << 16);
            q.c[k] = (__mul24(dX, cy - r.Y[ia]) - __mul24(dY, cx - r.X[ia])) + (int)((r.flags >> (k + 1)) & 1u);
        }
        q.dz = ((cx - r.X[0]) & 0xFFFF) | ((cy - r.Y[0]) << 16);
        q.z0 = r.z0; q.zx = r.zx; q.zy = r.zy;
        q.t = t;
        q.pk = (unsigned)(bw - 1) | ((unsigned)((y0 - py0) * KS + (x0 - px0)) << 5) | ((unsigned)pex << PK_SLOT);
        st->tri[rank] = q;
    }
    wave_sync();
    int base = 0;                                       // triangles begun before this pass
    for (int s0 = 0; s0 < N; s0 += 64) {
        st->mark[lane] = 0;
        wave_sync();
        if (c > 0 && pex >= s0 && pex < s0 + 64) st->mark[pex - s0] = 1;
        wave_sync();
        int f = st->mark[lane];
        unsigned long long M = __ballot(f != 0);
        int rr = base + (int)__builtin_amdgcn_mbcnt_hi((unsigned)(M >> 32),
                                                       __builtin_amdgcn_mbcnt_lo((unsigned)M, 0u)) + f - 1;
        base += __popcll(M);
        int sl = s0 + lane;
        if (sl < N) {
            const PTri q = st->tri[rr];
            const int idx = sl - (int)(q.pk >> PK_SLOT);
            const unsigned w4 = q.pk & 0x1Cu;           // 4 (slots per row - 1)
            int dy;                                     // idx / slots per row
            if constexpr (TILE <= 16) {
                // idx < 64, at most 4 slots: idx * ceil(128 / slots) >> 7
                dy = (int)(__umul24((unsigned)idx, (0x202B4080u >> (2u * w4)) & 0xFFu) >> 7);
            } else {
                dy = (int)(((float)idx + 0.5f) * __builtin_amdgcn_rcpf((float)((w4 >> 2) + 1u)));
            }
            const int dx = 4 * idx - __mul24(dy, (int)w4 + 4);
            int e[3], a[3];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const int dX = (int)(short)q.d[k], dY = q.d[k] >> 16;
                a[k] = 256 * dY;
                e[k] = (__mul24(dX, 256 * dy) + q.c[k]) - __mul24(dY, 256 * dx);
            }
            float xf = (float)(256 * dx + (int)(short)q.dz);
            const float zrow = q.zy * (float)(256 * dy + (q.dz >> 16));
            unsigned long long* kp = key;
            const int off = (int)((q.pk >> 5) & ((1u << (PK_SLOT - 5)) - 1u)) + dy * KS + dx;
#pragma unroll
            for (int k = 0; k < SL; ++k) {
                const bool in = !DEEP || k == 0 || dx + k <= (int)(q.pk & 31u);
                if (in && min(e[0], min(e[1], e[2])) > 0) {
                    float z = (q.z0 + q.zx * xf) + zrow;
                    z = fmaxf(z, 0.0f);                 // 0 for negative values and NaN
                    insert_key<DEEP>(kp, off + k, ((unsigned long long)__float_as_uint(z) << 32) | q.t, L);
                }
                e[0] -= a[0];
                e[1] -= a[1];
                e[2] -= a[2];
                xf += 256.0f;                           // (exact)
            }
        }
        wave_sync();
    }
}

// Raster of up to 64 triangles held one per lane (mine: the triangle index,
// valid for lanes below n): the small ones through the wave's stage, then
// the large ones one at a time, their records read from the lanes that hold
// them.
template <int TILE, bool DEEP>
__device__ __forceinline__ void raster_batch(const TriR* __restrict__ R, unsigned mine, unsigned n, int px0,
                                             int py0, int cx1, int cy1, int lane, unsigned long long* key, int L,
                                             RasterStage* stage) {
    TriR r{};
    int x0 = 0, y0 = 0, bw = 1, bh = 0;
    bool large = false;
    if ((unsigned)lane < n) {
        r = gload(&R[mine]);
        int x1, y1;
        tri_box(r, px0, py0, cx1, cy1, x0, x1, y0, y1);
        if (x0 <= x1 && y0 <= y1) {
            large = !(r.flags & TRI_SMALL);
            bw = x1 - x0 + 1;
            bh = large ? 0 : y1 - y0 + 1;
        }
    }
    raster_staged<TILE, DEEP>(stage, r, mine, x0, y0, bw, bh, px0, py0, lane, key, L);
    unsigned long long big = __ballot(large);
    while (big) {
        const int j = __ffsll((long long)big) - 1;
        big &= big - 1ull;
        const int* mw = reinterpret_cast<const int*>(&r);
        TriR q;
        int* qw = reinterpret_cast<int*>(&q);
#pragma unroll
        for (int k = 0; k < (int)(sizeof(TriR) / 4); ++k) qw[k] = __builtin_amdgcn_readlane(mw[k], j);
        raster_tri<TILE, DEEP>(q, __builtin_amdgcn_readlane(mine, j), px0, py0, cx1, cy1, lane, key, L);
    }
}

// Record the largest bin occupancy.  The value only grows, so a workgroup
// that reads a value at least as large (possibly a stale one) may skip the
// atomic: almost all do, and the single counter no longer serialises a
// launch of a hundred thousand workgroups on one L2 channel.
__device__ __forceinline__ void note_max_bin(unsigned long long* stats, unsigned c) {
    unsigned long long seen = stats[ST_MAX_BIN];
    if ((unsigned long long)c > seen) atomicMax(&stats[ST_MAX_BIN], (unsigned long long)c);
}

// A bin of c entries, capacity cap: its overflow and occupancy statistics.
__device__ __forceinline__ void note_bin(unsigned long long* stats, unsigned c, unsigned cap) {
    if (c > cap) atomicAdd(&stats[ST_OVERFLOWS], 1ull);
    note_max_bin(stats, c);
}

// Every triangle of one render that may cover the tile, in batches of up to
// 64 per wave (wave `wave` of nw): the tile's bin of cnt entries; for a bin
// past its capacity the full bin and then the tile's entries of the render's
// spill list, or, when that list ran out of room, every valid triangle of the
// render whose pixel box meets the tile.  The spill list and the render are
// read 64 entries at a time, the hits packed to the low lanes, so the cost is
// a coalesced pass, not one dependent read per entry.  One loop serves the
// three sources, so the raster is compiled in once.  `note`: this wave counts
// a full scan in the statistics.
template <int TILE, bool DEEP>
__device__ __forceinline__ void raster_render(const TriR* __restrict__ R, const unsigned* __restrict__ bin,
                                              unsigned cnt, unsigned cap, const unsigned* spn,
                                              const unsigned long long* __restrict__ spill, int n_tris, int tile,
                                              int wave, int nw, int lane, int px0, int py0, int cx1, int cy1,
                                              unsigned long long* key, int L, RasterStage* stage,
                                              unsigned long long* stats, bool note) {
    enum { BIN, SPILL, SCAN };
    int src = BIN, next = BIN;
    unsigned limit = cnt, ns = 0u;
    if (cnt > cap) {
        limit = cap;
        ns = gload(&spn[0]);
        next = SPILL;
        if (ns > SPILL_CAP) {
            src = next = SCAN;
            limit = (unsigned)n_tris;
            if (note && lane == 0) atomicAdd(&stats[ST_FULL_SCANS], 1ull);
        }
    }
    unsigned base = src == BIN ? (unsigned)wave : 64u * (unsigned)wave;
    for (;; base += 64u * (unsigned)nw) {
        if (base >= limit) {
            if (src == next) break;
            src = next;                                  // the bin is done: the spill list
            limit = ns;
            base = 64u * (unsigned)wave;
            if (base >= limit) break;
        }
        unsigned mine = 0u, n;
        if (src == BIN) {
            // entries wave, wave + nw, wave + 2 nw, ...
            const unsigned k = base + (unsigned)lane * (unsigned)nw;
            if (k < limit) mine = gload(&bin[k]);
            n = min((limit - base + (unsigned)nw - 1u) / (unsigned)nw, 64u);
        } else {
            const unsigned j = base + (unsigned)lane;
            bool hit = false;
            unsigned t = j;
            if (j < limit) {
                if (src == SPILL) {
                    const unsigned long long e = gload(&spill[j]);
                    hit = (unsigned)(e >> 32) == (unsigned)tile;
                    t = (unsigned)e;
                } else {
                    const TriR* q = &R[j];
                    TriR b;                              // corners and flags (the first 28 B)
#pragma unroll
                    for (int k = 0; k < 3; ++k) {
                        b.X[k] = gload(&q->X[k]);
                        b.Y[k] = gload(&q->Y[k]);
                    }
                    int x0 = 1, x1 = 0, y0 = 1, y1 = 0;
                    if (gload(&q->flags) & TRI_VALID) tri_box(b, px0, py0, cx1, cy1, x0, x1, y0, y1);
                    hit = x0 <= x1 && y0 <= y1;
                }
            }
            const unsigned long long m = __ballot(hit);
            if (m == 0ull) continue;
            n = (unsigned)__popcll(m);
            const int below = (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32),
                                                             __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
            // a permutation of the lanes: the hits to the front, in lane order
            const int dst = hit ? below : (int)n + (lane - below);
            mine = (unsigned)__builtin_amdgcn_ds_permute(dst * 4, (int)t);
        }
        raster_batch<TILE, DEEP>(R, mine, n, px0, py0, cx1, cy1, lane, key, L, stage);
    }
}

// After the tile's raster: leave its bin empty for the next use, and the
// last overflowing tile of the render empties the render's spill list.
__device__ __forceinline__ void release_bin(unsigned* counts, int tile, unsigned cap, unsigned* spn) {
    const unsigned c = counts[tile];
    counts[tile] = 0u;
    if (c > cap && spn != nullptr && atomicSub(&spn[1], 1u) == 1u) spn[0] = 0u;
}

// ------------------------------------------------ tile-local aggregation --
//
// Contributions are summed per group inside the workgroup before they reach
// the global accumulators: an open-addressing table in LDS keyed by group
// (int64 sum + uint32 count per slot), flushed with one global atomic pair
// per distinct group of the tile.  Integer sums make the result identical
// to per-pixel global atomics.

#define HASH_EMPTY 0xFFFFFFFFu
#define HASH_PROBES 64

// A slot packs the group's sum and count into one 64-bit word,
// sum * 2^12 + count, so one LDS atomic adds both: a tile has at most 1024
// pixels, so the count stays below 2^12, and |sum| <= 1024 * 2^37 keeps the
// packed word within int64.
#define PACK_SHIFT 12
#define PACK_MASK ((1ull << PACK_SHIFT) - 1ull)

template <int LOG2T>
struct GroupTable {
    unsigned key[1 << LOG2T];
    unsigned long long sum[1 << LOG2T];     // packed sum and count
};

__device__ __forceinline__ unsigned long long pack_sc(long long q, unsigned c) {
    return ((unsigned long long)q << PACK_SHIFT) + (unsigned long long)c;
}

__device__ __forceinline__ void unpack_sc(unsigned long long w, long long& q, unsigned& c) {
    c = (unsigned)(w & PACK_MASK);
    q = (long long)(w - c) >> PACK_SHIFT;
}

__device__ __forceinline__ void global_add(long long* __restrict__ Rp, unsigned* __restrict__ K, long long g,
                                           long long q, unsigned c) {
    if (q != 0)
        __hip_atomic_fetch_add((DRD_GLOBAL unsigned long long*)&Rp[g], (unsigned long long)q, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_fetch_add((DRD_GLOBAL unsigned*)&K[g], c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <int LOG2T>
__device__ __forceinline__ void table_add(GroupTable<LOG2T>& tb, long long* __restrict__ Rp,
                                          unsigned* __restrict__ K, unsigned g, long long q, unsigned c) {
    constexpr unsigned MASK = (1u << LOG2T) - 1u;
    // multiplicative hash in 24-bit multiplies (full rate; the 32-bit one is
    // quarter rate), the high byte folded in first
    unsigned h = (__umul24(g ^ (g >> 24), 0x9E3779u) >> (24 - LOG2T)) & MASK;
    for (int probe = 0; probe < HASH_PROBES; ++probe) {
        unsigned k = __hip_atomic_load(&tb.key[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (k == HASH_EMPTY) k = atomicCAS(&tb.key[h], HASH_EMPTY, g);
        if (k == HASH_EMPTY || k == g) {
            atomicAdd(&tb.sum[h], pack_sc(q, c));
            return;
        }
        h = (h + 1u) & MASK;
    }
    global_add(Rp, K, g, q, c);      // crowded table: go straight to memory
}

// Subdivision surface: pixels whose + and - renders show the same
// tessellated triangle are combined per wave -- lanes with equal triangle
// ids are summed with a butterfly -- and the wave's lanes then share the
// table adds of that triangle's control-vertex list.  Must be called by
// every lane of the wave.
template <int LOG2T>
__device__ __forceinline__ void wave_ctrl(GroupTable<LOG2T>& tb, long long* __restrict__ Rp,
                                          unsigned* __restrict__ K, const DScene& sc, bool active, unsigned tri,
                                          long long q) {
    int lane = threadIdx.x & 63;
    unsigned long long pending = __ballot(active);
    while (pending) {
        int leader = __ffsll((unsigned long long)pending) - 1;
        unsigned lt = __builtin_amdgcn_readfirstlane(__shfl(tri, leader));
        bool mine = active && tri == lt;
        unsigned long long m = __ballot(mine);
        long long v = mine ? q : 0;
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
        unsigned c = (unsigned)__popcll(m);
        int b0 = sc.tri_rowptr[lt], b1 = sc.tri_rowptr[lt + 1];
        for (int j = b0 + lane; j < b1; j += 64) table_add<LOG2T>(tb, Rp, K, (unsigned)sc.tri_cols[j], v, c);
        if (mine) active = false;
        pending &= ~m;
    }
}

// The union of two tessellated triangles' control vertices (both lists
// ascending), each once, for one pixel.
template <int LOG2T>
__device__ __forceinline__ void ctrl_union_add(GroupTable<LOG2T>& tb, long long* __restrict__ Rp,
                                               unsigned* __restrict__ K, const DScene& sc, unsigned t0,
                                               unsigned t1, long long q) {
    int a0 = 0, a1 = 0, b0 = 0, b1 = 0;
    if (t0 != DRD_BG) { a0 = sc.tri_rowptr[t0]; a1 = sc.tri_rowptr[t0 + 1]; }
    if (t1 != DRD_BG) { b0 = sc.tri_rowptr[t1]; b1 = sc.tri_rowptr[t1 + 1]; }
    int i = a0, j = b0;
    while (i < a1 || j < b1) {
        int ga = i < a1 ? sc.tri_cols[i] : 0x7FFFFFFF;
        int gb = j < b1 ? sc.tri_cols[j] : 0x7FFFFFFF;
        int g = ga < gb ? ga : gb;
        if (ga == g) ++i;
        if (gb == g) ++j;
        table_add<LOG2T>(tb, Rp, K, (unsigned)g, q, 1u);
    }
}

// Opaque tile kernels of 8- and 16-pixel tiles are asked for 8 resident
// waves per SIMD (at most 64 VGPRs): 16-pixel tiles hold 18.7 KB of LDS, so
// eight blocks of four waves share a CU's 160 KB.  Larger tiles and deep
// buffers are held to fewer waves by their LDS anyway.
#define TILE_MIN_WAVES 8

template <int TILE>
struct TileCfg {
    static constexpr int LOG2T = TILE == 8 ? 9 : (TILE == 16 ? 10 : 11);
};


// Everything the tile body needs, resolved by the kernel's prologue.
struct TileJob {
    const DScene* sc;
    const DView* vw;
    const float* theta;
    const uint32_t* pb;                  // sign bits of the pair (null: unperturbed)
    const float* eps;                    // per block
    float sgn[2];
    const TriR* recR[2];                 // records of each sign (index = triangle)
    const TriS* recS[2];
    const TriG* recG[2];                 // GGX records of each sign
    unsigned* counts[2];                 // bin counters of each sign (index = tile)
    const unsigned* bins[2];             // bin entries of each sign (tile * cap + k)
    unsigned* spn[2];                    // spill counters of each sign, or null
    const unsigned long long* spill[2];  // spill lists of each sign
    int cap;
    int tile;
    unsigned long long* stats;
    // estimate
    const float* targets;                // this view's target image (image form: dL/dI)
    int img;                             // image form of the per-pixel difference
    long long* Rp;                       // group sums of the pair
    unsigned* K;
    int act_pos, any_act;
    const int* act_cls;
    // render
    float* out_rgb;
    unsigned* out_id;
    float* out_uv;
    // loss
    double* partial;
    // full-image estimate: the pair's total of fixed-point differences
    long long* qtot;
};

// MODE: 0 estimate (both signs, scatter), 1 render (write rgb/id/uv),
// 2 loss (per-tile sum of the per-pixel L2 error f_{w,h}), 3 full-image
// estimate (both signs, per-tile sum of the fixed-point differences).
template <int TILE, int MODE>
struct TileShared {
    static constexpr int NPIX = TILE * TILE;
    static constexpr int PPT = NPIX > 256 ? NPIX / 256 : 1;
    static constexpr int TB = NPIX / PPT;
    static constexpr int NS = (MODE == 0 || MODE == 3) ? 2 : 1;
    static constexpr int LOG2T = MODE == 0 ? TileCfg<TILE>::LOG2T : 1;
    static constexpr int KS = KeyRow<TILE, false>::N;
    unsigned long long key[NS][TILE * KS];
    // the raster's per-wave stages, then (estimate) the group table
    union {
        RasterStage stage[TB / 64];
        GroupTable<LOG2T> table;
    } u;
    double red[MODE == 2 ? TB : 1];
    long long qred[MODE == 3 ? TB : 1];
    unsigned nfl;                        // occupied table slots (flush)
};

template <int TILE, int MODE, int SHADE>
__device__ __forceinline__ void tile_body(const TileJob& J, TileShared<TILE, MODE>& S) {
    using SH = TileShared<TILE, MODE>;
    constexpr int NPIX = SH::NPIX, PPT = SH::PPT, TB = SH::TB, NS = SH::NS;
    constexpr int NW = TB / 64;
    constexpr int LOG2T = SH::LOG2T;
    constexpr int TSIZE = 1 << LOG2T;
    const DScene& sc = *J.sc;
    const DView& vw = *J.vw;
    int tx = J.tile % vw.tiles_x, ty = J.tile / vw.tiles_x;
    int px0 = tx * TILE, py0 = ty * TILE;
    const int cx1 = min(px0 + TILE - 1, vw.W - 1), cy1 = min(py0 + TILE - 1, vw.H - 1);   // last pixel in view
    int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    if constexpr (MODE == 0 || MODE == 3) {
        // no triangle of either render touches the tile: every pixel is
        // background in both, so the tile adds nothing (its bins are empty)
        if ((J.counts[0][J.tile] | J.counts[NS - 1][J.tile]) == 0u) return;
    }
    for (int j = tid; j < NS * TILE * SH::KS; j += TB) (&S.key[0][0])[j] = ~0ull;
    __syncthreads();

    // Both signs' bins: with two signs and several waves, half of the
    // waves take each sign, so the two chains of dependent reads (bin
    // counter, entries, records) run at once; one wave takes both in turn.
    {
        constexpr int SPLIT = (NS == 2 && NW >= 2) ? 2 : 1;
        constexpr int NWS = NW / SPLIT;                  // waves per sign
        const int s_lo = SPLIT == 2 ? wave / NWS : 0;
        const int s_hi = SPLIT == 2 ? s_lo + 1 : NS;
        const int wv = wave - s_lo * NWS;
        for (int s = s_lo; s < s_hi; ++s) {
            // the sign picked by selects: a run-time index into J's arrays
            // would move J to private memory
            const bool s1 = NS == 2 && s == 1;
            const TriR* __restrict__ R = s1 ? J.recR[NS - 1] : J.recR[0];
            const unsigned* bins = s1 ? J.bins[NS - 1] : J.bins[0];
            unsigned* counts = s1 ? J.counts[NS - 1] : J.counts[0];
            const unsigned* spn = s1 ? J.spn[NS - 1] : J.spn[0];
            const unsigned long long* spill = s1 ? J.spill[NS - 1] : J.spill[0];
            unsigned long long* key = s1 ? S.key[NS - 1] : S.key[0];
            unsigned cnt = counts[J.tile];
            if (wv == 0 && lane == 0) note_bin(J.stats, cnt, (unsigned)J.cap);
            raster_render<TILE, false>(R, bins + (long long)J.tile * J.cap, cnt, (unsigned)J.cap, spn, spill,
                                       sc.n_tris, J.tile, wv, NWS, lane, px0, py0, cx1, cy1, key, 1,
                                       &S.u.stage[wave], J.stats, wv == 0);
        }
    }
    __syncthreads();
    if (tid < NS) {                              // leave the bins empty for the next use
        const bool s1 = NS == 2 && tid == 1;
        release_bin(s1 ? J.counts[NS - 1] : J.counts[0], J.tile, (unsigned)J.cap, s1 ? J.spn[NS - 1] : J.spn[0]);
    }
    if constexpr (MODE == 0) {
        // the stages are done with: the group table takes their place
        if (tid == 0) S.nfl = 0u;
        for (int j = tid; j < TSIZE; j += TB) {
            S.u.table.key[j] = HASH_EMPTY;
            S.u.table.sum[j] = 0ull;
        }
    }

    double loss_acc = 0.0;
    long long qsum = 0;
    for (int j = 0; j < PPT; ++j) {
        int local = tid + j * TB;
        int lx = local % TILE, ly = local / TILE;
        int x = px0 + lx, y = py0 + ly;
        bool inpix = x < vw.W && y < vw.H;
        int px = 256 * x + 128, py = 256 * y + 128;
        unsigned id[NS];
        float rgb[NS][3], uv[NS][2];
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            unsigned long long k = inpix ? S.key[s][ly * SH::KS + lx] : ~0ull;
            id[s] = (k == ~0ull) ? DRD_BG : (unsigned)(k & 0xFFFFFFFFull);
            rgb[s][0] = 0.0f; rgb[s][1] = 0.0f; rgb[s][2] = 0.0f;
            uv[s][0] = 0.0f; uv[s][1] = 0.0f;
            if (id[s] != DRD_BG) {
                TriR r = gload(&J.recR[s][id[s]]);
                TriS sh = gload(&J.recS[s][id[s]]);
                CornerUV cu = load_cuv(sc, id[s]);
                float alpha;
                shade_pixel<SHADE, false>(sc, vw, J.theta, J.pb, J.eps, J.sgn[s], r, sh, J.recG[s] + id[s], cu, px, py,
                                          rgb[s], uv[s], alpha);
            }
        }
        long long pix = (long long)y * vw.W + x;
        if constexpr (MODE == 2) {
            if (inpix) {
                const float* tg = J.targets + 3 * pix;
                float dr = rgb[0][0] - tg[0], dg = rgb[0][1] - tg[1], db = rgb[0][2] - tg[2];
                loss_acc += (double)((dr * dr + dg * dg) + db * db);
            }
        } else if constexpr (MODE == 3) {
            if (inpix && (id[0] != DRD_BG || id[1] != DRD_BG)) {
                int flag;
                qsum += quantize(pixel_delta(rgb[0], rgb[1], J.targets + 3 * pix, J.img), flag);
                if (flag) atomicAdd(&J.stats[flag == 1 ? ST_SATURATIONS : ST_NONFINITE], 1ull);
            }
        } else if constexpr (MODE == 1) {
            if (!inpix) continue;
            if (J.out_rgb) {
                J.out_rgb[3 * pix + 0] = rgb[0][0];
                J.out_rgb[3 * pix + 1] = rgb[0][1];
                J.out_rgb[3 * pix + 2] = rgb[0][2];
            }
            if (J.out_id) J.out_id[pix] = id[0];
            if (J.out_uv) {
                J.out_uv[2 * pix + 0] = uv[0][0];
                J.out_uv[2 * pix + 1] = uv[0][1];
            }
        } else {
            // an empty contribution set (background in both renders) adds nothing
            bool act = inpix && (id[0] != DRD_BG || id[1] != DRD_BG) && J.any_act;
            long long q = 0;
            if (act) {
                int flag;
                q = quantize(pixel_delta(rgb[0], rgb[1], J.targets + 3 * pix, J.img), flag);
                if (flag) atomicAdd(&J.stats[flag == 1 ? ST_SATURATIONS : ST_NONFINITE], 1ull);
            }
            if (j == 0) __syncthreads();         // the group table is cleared
            if (J.act_pos && sc.n_ctrl > 0) {
                bool same = act && id[0] == id[1];
                wave_ctrl<LOG2T>(S.u.table, J.Rp, J.K, sc, same, id[0], q);
                if (act && !same) ctrl_union_add<LOG2T>(S.u.table, J.Rp, J.K, sc, id[0], id[1], q);
            } else if (J.act_pos && act) {
                // the union of the two renders' triangles' vertices, each once
                int v0[3] = {-1, -1, -1};
                if (id[0] != DRD_BG) {
#pragma unroll
                    for (int k = 0; k < 3; ++k) {
                        v0[k] = gload(&sc.tri[3 * (long long)id[0] + k]);
                        table_add<LOG2T>(S.u.table, J.Rp, J.K, (unsigned)v0[k], q, 1u);
                    }
                }
                if (id[1] != DRD_BG && id[1] != id[0]) {
#pragma unroll
                    for (int k = 0; k < 3; ++k) {
                        int g = gload(&sc.tri[3 * (long long)id[1] + k]);
                        bool dup = (g == v0[0]) || (g == v0[1]) || (g == v0[2]);
                        if (!dup) table_add<LOG2T>(S.u.table, J.Rp, J.K, (unsigned)g, q, 1u);
                    }
                }
            }
            if (act) {
                for (int c = 0; c < sc.n_cls; ++c) {
                    if (!J.act_cls[c]) continue;
                    int W = sc.cls_w[c], H = sc.cls_h[c];
                    unsigned base = (unsigned)sc.cls_goff[c];
                    unsigned gs[NS][4];
#pragma unroll
                    for (int s = 0; s < NS; ++s) {
                        gs[s][0] = gs[s][1] = gs[s][2] = gs[s][3] = HASH_EMPTY;
                        if (id[s] == DRD_BG) continue;
                        Foot f = footprint(uv[s][0], uv[s][1], W, H);
                        if (sc.tex_mode == 1) {
                            int xn = (f.fx >= 0.5f) ? f.xb : f.xa;
                            int yn = (f.fy >= 0.5f) ? f.yb : f.ya;
                            gs[s][0] = base + (__umul24((unsigned)yn, (unsigned)W) + (unsigned)xn);
                        } else {
                            gs[s][0] = base + (__umul24((unsigned)f.ya, (unsigned)W) + (unsigned)f.xa);
                            gs[s][1] = base + (__umul24((unsigned)f.ya, (unsigned)W) + (unsigned)f.xb);
                            gs[s][2] = base + (__umul24((unsigned)f.yb, (unsigned)W) + (unsigned)f.xa);
                            gs[s][3] = base + (__umul24((unsigned)f.yb, (unsigned)W) + (unsigned)f.xb);
                        }
                    }
#pragma unroll
                    for (int s = 0; s < NS; ++s)
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            unsigned g = gs[s][k];
                            if (g == HASH_EMPTY) continue;
                            bool dup = false;
#pragma unroll
                            for (int j2 = 0; j2 < 4; ++j2)
                                if (j2 < k && gs[s][j2] == g) dup = true;
                            if (s == 1) {
#pragma unroll
                                for (int j2 = 0; j2 < 4; ++j2)
                                    if (gs[0][j2] == g) dup = true;
                            }
                            if (!dup) table_add<LOG2T>(S.u.table, J.Rp, J.K, g, q, 1u);
                        }
                }
            }
        }
    }
    if constexpr (MODE == 2) {
        // fixed-order tree reduction of the tile's per-pixel errors
        S.red[tid] = loss_acc;
        __syncthreads();
        for (int w = TB / 2; w > 0; w >>= 1) {
            if (tid < w) S.red[tid] = S.red[tid] + S.red[tid + w];
            __syncthreads();
        }
        if (tid == 0) *J.partial = S.red[0];
    }
    if constexpr (MODE == 3) {
        // integer sums: the order of the additions does not matter
        S.qred[tid] = qsum;
        __syncthreads();
        for (int w = TB / 2; w > 0; w >>= 1) {
            if (tid < w) S.qred[tid] = S.qred[tid] + S.qred[tid + w];
            __syncthreads();
        }
        if (tid == 0 && S.qred[0] != 0) atomicAdd((unsigned long long*)J.qtot, (unsigned long long)S.qred[0]);
    }
    if constexpr (MODE == 0) {
        __syncthreads();
        if constexpr (TILE >= 16) {
            // occupied slots first gathered into a dense list (in the key
            // buffers, free by now and large enough from 16-pixel tiles
            // on), so the global atomics go out in full waves
            unsigned* list = reinterpret_cast<unsigned*>(&S.key[0][0]);
            for (int j = tid; j < TSIZE; j += TB) {
                bool occ = S.u.table.key[j] != HASH_EMPTY;
                unsigned long long m = __ballot(occ);
                unsigned base = 0;
                if (lane == 0 && m) base = atomicAdd(&S.nfl, (unsigned)__popcll(m));
                base = __shfl(base, 0);
                if (occ) list[base + __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u))] = (unsigned)j;
            }
            __syncthreads();
            unsigned n = S.nfl;
            for (unsigned i = (unsigned)tid; i < n; i += TB) {
                unsigned j = list[i];
                long long q;
                unsigned c;
                unpack_sc(S.u.table.sum[j], q, c);
                global_add(J.Rp, J.K, (long long)S.u.table.key[j], q, c);
            }
        } else {
            for (int j = tid; j < TSIZE; j += TB) {
                unsigned g = S.u.table.key[j];
                if (g != HASH_EMPTY) {
                    long long q;
                    unsigned c;
                    unpack_sc(S.u.table.sum[j], q, c);
                    global_add(J.Rp, J.K, (long long)g, q, c);
                }
            }
        }
    }
}


// ------------------------------------------------- semi-transparent tile --
//
// Sec. 4.4 "Transparent geometry": the raster keeps, per pixel and sign,
// the L nearest fragments in front-to-back order (a deep ID buffer in LDS,
// built by the atomic-min cascade of raster_tri), the shading pass
// composites them over black, C = sum_l T_l alpha_l c_l with
// T_{l+1} = T_l (1 - alpha_l), and the scatter credits the union over both
// renders and all listed layers of the layers' vertices and footprint
// texels, each group once per pixel.  Tiles are 8 or 16 pixels (one pixel
// per lane).

template <int TILE, int MODE>
struct DeepShared {
    static constexpr int NPIX = TILE * TILE;
    static constexpr int TB = NPIX;
    static constexpr int NS = (MODE == 0 || MODE == 3) ? 2 : 1;
    static constexpr int LOG2T = MODE == 0 ? TileCfg<TILE>::LOG2T : 1;
    unsigned long long key[NS][NPIX * DRD_MAX_LAYERS];
    // the raster's per-wave stages, then (estimate) the group table
    union {
        RasterStage stage[TB / 64 > 0 ? TB / 64 : 1];
        GroupTable<LOG2T> table;
    } u;
    double red[MODE == 2 ? TB : 1];
    long long qred[MODE == 3 ? TB : 1];
};

// Texel groups of one fragment in class c: the bilinear footprint, or the
// nearest texel (the other entries HASH_EMPTY).
__device__ __forceinline__ void texel_groups(const DScene& sc, int c, float u, float v, unsigned* gs) {
    int W = sc.cls_w[c], H = sc.cls_h[c];
    unsigned base = (unsigned)sc.cls_goff[c];
    Foot f = footprint(u, v, W, H);
    if (sc.tex_mode == 1) {
        int xn = (f.fx >= 0.5f) ? f.xb : f.xa;
        int yn = (f.fy >= 0.5f) ? f.yb : f.ya;
        gs[0] = base + (__umul24((unsigned)yn, (unsigned)W) + (unsigned)xn);
        gs[1] = gs[2] = gs[3] = HASH_EMPTY;
    } else {
        gs[0] = base + (__umul24((unsigned)f.ya, (unsigned)W) + (unsigned)f.xa);
        gs[1] = base + (__umul24((unsigned)f.ya, (unsigned)W) + (unsigned)f.xb);
        gs[2] = base + (__umul24((unsigned)f.yb, (unsigned)W) + (unsigned)f.xa);
        gs[3] = base + (__umul24((unsigned)f.yb, (unsigned)W) + (unsigned)f.xb);
    }
}

template <int TILE, int MODE, int SHADE>
__device__ __forceinline__ void tile_body_deep(const TileJob& J, DeepShared<TILE, MODE>& S) {
    using SH = DeepShared<TILE, MODE>;
    constexpr int NPIX = SH::NPIX, TB = SH::TB, NS = SH::NS;
    constexpr int NW = TB / 64 > 0 ? TB / 64 : 1;
    constexpr int LOG2T = SH::LOG2T;
    constexpr int TSIZE = 1 << LOG2T;
    constexpr int LM = DRD_MAX_LAYERS;
    constexpr int NE = NS * LM;                    // fragment entries per pixel
    const DScene& sc = *J.sc;
    const DView& vw = *J.vw;
    const int L = sc.layers;
    int tx = J.tile % vw.tiles_x, ty = J.tile / vw.tiles_x;
    int px0 = tx * TILE, py0 = ty * TILE;
    const int cx1 = min(px0 + TILE - 1, vw.W - 1), cy1 = min(py0 + TILE - 1, vw.H - 1);   // last pixel in view
    int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    if constexpr (MODE == 0 || MODE == 3) {
        // no fragment in either render: the tile adds nothing
        if ((J.counts[0][J.tile] | J.counts[NS - 1][J.tile]) == 0u) return;
    }
    for (int j = tid; j < NS * NPIX * LM; j += TB) (&S.key[0][0])[j] = ~0ull;
    __syncthreads();

#pragma unroll
    for (int s = 0; s < NS; ++s) {
        unsigned cnt = J.counts[s][J.tile];
        if (tid == 0) note_bin(J.stats, cnt, (unsigned)J.cap);
        const TriR* __restrict__ R = J.recR[s];
        raster_render<TILE, true>(R, J.bins[s] + (long long)J.tile * J.cap, cnt, (unsigned)J.cap, J.spn[s],
                                  J.spill[s], sc.n_tris, J.tile, wave, NW, lane, px0, py0, cx1, cy1, S.key[s], L,
                                  &S.u.stage[wave], J.stats, wave == 0);
    }
    __syncthreads();
    if (tid == 0) {
#pragma unroll
        for (int s = 0; s < NS; ++s) release_bin(J.counts[s], J.tile, (unsigned)J.cap, J.spn[s]);
    }
    if constexpr (MODE == 0) {
        // the stages are done with: the group table takes their place
        for (int j = tid; j < TSIZE; j += TB) {
            S.u.table.key[j] = HASH_EMPTY;
            S.u.table.sum[j] = 0ull;
        }
    }

    int local = tid;
    int lx = local % TILE, ly = local / TILE;
    int x = px0 + lx, y = py0 + ly;
    bool inpix = x < vw.W && y < vw.H;
    int px = 256 * x + 128, py = 256 * y + 128;
    long long pix = (long long)y * vw.W + x;
    // Lists fill from the front, so a list is empty when its first layer is.
    // The loops over layers stay rolled (the fragments are re-read from the
    // LDS list, their UVs recomputed where needed) so that nothing indexed
    // by layer has to live in registers.
    float rgb[NS][3];
    bool any = false;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        rgb[s][0] = 0.0f; rgb[s][1] = 0.0f; rgb[s][2] = 0.0f;
        float T = 1.0f;
        for (int l = 0; l < L; ++l) {
            unsigned long long k = inpix ? S.key[s][local * LM + l] : ~0ull;
            unsigned id = (k == ~0ull) ? DRD_BG : (unsigned)(k & 0xFFFFFFFFull);
            float uv[2] = {0.0f, 0.0f};
            if (id != DRD_BG) {
                any = true;
                TriR r = gload(&J.recR[s][id]);
                TriS sh = gload(&J.recS[s][id]);
                CornerUV cu = load_cuv(sc, id);
                float c[3], al;
                shade_pixel<SHADE, true>(sc, vw, J.theta, J.pb, J.eps, J.sgn[s], r, sh, J.recG[s] + id, cu, px, py, c,
                                         uv, al);
                float wt = T * al;
                rgb[s][0] = rgb[s][0] + wt * c[0];
                rgb[s][1] = rgb[s][1] + wt * c[1];
                rgb[s][2] = rgb[s][2] + wt * c[2];
                T = T * (1.0f - al);
            }
            if constexpr (MODE == 1) {
                if (inpix) {
                    long long e = pix * L + l;
                    if (J.out_id) J.out_id[e] = id;
                    if (J.out_uv) {
                        J.out_uv[2 * e + 0] = uv[0];
                        J.out_uv[2 * e + 1] = uv[1];
                    }
                }
            }
        }
    }

    if constexpr (MODE == 1) {
        if (inpix && J.out_rgb) {
            J.out_rgb[3 * pix + 0] = rgb[0][0];
            J.out_rgb[3 * pix + 1] = rgb[0][1];
            J.out_rgb[3 * pix + 2] = rgb[0][2];
        }
        return;
    }
    if constexpr (MODE == 2) {
        double loss_acc = 0.0;
        if (inpix) {
            const float* tg = J.targets + 3 * pix;
            float dr = rgb[0][0] - tg[0], dg = rgb[0][1] - tg[1], db = rgb[0][2] - tg[2];
            loss_acc = (double)((dr * dr + dg * dg) + db * db);
        }
        S.red[tid] = loss_acc;
        __syncthreads();
        for (int w = TB / 2; w > 0; w >>= 1) {
            if (tid < w) S.red[tid] = S.red[tid] + S.red[tid + w];
            __syncthreads();
        }
        if (tid == 0) *J.partial = S.red[0];
        return;
    }
    if constexpr (MODE == 3) {
        long long qsum = 0;
        if (inpix && any) {
            int flag;
            qsum = quantize(pixel_delta(rgb[0], rgb[1], J.targets + 3 * pix, J.img), flag);
            if (flag) atomicAdd(&J.stats[flag == 1 ? ST_SATURATIONS : ST_NONFINITE], 1ull);
        }
        S.qred[tid] = qsum;
        __syncthreads();
        for (int w = TB / 2; w > 0; w >>= 1) {
            if (tid < w) S.qred[tid] = S.qred[tid] + S.qred[tid + w];
            __syncthreads();
        }
        if (tid == 0 && S.qred[0] != 0) atomicAdd((unsigned long long*)J.qtot, (unsigned long long)S.qred[0]);
        return;
    }
    if constexpr (MODE == 0) {
        __syncthreads();                             // the group table is cleared
        bool act = inpix && any && J.any_act;
        if (act) {
            int flag;
            long long q = quantize(pixel_delta(rgb[0], rgb[1], J.targets + 3 * pix, J.img), flag);
            if (flag) atomicAdd(&J.stats[flag == 1 ? ST_SATURATIONS : ST_NONFINITE], 1ull);
            // fragment e = s * L + l; each group is added by the first
            // fragment that holds it
            const int NF = NS * L;
            for (int e = 0; e < NF; ++e) {
                int s1 = e / L, l1 = e % L;
                unsigned long long k1 = (&S.key[0][0])[(s1 * NPIX + local) * LM + l1];
                if (k1 == ~0ull) continue;
                unsigned id1 = (unsigned)(k1 & 0xFFFFFFFFull);
                if (J.act_pos) {
                    int v1[3];
#pragma unroll
                    for (int k = 0; k < 3; ++k) v1[k] = gload(&sc.tri[3 * (long long)id1 + k]);
                    bool dup[3] = {false, false, false};
                    for (int e2 = 0; e2 < e; ++e2) {
                        unsigned long long k2 = (&S.key[0][0])[((e2 / L) * NPIX + local) * LM + e2 % L];
                        if (k2 == ~0ull) continue;
                        const int* t2 = sc.tri + 3 * (long long)(unsigned)(k2 & 0xFFFFFFFFull);
                        int v2[3] = {gload(&t2[0]), gload(&t2[1]), gload(&t2[2])};
#pragma unroll
                        for (int k = 0; k < 3; ++k)
                            dup[k] = dup[k] || v1[k] == v2[0] || v1[k] == v2[1] || v1[k] == v2[2];
                    }
#pragma unroll
                    for (int k = 0; k < 3; ++k)
                        if (!dup[k]) table_add<LOG2T>(S.u.table, J.Rp, J.K, (unsigned)v1[k], q, 1u);
                }
                if (J.any_act && sc.n_cls > 0) {
                    Attr a1 = frag_attr(sc, (s1 ? J.recR[1] : J.recR[0])[id1], (s1 ? J.recS[1] : J.recS[0])[id1],
                                        load_cuv(sc, id1), px, py);
                    for (int c = 0; c < sc.n_cls; ++c) {
                        if (!J.act_cls[c]) continue;
                        unsigned gs[4];
                        texel_groups(sc, c, a1.u, a1.v, gs);
                        bool dup[4];
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            dup[k] = gs[k] == HASH_EMPTY;
#pragma unroll
                            for (int k2 = 0; k2 < 4; ++k2)
                                if (k2 < k && gs[k2] == gs[k]) dup[k] = true;
                        }
                        for (int e2 = 0; e2 < e; ++e2) {
                            unsigned long long k2 = (&S.key[0][0])[((e2 / L) * NPIX + local) * LM + e2 % L];
                            if (k2 == ~0ull) continue;
                            unsigned id2 = (unsigned)(k2 & 0xFFFFFFFFull);
                            Attr a2 = frag_attr(sc, (e2 >= L ? J.recR[1] : J.recR[0])[id2],
                                                (e2 >= L ? J.recS[1] : J.recS[0])[id2], load_cuv(sc, id2), px, py);
                            unsigned gs2[4];
                            texel_groups(sc, c, a2.u, a2.v, gs2);
#pragma unroll
                            for (int k = 0; k < 4; ++k)
                                dup[k] = dup[k] || gs[k] == gs2[0] || gs[k] == gs2[1] || gs[k] == gs2[2] ||
                                         gs[k] == gs2[3];
                        }
#pragma unroll
                        for (int k = 0; k < 4; ++k)
                            if (!dup[k]) table_add<LOG2T>(S.u.table, J.Rp, J.K, gs[k], q, 1u);
                    }
                }
            }
        }
        __syncthreads();
        for (int j = tid; j < TSIZE; j += TB) {
            unsigned g = S.u.table.key[j];
            if (g != HASH_EMPTY) {
                long long q;
                unsigned c;
                unpack_sc(S.u.table.sum[j], q, c);
                global_add(J.Rp, J.K, (long long)g, q, c);
            }
        }
    }
}

// One (item, tile) of a single-scene launch: opaque or semi-transparent
// body, specialised for the scene's shading (three kernels of 43 to 52 KB of
// code and 56 registers in place of one of 90 KB and 77: the instruction
// cache holds 64 KB).  The job is built here, in the kernel itself, so that the argument
// block is read in place from the kernel-argument segment (scalar loads).
//
// interleave: the grid walks the call's tile units in (view, tile, pair)
// order, so the pairs of one tile follow each other, run at about the same
// time on one XCD and share its L2 for what they have in common: the texels
// and target pixels of the tile.  Otherwise the grid is (tile, item).
// Measured at 1024 px, 46080 triangles, GGX, 32 items: 1989 -> 1586 us
// (specialised and interleaved; the interleaved general kernel 1640 us).
template <int TILE, int MODE, bool DEEP, int SHADE>
__global__ void __launch_bounds__((TILE * TILE > 256) ? 256 : TILE * TILE, (DEEP || TILE > 16) ? 1 : TILE_MIN_WAVES)
k_tile(TileArgs a) {
    using SH = std::conditional_t<DEEP, DeepShared<TILE, MODE>, TileShared<TILE, MODE>>;
    __shared__ SH S;
    constexpr int NS = SH::NS;
    const DScene& sc = a.sc;
    int li, pair, view, tile;
    if (a.interleave) {
        const unsigned P = (unsigned)a.n_items / (unsigned)a.n_views;
        const unsigned L = (unsigned)xcd_tile(blockIdx.x, gridDim.x);
        view = 0;
        while (view + 1 < a.n_views && L >= P * (unsigned)a.views.tsum[view + 1]) ++view;
        const unsigned r = L - P * (unsigned)a.views.tsum[view];
        tile = (int)(r / P);
        pair = (int)(r - (unsigned)tile * P);
        li = pair * a.n_views + view;
    } else {
        li = blockIdx.y;
        const int item = a.item0 + li;
        pair = item / a.n_views;
        view = item - pair * a.n_views;
        tile = xcd_tile(blockIdx.x, gridDim.x);
    }
    const DView& vw = a.views.v[view];
    if (tile >= vw.tiles_x * vw.tiles_y) return;
    TileJob J;
    J.sc = &a.sc;
    J.vw = &vw;
    J.theta = a.theta;
    J.pb = a.pert.bits ? a.pert.bits + (long long)pair * sc.words : nullptr;
    J.eps = a.pert.eps;
    J.sgn[0] = a.sgn[0];
    J.sgn[1] = a.sgn[1];
    const int gslot = (pair - a.item0 / a.n_views) * NS;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const int s1 = s < NS ? s : 0;
        const int slot = li * NS + s1;
        const long long base = bin_base(a.whole, a.views, a.n_views, NS, a.max_tiles, li, s1);
        J.recR[s] = a.recR + (long long)slot * sc.n_tris;
        J.recS[s] = a.recS + (long long)slot * sc.n_tris;
        J.recG[s] = a.recG + (long long)(gslot + s1) * sc.n_tris;
        J.counts[s] = a.counts + base;
        J.bins[s] = a.bins + base * a.cap;
        J.spn[s] = a.spn + 2ll * slot;
        J.spill[s] = a.spill + (long long)slot * SPILL_CAP;
    }
    J.cap = a.cap;
    J.tile = tile;
    J.stats = a.stats;
    J.targets = a.targets ? a.targets + vw.tgt_off : nullptr;
    J.img = a.img_grad;
    J.Rp = (MODE == 0) ? a.R + (long long)pair * sc.G : nullptr;
    J.K = a.K;
    J.act_pos = a.act_pos;
    J.any_act = a.any_act;
    J.act_cls = a.act_cls;
    J.out_rgb = a.out_rgb;
    J.out_id = a.out_id;
    J.out_uv = a.out_uv;
    J.partial = a.partials ? a.partials + (long long)li * a.max_tiles + tile : nullptr;
    J.qtot = (MODE == 3) ? a.qtot + pair : nullptr;
    if constexpr (DEEP) tile_body_deep<TILE, MODE, SHADE>(J, S);
    else tile_body<TILE, MODE, SHADE>(J, S);
}

// Raster / shade / scatter of every (scene, pair, view, tile) unit of a
// batch of several scenes: one workgroup per unit, units in the XCD-aware
// order of xcd_tile(), items of the costliest scenes first.
template <int TILE, int SHADE>
__global__ void __launch_bounds__((TILE * TILE > 256) ? 256 : TILE * TILE, TILE > 16 ? 1 : TILE_MIN_WAVES)
k_tile_b(BatchArgs b) {
    __shared__ TileShared<TILE, 0> S;
    const long long w = b.unit0 + xcd_tile(blockIdx.x, gridDim.x);
    if (w >= b.total_tiles) return;
    const int it = __builtin_amdgcn_readfirstlane(last_le((const char*)&b.items[0].tile0, sizeof(BItem), b.n_items, w));
    const BItem& I = b.items[it];
    const BScene& Sc = b.scenes[I.scene];
    const DScene& sc = Sc.sc;
    const DView& vw = b.views[I.view];
    const int tiles = vw.tiles_x * vw.tiles_y;
    TileJob J;
    J.sc = &sc;
    J.vw = &vw;
    J.theta = Sc.theta;
    J.pb = Sc.bits + (long long)I.pair * sc.words;
    J.eps = Sc.eps;
    J.sgn[0] = 1.0f;
    J.sgn[1] = -1.0f;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        J.recR[s] = b.recR + I.rec_off + (long long)s * sc.n_tris;
        J.recS[s] = b.recS + I.rec_off + (long long)s * sc.n_tris;
        J.recG[s] = b.recG + I.g_off + (long long)s * sc.n_tris;
        J.counts[s] = b.counts + I.cnt_off + (long long)s * tiles;
        J.bins[s] = b.bins + I.bin_off + (long long)s * tiles * I.cap;
        J.spn[s] = b.spn + 2 * (I.sp_off + s);
        J.spill[s] = b.spill + (I.sp_off + s) * SPILL_CAP;
    }
    J.cap = I.cap;
    J.tile = (int)(w - I.tile0);
    J.stats = b.stats;
    J.targets = Sc.targets + vw.tgt_off;
    J.img = 0;
    J.Rp = Sc.R + (long long)I.pair * sc.G;
    J.K = Sc.K;
    J.act_pos = Sc.act_pos;
    J.any_act = Sc.any_act;
    J.act_cls = Sc.act_cls;
    J.out_rgb = nullptr;
    J.out_id = nullptr;
    J.out_uv = nullptr;
    J.partial = nullptr;
    J.qtot = nullptr;
    tile_body<TILE, 0, SHADE>(J, S);
}

template <int TILE, bool DEEP, int SHADE>
static void launch_tile_mode(hipStream_t st, const TileArgs& a, int mode, dim3 grid) {
    dim3 block((TILE * TILE > 256) ? 256 : TILE * TILE);
    if (mode == 0) hipLaunchKernelGGL((k_tile<TILE, 0, DEEP, SHADE>), grid, block, 0, st, a);
    else if (mode == 1) hipLaunchKernelGGL((k_tile<TILE, 1, DEEP, SHADE>), grid, block, 0, st, a);
    else if (mode == 2) hipLaunchKernelGGL((k_tile<TILE, 2, DEEP, SHADE>), grid, block, 0, st, a);
    else hipLaunchKernelGGL((k_tile<TILE, 3, DEEP, SHADE>), grid, block, 0, st, a);
}

template <int TILE, bool DEEP>
static hipError_t launch_tile_shade(hipStream_t st, const TileArgs& a, int mode, dim3 grid) {
    const int shade = scene_shade(a.sc);
    if (shade == 0) launch_tile_mode<TILE, DEEP, 0>(st, a, mode, grid);
    else if (shade == 1) launch_tile_mode<TILE, DEEP, 1>(st, a, mode, grid);
    else if (shade == 2) launch_tile_mode<TILE, DEEP, 2>(st, a, mode, grid);
    else launch_tile_mode<TILE, DEEP, SHADE_ANY>(st, a, mode, grid);
    return hipGetLastError();
}

template <int TILE>
hipError_t launch_tile_t(hipStream_t st, const TileArgs& a, int mode, dim3 grid) {
    return launch_tile_shade<TILE, false>(st, a, mode, grid);
}

template <int TILE>
hipError_t launch_tile_deep_t(hipStream_t st, const TileArgs& a, int mode, dim3 grid) {
    return launch_tile_shade<TILE, true>(st, a, mode, grid);
}

template <int TILE>
hipError_t launch_batch_tile_t(hipStream_t st, const BatchArgs& b, unsigned grid) {
    dim3 block((TILE * TILE > 256) ? 256 : TILE * TILE);
    if (b.shade == 0) hipLaunchKernelGGL((k_tile_b<TILE, 0>), dim3(grid), block, 0, st, b);
    else if (b.shade == 1) hipLaunchKernelGGL((k_tile_b<TILE, 1>), dim3(grid), block, 0, st, b);
    else if (b.shade == 2) hipLaunchKernelGGL((k_tile_b<TILE, 2>), dim3(grid), block, 0, st, b);
    else hipLaunchKernelGGL((k_tile_b<TILE, SHADE_ANY>), dim3(grid), block, 0, st, b);
    return hipGetLastError();
}
