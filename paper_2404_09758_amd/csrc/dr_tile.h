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

// Offer depth|id key k to pixel li of the tile.  Opaque (LM 0): key[pixel] keeps
// the least (64-bit atomic min).  Deep: key[pixel * LM + l] keeps the L <= LM
// least keys in order, by an atomic-min cascade -- the key is offered to layer
// 0, and whichever of the offered and the resident key is larger moves on to
// the next layer (an empty slot ends the cascade).  Every layer thus ends with
// the least key that reached it, i.e. the l-th least key of the pixel, whatever
// the interleaving of the lanes and waves.
template <int LM>
__device__ __forceinline__ void insert_key(unsigned long long* key, int li, unsigned long long k, int L) {
    if constexpr (LM > 0) {
        unsigned long long* list = key + li * LM;
        for (int l = 0; l < L; ++l) {
            unsigned long long old = atomicMin(&list[l], k);
            if (old == ~0ull) break;
            k = old > k ? old : k;
        }
    } else {
        atomicMin(&key[li], k);
    }
}

// Work split of one tile.  Opaque: a thread takes a pixel and shades both its
// signs, so the two chains of dependent reads overlap (the loss of a 32-pixel
// tile: four pixels, which keeps the order of its sum; MODE 3 of one: four,
// where there are blocks enough, see launch_tile_mode).  Deep: a thread takes
// one side of a pixel, lanes l and l + 32 of a wave holding the + and - side;
// half the layers per thread.
template <int TILE, int MODE, int LM>
struct TileCfg {
    static constexpr bool DEEP = LM > 0;
    static constexpr int NS = (MODE == 0 || MODE >= 3) ? 2 : 1;
    static constexpr int NPIX = TILE * TILE;
    static constexpr int TB = DEEP ? NS * NPIX : ((MODE == 2 || MODE == 3) && NPIX > 256 ? 256 : NPIX);
    static constexpr int NW = TB / 64;
    // the group table: slots without and with a texel box beside them, and
    // the box's texels.  Up to two layers leave room for twice the slots at the
    // same occupancy (512 px, two layers, 32 items: 674 -> 644 us); with four
    // they would cost two of eight waves (900 x 800, three layers: 753 -> 854).
    static constexpr int LOG2T = (TILE == 8 ? 8 : (TILE == 16 ? 10 : 11)) + (LM == 2 ? 1 : 0);
    static constexpr int LOG2B = TILE == 8 ? 7 : (TILE == 16 ? 9 : 10);
    static constexpr int BOX = DEEP ? 0 : TILE == 8 ? 320 : (TILE == 16 ? 1120 : 1536);
    // triangles rasterised at a time: tiles at a silhouette hold 200 to 250, and
    // end the launch when they take a second batch (192 against 256, whole
    // steps: launches of one 512 px item 3265 / 3088 us, 12 uneven scenes
    // 1195 / 1175, two layers 644 / 638, others even); four layers' keys leave
    // room for 192.  32-pixel tiles hold four times as many, and wait for each
    // batch (128 against 256, one render of 11520 triangles at 64 px 72 / 46 us,
    // four pairs of them 243 / 180); MODE 3 of them is held to fewer blocks by the
    // larger stage (1024 px, two views x 16 pairs 546 / 614)
    static constexpr int NEMAX = LM == 4 ? 192 : (TILE == 32 && MODE == 3 ? 128 : 256);
    static constexpr int NE = TB < NEMAX ? TB : NEMAX;
};

// Keys per row of a tile: spare ones after its pixels for opaque tiles, since
// a raster slot that starts at the row's last pixel runs three past it.
template <int TILE, bool DEEP>
struct KeyRow {
    static constexpr int N = DEEP ? TILE : TILE + 4;
};

// LDS staging of a batch of small triangles for the raster (48 B each, three
// 16-byte reads): edge k over the triangle's clipped bounding box is
// e_k(dx, dy) = 256 dX_k dy - 256 dY_k dx + c_k at pixel (x0 + dx, y0 + dy).
// 16-bit fields hold differences of snapped corners, which a TRI_SMALL
// triangle keeps within +-2^15.
struct __align__(16) PTri {
    int c[3];            // edge k at the box's corner pixel, plus 1 on a top-left edge
    unsigned t;
    int d[3];            // dX_k (low half), dY_k (high half)
    unsigned pk;         // box width - 1, key index of the corner pixel, first slot (PackBits)
    float z0, zx, zy;    // depth plane
    int dz;              // corner pixel centre minus vertex 0, in subpixels: x low, y high
};
// PTri::pk, from bit 0: box width - 1, for 32-pixel tiles in whole slots (their
// batch has up to 2^16 slots); 12 bits of key index; the triangle's first slot.
template <int TILE>
struct PackBits {
    static constexpr int DROP = TILE == 32 ? 2 : 0, KEY = 5 - DROP, SLOT = KEY + 12;
};

static_assert(sizeof(PTri) == 48, "PTri layout");

template <int TILE, int NE, int NW>
struct RasterShared {
    union {
        PTri tri[NE];
        unsigned hit[NE];        // overflowing bins: triangles found (bit 31: sign), until they are staged
    };
    // bit i: a triangle begins at slot i of the batch
    unsigned long long begin[NE * TILE * (TILE / 4) / 64];
    unsigned wtot[NW];           // slots and triangles staged by each wave
    unsigned nbig;               // large triangles of the batch: tri[NE - 1 - i].t (bit 31: sign)
    unsigned nhit;
};

// Where one tile's triangles come from: counters, bins, records and spill
// lists of the two signs (sign 1's follow sign 0's at a fixed distance).
struct RasterJob {
    const TriR* rec;             // [NS, n_tris]
    int n_tris;
    unsigned* counts;            // of the tile; sign 1's tstride further
    const unsigned* bins;        // of the tile; sign 1's tstride * cap further
    long long tstride;
    int cap;
    unsigned* spn;               // [NS, 2]
    const unsigned long long* spill;   // [NS, SPILL_CAP]
    int tile;
    int px0, py0, cx1, cy1;      // the tile's pixels that lie in the view
    unsigned long long* stats;
};

// Rasterise the tile's triangles of both signs into key[] (sign 1's keys
// TILE * KeyRow further).
//
// Batches of up to NE triangles, the bins of both signs laid end to end, go
// through LDS: each thread stages one triangle; its clipped box is cut into
// slots of RASTER_SLOT horizontally adjacent pixels (a row of w pixels gives
// ceil(w / RASTER_SLOT) slots), the batch's slots are laid end to end over
// the block, and each wave takes an even share of them, one slot per lane and
// pass: one read of the staged record and one index computation serve all the
// slot's pixels.  The triangle of a slot is the number of triangles begun up
// to it: a bit per slot marks the beginnings, so a pass reads its 64 bits
// (the same for all lanes) and counts the ones up to each lane.  Edge values
// are exact: a TRI_SMALL triangle spans less than 32000 subpixels, so at every
// pixel of the box and up to three to its right both products of an edge
// function stay below 2^30 + 2^25 in magnitude and the edge value (plus 1)
// fits in 32 bits; the wrapped 32-bit sums equal it, as do the slot's further
// pixels' values, each its left neighbour's minus 256 dY.
// e > 0 || (e == 0 && top-left) is e + [top-left] > 0.  A slot's pixels beyond
// the box are not covered, unless the box was clipped at the tile's or the
// view's edge: those keys fall on the row's spare columns, or on pixels that
// are not in the view and are not read (opaque; deep tiles test the box).
// Large triangles of a batch follow one at a time, 64 pixels per wave.
//
// Entries of a bin past its capacity are in the render's spill list, or, when
// that list ran out of room, anywhere in the render: the waves look through
// either up to 192 entries at a time and gather the tile's into batches.  A scan's
// batch goes once a wave's hits find no room in it: neighbouring triangles cover
// the same tile, so one wave's look is often all hits, and others that went on
// looking kept it waiting (162000 triangles at 256 px: one render with 32 px tiles
// 568 -> 232 us, 4 pairs of renders 2037 -> 1118, with 16 px tiles 2036 -> 1661).
// A spill list is short, and its batches are better full (2 to 6 %).
//
// Bound by vector issue, in small launches by the latency of its chain.
// Staging by the block instead of by each wave for its own share of one
// sign's bin: every triangle is staged by a full wave and the passes are even
// over the waves whatever the bins hold.  Slots of 4 pixels: measured on the
// paper-scale step against 2, 3, 6 and 8 (2 -> 4: tile kernel -2 % at the
// start of an optimisation run, -9 % after 50 Adam steps, when the triangles
// have grown; 6 and 8 within 2 % of 4).
#define RASTER_SLOT 4
#define HITS_FULL 0x80000000u    // (nhit) a wave's hits found no room

template <int TILE, int LM, int NS, int TB, int NE>
__device__ __forceinline__ void raster_tile(const RasterJob& J, RasterShared<TILE, NE, TB / 64>& S,
                                            unsigned long long* key, int L) {
    constexpr bool DEEP = LM > 0;
    constexpr int SL = RASTER_SLOT, KS = KeyRow<TILE, DEEP>::N, NW = TB / 64;
    constexpr int MW = NE * TILE * (TILE / SL) / 64;     // words of begin[]
    constexpr int GATHER = NE / 64 < 3 ? NE / 64 : 3;    // a wave's hits of one look fit an empty list
    constexpr int PK_KEY = PackBits<TILE>::KEY, PK_SLOT = PackBits<TILE>::SLOT, PK_DROP = PackBits<TILE>::DROP;
    static_assert(SL == 4 && (1 << PK_DROP) <= SL && !(DEEP && PK_DROP), "PTri::pk box width");
    static_assert(NS * TILE * KS <= (1 << (PK_SLOT - PK_KEY)), "PTri::pk key index");
    static_assert(64 * MW <= (1 << (32 - PK_SLOT)), "PTri::pk first slot");
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const unsigned cap = (unsigned)J.cap;
    unsigned cnt[NS], nb[NS];                            // entries of each sign; those read from its bin
    bool over = false;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        cnt[s] = gload(&J.counts[s * J.tstride]);
        nb[s] = cnt[s];
        if (cnt[s] > cap) {
            over = true;
            nb[s] = gload(&J.spn[2 * s]) > SPILL_CAP ? 0u : cap;
            if (tid == 0) {
                atomicAdd(&J.stats[ST_OVERFLOWS], 1ull);
                if (nb[s] == 0u) atomicAdd(&J.stats[ST_FULL_SCANS], 1ull);
            }
        }
    }
    if (tid == 0) {
        const unsigned mx = NS == 2 ? max(cnt[0], cnt[NS - 1]) : cnt[0];
        // the value only grows, so a workgroup that reads one at least as
        // large (possibly stale) may skip the atomic: almost all do
        if ((unsigned long long)mx > J.stats[ST_MAX_BIN]) atomicMax(&J.stats[ST_MAX_BIN], (unsigned long long)mx);
        S.nhit = 0u;
    }
    const unsigned total = nb[0] + (NS == 2 ? nb[NS - 1] : 0u);
    unsigned pos = 0u;                                   // bin entries done (both signs end to end)
    int gs = -1;                                         // sign whose overflow is gathered (-1: bins)
    unsigned gpos = 0u, glimit = 0u;                     // this wave's place in it
    for (;;) {
        // ---- this thread's triangle of the batch
        bool has = false;
        unsigned t = 0u;
        int s = 0;
        if (gs < 0 && pos >= total) {
            if (!over) break;
            gs = 0;
            gpos = glimit = 0u;
            if (cnt[0] > cap) {
                glimit = nb[0] == 0u ? (unsigned)J.n_tris : gload(&J.spn[0]);
                gpos = 64u * GATHER * (unsigned)wave;
            }
        }
        if (gs < 0) {
            const unsigned e = pos + (unsigned)tid;
            has = tid < NE && e < total;
            if (has) {
                s = (NS == 2 && e >= nb[0]) ? 1 : 0;
                const unsigned k = s ? e - nb[0] : e;
                t = gload(&J.bins[s * J.tstride * (long long)cap + k]);
            }
            pos += NE;
        } else {
            __syncthreads();
            const bool scan = nb[NS == 2 && gs ? NS - 1 : 0] == 0u;
            const TriR* R = J.rec + (long long)gs * J.n_tris;
            while (gpos < glimit) {
                // GATHER times 64 entries, their reads all in flight together
                bool hit[GATHER];
                unsigned tj[GATHER];
                if (!scan) {
                    unsigned long long e[GATHER];
#pragma unroll
                    for (int i = 0; i < GATHER; ++i)
                        e[i] = gload(&J.spill[(long long)gs * SPILL_CAP + min(gpos + 64u * i + (unsigned)lane, glimit - 1u)]);
#pragma unroll
                    for (int i = 0; i < GATHER; ++i) {
                        hit[i] = gpos + 64u * i + (unsigned)lane < glimit && (unsigned)(e[i] >> 32) == (unsigned)J.tile;
                        tj[i] = (unsigned)e[i];
                    }
                } else {
                    struct __align__(16) Corners { int X[3], Y[3]; unsigned flags, pad; };      // (TriR's first 32 B)
                    Corners q[GATHER];
#pragma unroll
                    for (int i = 0; i < GATHER; ++i) {
                        tj[i] = min(gpos + 64u * i + (unsigned)lane, glimit - 1u);
                        q[i] = gload((const Corners*)&R[tj[i]]);
                    }
#pragma unroll
                    for (int i = 0; i < GATHER; ++i) {
                        TriR b;
#pragma unroll
                        for (int k = 0; k < 3; ++k) { b.X[k] = q[i].X[k]; b.Y[k] = q[i].Y[k]; }
                        int x0, x1, y0, y1;
                        tri_box(b, J.px0, J.py0, J.cx1, J.cy1, x0, x1, y0, y1);
                        hit[i] = gpos + 64u * i + (unsigned)lane < glimit && (q[i].flags & TRI_VALID) && x0 <= x1 && y0 <= y1;
                    }
                }
                unsigned n = 0u, place[GATHER];          // all of the wave's hits, in order
#pragma unroll
                for (int i = 0; i < GATHER; ++i) {
                    const unsigned long long m = __ballot(hit[i]);
                    place[i] = n + lanes_below(m);
                    n += (unsigned)__popcll(m);
                }
                if (n > 0u) {
                    // room for all of them, or this wave waits for the next batch
                    // (a scan's other waves too, from their next look on)
                    unsigned at = 0xFFFFFFFFu;
                    if (lane == 0) {
                        unsigned old = S.nhit;
                        while (old + n <= (unsigned)NE) {
                            const unsigned seen = atomicCAS(&S.nhit, old, old + n);
                            if (seen == old) {
                                at = old;
                                break;
                            }
                            old = seen;
                        }
                        if (NW > 1 && scan && at == 0xFFFFFFFFu) atomicOr(&S.nhit, HITS_FULL);
                    }
                    at = (unsigned)__builtin_amdgcn_readfirstlane((int)at);
                    if (at == 0xFFFFFFFFu) break;
#pragma unroll
                    for (int i = 0; i < GATHER; ++i)
                        if (hit[i]) S.hit[at + place[i]] = tj[i] | ((unsigned)gs << 31);
                }
                gpos += 64u * GATHER * NW;
                if (NW > 1 && (__hip_atomic_load(&S.nhit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) & HITS_FULL))
                    break;
            }
            __syncthreads();
            const unsigned nh = S.nhit & ~HITS_FULL;
            if (nh == 0u) {                              // this sign's are all done
                if (++gs == NS) break;
                gpos = glimit = 0u;
                if (NS == 2 && cnt[NS - 1] > cap) {
                    glimit = nb[NS - 1] == 0u ? (unsigned)J.n_tris : gload(&J.spn[2]);
                    gpos = 64u * GATHER * (unsigned)wave;
                }
                continue;
            }
            has = (unsigned)tid < nh;
            if (has) {
                t = S.hit[tid] & 0x7FFFFFFFu;
                s = (int)(S.hit[tid] >> 31);
            }
        }
        // ---- stage it
        TriR r{};
        int x0 = 0, y0 = 0, bw = 1, bh = 0;
        bool large = false;
        if (has) {
            r = gload(&J.rec[(long long)s * J.n_tris + t]);
            int x1, y1;
            tri_box(r, J.px0, J.py0, J.cx1, J.cy1, x0, x1, y0, y1);
            if (x0 <= x1 && y0 <= y1) {
                large = !(r.flags & TRI_SMALL);
                bw = x1 - x0 + 1;
                bh = large ? 0 : y1 - y0 + 1;
            }
        }
        const int c = ((bw + SL - 1) / SL) * bh;         // slots
        const unsigned mine = ((unsigned)c << 9) | (c > 0 ? 1u : 0u);
        const unsigned incl = (unsigned)wave_inclusive_sum((int)mine);
        if (lane == 63) S.wtot[wave] = incl;
        for (int j = tid; j < MW; j += TB) S.begin[j] = 0ull;
        if (tid == 0) S.nbig = 0u;                       // (read by all before the last barrier)
        __syncthreads();
        unsigned before = 0u, all = 0u;
#pragma unroll
        for (int w = 0; w < (NE + 63) / 64; ++w) {
            const unsigned v = S.wtot[w];
            all += v;
            if (w < wave) before += v;
        }
        const int N = (int)(all >> 9);
        if (c > 0) {
            const unsigned ex = before + incl - mine;
            const unsigned pex = ex >> 9;
            PTri q;
            const int cx = 256 * x0 + 128, cy = 256 * y0 + 128;
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const int ia = (k + 1) % 3, ib = (k + 2) % 3;
                const int dX = r.X[ib] - r.X[ia], dY = r.Y[ib] - r.Y[ia];
                q.d[k] = (dX & 0xFFFF) | (dY << 16);
                q.c[k] = (__mul24(dX, cy - r.Y[ia]) - __mul24(dY, cx - r.X[ia])) + (int)((r.flags >> (k + 1)) & 1u);
            }
            q.dz = ((cx - r.X[0]) & 0xFFFF) | ((cy - r.Y[0]) << 16);
            q.z0 = r.z0; q.zx = r.zx; q.zy = r.zy;
            q.t = t;
            q.pk = ((unsigned)(bw - 1) >> PK_DROP) | ((unsigned)((s * TILE + y0 - J.py0) * KS + (x0 - J.px0)) << PK_KEY) |
                   (pex << PK_SLOT);
            S.tri[ex & 511u] = q;
            atomicOr(reinterpret_cast<unsigned*>(S.begin) + (pex >> 5), 1u << (pex & 31u));
        }
        const unsigned long long lm = __ballot(large);
        if (lm) {
            unsigned at = 0u;
            if (lane == 0) at = atomicAdd(&S.nbig, (unsigned)__popcll(lm));
            at = (unsigned)__builtin_amdgcn_readfirstlane((int)at);
            if (large) S.tri[NE - 1 - (int)(at + lanes_below(lm))].t = t | ((unsigned)s << 31);
        }
        if (tid == 0) S.nhit = 0u;
        __syncthreads();
        // ---- its slots, an even share of the passes per wave
        const int nwin = (N + 63) >> 6;
        const int w0 = wave * nwin / NW, w1 = (wave + 1) * nwin / NW;
        int base = 0;                                    // triangles begun before window w0
        if (w0 > 0 && w0 < w1) {
            for (int j = lane; j < w0; j += 64) base += __popcll(S.begin[j]);
            base = __builtin_amdgcn_readlane(wave_inclusive_sum(base), 63);
        }
        for (int w = w0; w < w1; ++w) {
            const unsigned long long Mv = S.begin[w];    // (the same for all lanes)
            const unsigned mlo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)Mv);
            const unsigned mhi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(Mv >> 32));
            const unsigned long long M = ((unsigned long long)mhi << 32) | mlo;
            // begun at or before the lane's slot, less one
            const int rr = base + (int)(mlo & 1u) - 1 + (int)lanes_below(M >> 1);
            base += __popcll(M);
            const int sl = 64 * w + lane;
            if (sl < N) {
                const PTri q = S.tri[rr];
                const int idx = sl - (int)(q.pk >> PK_SLOT);
                const unsigned w4 = (q.pk << PK_DROP) & 0x1Cu;       // 4 (slots per row - 1)
                int dy;                                  // idx / slots per row
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
                const int off = (int)((q.pk >> PK_KEY) & ((1u << (PK_SLOT - PK_KEY)) - 1u)) + dy * KS + dx;
#pragma unroll
                for (int k = 0; k < SL; ++k) {
                    const bool in = !DEEP || k == 0 || dx + k <= (int)(q.pk & 31u);
                    if (in && min(e[0], min(e[1], e[2])) > 0) {
                        float z = (q.z0 + q.zx * xf) + zrow;
                        z = fmaxf(z, 0.0f);              // 0 for negative values and NaN
                        insert_key<LM>(key, off + k, ((unsigned long long)__float_as_uint(z) << 32) | q.t, L);
                    }
                    e[0] -= a[0];
                    e[1] -= a[1];
                    e[2] -= a[2];
                    xf += 256.0f;                        // (exact)
                }
            }
        }
        // ---- its large triangles, 64 pixels of a box per wave and pass
        const unsigned nbig = S.nbig;
        for (unsigned i = 0; i < nbig; ++i) {
            const unsigned ts = (unsigned)__builtin_amdgcn_readfirstlane((int)S.tri[NE - 1 - (int)i].t);
            const unsigned tt = ts & 0x7FFFFFFFu;
            const int sb = (int)(ts >> 31);
            const TriR b = gload(&J.rec[(long long)sb * J.n_tris + tt]);
            int bx0, bx1, by0, by1;
            tri_box(b, J.px0, J.py0, J.cx1, J.cy1, bx0, bx1, by0, by1);
            const int w = bx1 - bx0 + 1, n = w * (by1 - by0 + 1);
            const unsigned m = ((1u << 20) + (unsigned)w - 1u) / (unsigned)w;     // exact for w <= 32, idx < 1024
            for (int idx = tid; idx < n; idx += TB) {
                const int dy = (int)(((unsigned)idx * m) >> 20);
                const int x = bx0 + idx - dy * w, y = by0 + dy;
                const int px = 256 * x + 128, py = 256 * y + 128;
                long long e0, e1, e2;
                if (!inside(b, px, py, e0, e1, e2)) continue;
                const float z = depth_at(b, px, py);
                insert_key<LM>(key, (sb * TILE + y - J.py0) * KS + (x - J.px0),
                                 ((unsigned long long)__float_as_uint(z) << 32) | tt, L);
            }
        }
        __syncthreads();
    }
    // leave the bins empty for the next use; the last overflowing tile of a
    // render empties the render's spill list
    if (tid == 0) {
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            J.counts[s * J.tstride] = 0u;
            if (cnt[s] > cap && atomicSub(&J.spn[2 * s + 1], 1u) == 1u) J.spn[2 * s] = 0u;
        }
    }
}

// ------------------------------------------------ tile-local aggregation --
//
// Contributions are summed per group inside the workgroup before they reach
// the global accumulators (int64 sum + uint32 count), which get one atomic
// pair per distinct group of the tile.  Integer sums make the result identical
// to per-pixel global atomics.
//
// Texels of class 0 go to a box: an array over the bounding rectangle of the
// tile's footprints, one LDS add per texel and no key to look up, whose rows
// leave as runs of neighbouring groups (an atomic is a 32-byte transaction
// that the lanes of one sector share).  Vertices, and the texels of a tile
// whose rectangle is too large (a seam of the UV map, a minified texture,
// unrelated triangles) or of other classes, go to an open-addressing table
// keyed by group.  Both are in one zeroed region; which part of it is table is
// settled once the rectangle is known.
// Bound by the latency of the table's dependent LDS operations, by same-address
// conflicts and by the memory's rate of atomics (1024 px GGX, 32 items: 1330 us
// a step, 1142 without the flush's atomics, before groups were hashed in runs).

#define HASH_NONE 0xFFFFFFFFu    // no group
// Slots looked at for a group before its sum goes straight to memory.  Tiles at
// a texture's pole or seam hold nearly as many texels as slots; with 64 slots
// looked at their adds ran along the full table, 27 us of a 47 us launch of
// one 512 px item.  Whole steps with 64 / 6 / 4 / 3 / 2 slots: 512 px, 128
// single-item launches 4886 / 3270 / 3256 / 3256 / 3225 us, four layers
// 270 / 246 / 245 / 245 / 249, 10240-triangle soup (nearest texels, about 500
// groups a tile) 1399 / 1388 / 1387 / 1452 / 1971, 1024 px GGX
// 1337 / 1326 / 1323 / 1320 / 1319.
#define HASH_PROBES 5
// Neighbouring groups in neighbouring slots leave in one flush instruction, 8
// sums to a 64-byte line: the memory's atomics are what the flush waits for.
// Whole steps with runs of 1 / 2 / 4 / 8 / 16 / 32 groups: 512 px, two layers
// 1072 / 814 / 715 / 688 / 688 / 725 us, 1024 px GGX 1293 / 1264 / 1245 / 1234 /
// 1229 / 1231, subdivision 1438 / 1384 / 1357 / 1342 / 1337 / 1339, 10240-triangle
// soup 1315 / 1294 / 1289 / 1286 / 1284 / 1308, launches of one 512 px item
// 3101 / 3086 / 3051 / 3042 / 3074 / 3107.
#define HASH_RUN 3

// A slot packs the group's sum and count into one 64-bit word,
// sum * 2^12 + count, so one LDS atomic adds both: a tile has at most 1024
// pixels, so the count stays below 2^12 (a subdivision surface's control
// vertex is counted once per pixel too), and |sum| <= 1024 * 2^37 keeps the
// packed word within int64.
#define PACK_SHIFT 12
#define PACK_MASK ((1ull << PACK_SHIFT) - 1ull)

template <typename C>
struct GroupMem {
    static constexpr int BYTES_T = 12 << C::LOG2T, BYTES_B = (12 << C::LOG2B) + 8 * C::BOX;
    static constexpr int WORDS = (BYTES_T > BYTES_B ? BYTES_T : BYTES_B) / 16;
    uint4 w[WORDS];
    unsigned lo[C::NW], hi[C::NW];       // each wave's footprint corners, least and largest (x low, y high half)
    unsigned n_list;                     // occupied slots (flush)
};

// Modes that do not scatter, where the table's room would cost them blocks: at
// 32 pixels (8- and 16-pixel tiles have 7 and 8 waves per SIMD with it; full-image
// calls are 0 to 2 % slower without).
struct NoGroups {};

// The region as the tile uses it: 2^logt slots of sums and of keys (group + 1;
// 0: empty), then the box (bw = 0: none).
struct GroupTable {
    unsigned long long* sum;
    unsigned* key;
    int logt;
    unsigned long long* box;
    int bx, by, bw, bh;
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

__device__ __forceinline__ void table_add(const GroupTable& tb, long long* __restrict__ Rp,
                                          unsigned* __restrict__ K, unsigned g, long long q, unsigned c) {
    const unsigned mask = (1u << tb.logt) - 1u;
    // Aligned runs of 2^HASH_RUN groups are hashed, a run's groups take
    // neighbouring slots.  Multiplicative hash in 24-bit multiplies (full rate;
    // the 32-bit one is quarter rate), the high byte folded in first.
    const unsigned run = g >> HASH_RUN;
    unsigned h = (((__umul24(run ^ (run >> 24), 0x9E3779u) >> (24 + HASH_RUN - tb.logt)) << HASH_RUN) |
                  (g & ((1u << HASH_RUN) - 1u))) & mask;
    for (int probe = 0; probe < HASH_PROBES; ++probe) {
        unsigned k = __hip_atomic_load(&tb.key[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (k == 0u) k = atomicCAS(&tb.key[h], 0u, g + 1u);
        if (k == 0u || k == g + 1u) {
            atomicAdd(&tb.sum[h], pack_sc(q, c));
            return;
        }
        h = (h + (1u << HASH_RUN)) & mask;
    }
    global_add(Rp, K, g, q, c);      // crowded table: go straight to memory
}

// Adds (q, 1) to N groups (HASH_NONE: none), one after another: requesting
// all their slots at once was 2 to 5 % slower (more of them are then found
// empty and compare-and-swap on the same words).
template <int N>
__device__ __forceinline__ void table_add_all(const GroupTable& tb, long long* __restrict__ Rp,
                                              unsigned* __restrict__ K, const unsigned (&g)[N], long long q) {
#pragma unroll
    for (int i = 0; i < N; ++i)
        if (g[i] != HASH_NONE) table_add(tb, Rp, K, g[i], q, 1u);
}

// Subdivision surface: a pixel credits the control vertices of both its sides'
// tessellated triangles, about 15 each and mostly the same ones.  The tile
// first sums its pixels by their pair of triangles (DRD_BG: none), in a table
// with a slot per pixel (so every pair finds one) that takes the keys' place,
// and then adds each distinct pair's sum to the union of its two lists once,
// 16 lanes to a pair (before: a butterfly sum per distinct triangle of a wave,
// and a merge of the two lists per pixel where they differed).  Vertices before
// texels: in a crowded table the texels' many groups would take the slots of the
// few that every pixel adds to (the other order: 1487 -> 2306 us).
struct PairSlot {
    unsigned long long key;              // + triangle + 1 (high half), - triangle + 1; 0: empty
    unsigned long long sum;              // packed sum and count
};

// Every lane of a wave calls; list: the slots in use, *n_list of them.
template <int N>
__device__ __forceinline__ void pair_add(PairSlot* slots, unsigned short* list, unsigned* n_list, bool act,
                                         unsigned tp, unsigned tm, long long q) {
    const unsigned long long k = ((unsigned long long)(tp + 1u) << 32) | (tm + 1u);
    unsigned h = ((tp * 0x9E3779B1u) ^ (tm * 0x85EBCA6Bu)) >> 16;
    bool fresh = false;
    if (act) {
        for (int probe = 0; probe < N; ++probe, ++h) {
            PairSlot& p = slots[h & (N - 1)];
            unsigned long long seen = __hip_atomic_load(&p.key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            if (seen == 0ull) {
                seen = atomicCAS(&p.key, 0ull, k);
                fresh = seen == 0ull;
            }
            if (fresh || seen == k) {
                atomicAdd(&p.sum, pack_sc(q, 1u));
                break;
            }
        }
    }
    const unsigned long long m = __ballot(fresh);
    unsigned base = 0;
    if ((threadIdx.x & 63) == 0 && m) base = atomicAdd(n_list, (unsigned)__popcll(m));
    base = (unsigned)__builtin_amdgcn_readfirstlane((int)base);
    if (fresh) list[base + lanes_below(m)] = (unsigned short)(h & (N - 1));
}

// Whether x is among the 16-lane row's values of y (each lane compares with the
// row's sixteen, turned past it by DPP moves; every lane calls).
__device__ __forceinline__ bool in_row(int x, int y) {
    bool hit = x == y;
#define DRD_TURN(n) hit = hit | (x == __builtin_amdgcn_update_dpp(0, y, 0x120 + n, 0xf, 0xf, false));
    DRD_TURN(1) DRD_TURN(2) DRD_TURN(3) DRD_TURN(4) DRD_TURN(5) DRD_TURN(6) DRD_TURN(7) DRD_TURN(8)
    DRD_TURN(9) DRD_TURN(10) DRD_TURN(11) DRD_TURN(12) DRD_TURN(13) DRD_TURN(14) DRD_TURN(15)
#undef DRD_TURN
    return hit;
}

// Adds the distinct pairs' sums to their control vertices, a row of 16 lanes
// to a pair.  Both lists hold each control vertex once; an entry of the - side's
// that the + side holds too is left to the + side.
// Bound by the latency of the list reads.  Measured at 1024 px, 48000
// tessellated triangles, GGX, 32 items (whole step): 1920 -> 1499 us.
template <int TB>
__device__ __forceinline__ void pair_expand(const PairSlot* slots, const unsigned short* list, int n,
                                            const GroupTable& tb, long long* __restrict__ Rp,
                                            unsigned* __restrict__ K, const DScene& sc, int tid) {
    const int l = tid & 15;
    for (int i0 = 0; i0 < n; i0 += TB / 16) {
        const int i = i0 + (tid >> 4);
        int a0 = 0, a1 = 0, b0 = 0, b1 = 0;
        long long q = 0;
        unsigned c = 0u;
        if (i < n) {
            const PairSlot p = slots[list[i]];
            unpack_sc(p.sum, q, c);
            const unsigned tp = (unsigned)(p.key >> 32), tm = (unsigned)p.key;       // plus 1
            if (tp != 0u) { a0 = gload(&sc.tri_rowptr[tp - 1u]); a1 = gload(&sc.tri_rowptr[tp]); }
            if (tm != 0u && tm != tp) { b0 = gload(&sc.tri_rowptr[tm - 1u]); b1 = gload(&sc.tri_rowptr[tm]); }
        }
        // 16 entries of either list at a time; the first of both, as a rule all
        // there are, read together
        int ga = a0 + l < a1 ? gload(&sc.tri_cols[a0 + l]) : -1;
        for (int j0 = 0; __ballot(b0 + j0 < b1); j0 += 16) {
            const int g = b0 + j0 + l < b1 ? gload(&sc.tri_cols[b0 + j0 + l]) : -2;
            bool dup = in_row(g, ga);
            for (int k0 = 16; __ballot(a0 + k0 < a1); k0 += 16)
                dup |= in_row(g, a0 + k0 + l < a1 ? gload(&sc.tri_cols[a0 + k0 + l]) : -1);
            if (g >= 0 && !dup) table_add(tb, Rp, K, (unsigned)g, q, c);
        }
        for (int k0 = 0; __ballot(a0 + k0 < a1); k0 += 16) {
            if (k0 > 0) ga = a0 + k0 + l < a1 ? gload(&sc.tri_cols[a0 + k0 + l]) : -1;
            if (ga >= 0) table_add(tb, Rp, K, (unsigned)ga, q, c);
        }
    }
}

struct Tri3 { unsigned v[3]; };

// Whether the launch fills the chip (256 CUs of 2048 threads).  If so, what
// costs fewer operations wins; if not, the shorter chain of dependent ones.
// A mesh's vertices go by pairs of triangles in full launches: few adds, and few
// lanes on one vertex's slot, against two barriers and the list's chain of reads.
// Whole steps per pixel / by pairs: 1024 px GGX, 131072 tiles, 1320 / 1301 us;
// 10240-triangle soup, 131072 tiles, 1384 / 1323; 12 uneven scenes 1176 / 1149;
// launches of 1024 tiles 3082 / 3206.
template <int TB>
__device__ __forceinline__ bool full_launch() {
    return (long long)gridDim.x * gridDim.y > 256 * 2048 / TB;
}

// pair_expand for a mesh's own vertices, six lanes to a pair.
template <int TB>
__device__ __forceinline__ void pair_verts(const PairSlot* slots, const unsigned short* list, int n,
                                           const GroupTable& tb, long long* __restrict__ Rp,
                                           unsigned* __restrict__ K, const DScene& sc, int tid) {
    for (int i = tid; i < 6 * n; i += TB) {
        const int j = (int)(((unsigned)i * 10923u) >> 16), l = i - 6 * j;      // i / 6 (exact: i < 6144)
        const PairSlot p = slots[list[j]];
        const unsigned tp = (unsigned)(p.key >> 32), tm = (unsigned)p.key;       // plus 1
        const unsigned t = l < 3 ? tp : tm;
        if (t == 0u || (l >= 3 && tm == tp)) continue;
        const unsigned g = gload(&sc.tri[3 * (long long)(t - 1u) + (l < 3 ? l : l - 3)]);
        if (l >= 3 && tp != 0u) {
            const Tri3 a = gload((const Tri3*)(sc.tri + 3 * (long long)(tp - 1u)));
            if (g == a.v[0] || g == a.v[1] || g == a.v[2]) continue;
        }
        long long q;
        unsigned c;
        unpack_sc(p.sum, q, c);
        table_add(tb, Rp, K, g, q, c);
    }
}

// Tile kernels of 8- and 16-pixel tiles are asked for 8 resident waves per SIMD
// (at most 64 VGPRs and 96 SGPRs) and get them where their LDS allows it, 20 KB
// per 4 waves: 16-pixel estimates, opaque 20.3 KB and deep 18.5, opaque renders of
// both sizes, 8-pixel estimates of two layers.  More LDS leaves 7 waves to opaque
// 8-pixel estimates (22.7 KB) and 16-pixel renders of four layers (20.5), 6 to
// 8-pixel estimates of four (25.1), 5 to renders of two (28.8, of which they use
// the raster's part); the compiler bounds those kernels' registers accordingly.
// Unasked, the deep estimates took 106 SGPRs and 7 waves (512 px, two layers, 32
// items 1124 -> 1087 us, four ragged layers 246 -> 227).  The GGX render spills at
// this bound and is still faster (145.5 us for four 1024 px views; 153.8 with 7
// waves and no spill).  32-pixel tiles are held to 4 to 8 waves by LDS and threads.
#define TILE_MIN_WAVES 8

// Everything the tile body needs, resolved by the kernel's prologue.
struct TileJob {
    const DScene* sc;
    const DView* vw;
    const float* theta;
    const uint8_t* sg;                   // group sign bytes of the pair (null: unperturbed)
    const float* eps;                    // per block
    unsigned flip;                       // one-sign modes: sign 0 is the minus render (all ones) or the plus one
    RasterJob ras;                       // (its tile's pixels are set by the body)
    const TriS* recS;                    // [NS, n_tris]
    const TriG* recG;
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

// The two sides' values of a pixel, known to both of its lanes: x of the
// lane below 32 (+) and of the lane above (-).
__device__ __forceinline__ void both_sides(unsigned x, unsigned& p, unsigned& m) {
    auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    p = r[0];
    m = r[1];
}

__device__ __forceinline__ void both_sides(float x, float& p, float& m) {
    unsigned a, b;
    both_sides(__float_as_uint(x), a, b);
    p = __uint_as_float(a);
    m = __uint_as_float(b);
}

// Texels of a footprint, as bits 2 row + column: those that repeat an earlier
// one of it, and those that another footprint holds too.
__device__ __forceinline__ unsigned foot_repeats(const FootBox& f) {
    const unsigned d = f.a ^ f.b;
    return ((d & 0xFFFFu) == 0u ? 0xAu : 0u) | ((d >> 16) == 0u ? 0xCu : 0u);
}

__device__ __forceinline__ unsigned foot_shared(const FootBox& f, const FootBox& o) {
    const unsigned xa = f.a & 0xFFFFu, xb = f.b & 0xFFFFu, ya = f.a >> 16, yb = f.b >> 16;
    const unsigned oxa = o.a & 0xFFFFu, oxb = o.b & 0xFFFFu, oya = o.a >> 16, oyb = o.b >> 16;
    const unsigned cols = ((xa == oxa || xa == oxb) ? 1u : 0u) | ((xb == oxa || xb == oxb) ? 2u : 0u);
    return ((ya == oya || ya == oyb) ? cols : 0u) | ((yb == oya || yb == oyb) ? cols << 2 : 0u);
}

// Adds (q, 1) to the footprint's texels of class c that are not in `skip`: in
// the box when `boxed`, else in the table.
__device__ __forceinline__ void foot_add(const GroupTable& tb, bool boxed, long long* __restrict__ Rp,
                                         unsigned* __restrict__ K, const DScene& sc, int c, const FootBox& f,
                                         unsigned skip, long long q) {
    const unsigned xa = f.a & 0xFFFFu, xb = f.b & 0xFFFFu, ya = f.a >> 16, yb = f.b >> 16;
    if (boxed) {
        const unsigned long long w = pack_sc(q, 1u);
        const int i0 = __mul24((int)ya - tb.by, tb.bw) + (int)xa - tb.bx, dx = (int)xb - (int)xa,
                  dy = __mul24((int)yb - (int)ya, tb.bw);
        if (!(skip & 1u)) atomicAdd(&tb.box[i0], w);
        if (!(skip & 2u)) atomicAdd(&tb.box[i0 + dx], w);
        if (!(skip & 4u)) atomicAdd(&tb.box[i0 + dy], w);
        if (!(skip & 8u)) atomicAdd(&tb.box[i0 + dy + dx], w);
    } else {
        const unsigned base = (unsigned)sc.cls_goff[c], W = (unsigned)sc.cls_w[c];
        const unsigned ra = base + __umul24(ya, W), rb = base + __umul24(yb, W);
        const unsigned g[4] = {(skip & 1u) ? HASH_NONE : ra + xa, (skip & 2u) ? HASH_NONE : ra + xb,
                               (skip & 4u) ? HASH_NONE : rb + xa, (skip & 8u) ? HASH_NONE : rb + xb};
        table_add_all(tb, Rp, K, g, q);
    }
}

typedef unsigned short drd_us2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ unsigned pk_min(unsigned a, unsigned b) {
    return __builtin_bit_cast(unsigned, __builtin_elementwise_min(__builtin_bit_cast(drd_us2, a), __builtin_bit_cast(drd_us2, b)));
}

__device__ __forceinline__ unsigned pk_max(unsigned a, unsigned b) {
    return __builtin_bit_cast(unsigned, __builtin_elementwise_max(__builtin_bit_cast(drd_us2, a), __builtin_bit_cast(drd_us2, b)));
}

// Least and largest halves over the wave (every lane calls; result in lane 63).
__device__ __forceinline__ void wave_corners(unsigned& lo, unsigned& hi) {
#define DRD_STEP(ctrl, rows)                                                                                     \
    lo = pk_min(lo, (unsigned)__builtin_amdgcn_update_dpp(-1, (int)lo, ctrl, rows, 0xf, false));                 \
    hi = pk_max(hi, (unsigned)__builtin_amdgcn_update_dpp(0, (int)hi, ctrl, rows, 0xf, false));
    DRD_STEP(0x111, 0xf)
    DRD_STEP(0x112, 0xf)
    DRD_STEP(0x114, 0xf)
    DRD_STEP(0x118, 0xf)
    DRD_STEP(0x142, 0xa)
    DRD_STEP(0x143, 0xc)
#undef DRD_STEP
}

// Whether a tile's class-0 texels may go to a box: only bilinear footprints,
// four texels a side; the nearest-texel mode's single one costs the table less
// than the rectangle (10240-triangle soup 1291 us, with boxes 1313).  Opaque
// tiles only: whole steps without / with boxes, 1024 px GGX 1259 / 1232 us,
// subdivision 1374 / 1340, 12 uneven scenes 1128 / 1114, two layers 676 / 687, four
// 214 / 217.  (Launches of one 512 px item: 2981 / 3032 without the code, but a
// choice by the launch's size there cost 3052, and the others 1 %.)
__device__ __forceinline__ bool boxable(const TileJob& J) {
    return J.sc->n_cls > 0 && J.act_cls[0] && J.sc->tex_mode == 0;
}

template <typename C>
__device__ __forceinline__ void groups_clear(GroupMem<C>& M, int tid) {
    for (int j = tid; j < GroupMem<C>::WORDS; j += C::TB) M.w[j] = make_uint4(0u, 0u, 0u, 0u);
    if (tid == 0) M.n_list = 0u;
}

// Lays the cleared region out.  lo, hi: this thread's least and largest
// footprint corners of class 0 (all ones and 0: none); boxed: class 0 is
// scattered at all.  Called by every thread; passes the barrier after which
// the region is clear.
template <typename C>
__device__ __forceinline__ GroupTable groups_open(GroupMem<C>& M, bool boxed, unsigned lo, unsigned hi, int tid) {
    GroupTable tb;
    tb.bw = tb.bh = tb.bx = tb.by = 0;
    boxed = boxed && C::BOX > 0;
    if (boxed) {                                 // (uniform)
        wave_corners(lo, hi);
        if ((tid & 63) == 63) {
            M.lo[tid >> 6] = lo;
            M.hi[tid >> 6] = hi;
        }
    }
    __syncthreads();
    if (boxed) {
        lo = 0xFFFFFFFFu;
        hi = 0u;
#pragma unroll
        for (int w = 0; w < C::NW; ++w) {
            lo = pk_min(lo, M.lo[w]);
            hi = pk_max(hi, M.hi[w]);
        }
        lo = (unsigned)__builtin_amdgcn_readfirstlane((int)lo);
        hi = (unsigned)__builtin_amdgcn_readfirstlane((int)hi);
        const int bw = (int)(hi & 0xFFFFu) - (int)(lo & 0xFFFFu) + 1, bh = (int)(hi >> 16) - (int)(lo >> 16) + 1;
        if (bw > 0 && bh > 0 && bw <= C::BOX && bh <= C::BOX && bw * bh <= C::BOX) {
            tb.bx = (int)(lo & 0xFFFFu);
            tb.by = (int)(lo >> 16);
            tb.bw = bw;
            tb.bh = bh;
        }
    }
    tb.logt = tb.bw > 0 ? C::LOG2B : C::LOG2T;
    tb.sum = reinterpret_cast<unsigned long long*>(M.w);
    tb.key = reinterpret_cast<unsigned*>(tb.sum + (1 << tb.logt));
    tb.box = reinterpret_cast<unsigned long long*>(tb.key + (1 << tb.logt));
    return tb;
}

// The tile's groups to the global accumulators: the table's occupied slots,
// gathered into a dense list first so the atomics go out in full waves (list:
// LDS for 2^LOG2T slot numbers), and the box's rows.
template <typename C>
__device__ __forceinline__ void groups_flush(const GroupTable& tb, unsigned short* list, unsigned* n_list, long long* Rp,
                                             unsigned* K, const DScene& sc, int tid) {
    const int lane = tid & 63;
    for (int j = tid; j < (1 << tb.logt); j += C::TB) {
        const bool occ = tb.key[j] != 0u;
        const unsigned long long m = __ballot(occ);
        unsigned base = 0;
        if (lane == 0 && m) base = atomicAdd(n_list, (unsigned)__popcll(m));
        base = (unsigned)__builtin_amdgcn_readfirstlane((int)base);
        if (occ) list[base + lanes_below(m)] = (unsigned short)j;
    }
    const int area = tb.bw * tb.bh;
    if (area > 0) {
        const float inv = 1.0f / (float)tb.bw;
        for (int j = tid; j < area; j += C::TB) {
            long long q;
            unsigned c;
            unpack_sc(tb.box[j], q, c);
            if (c == 0u) continue;
            const int y = (int)(((float)j + 0.5f) * inv);       // j / bw (exact: j < 2048)
            global_add(Rp, K, sc.cls_goff[0] + (long long)(tb.by + y) * sc.cls_w[0] + tb.bx + (j - y * tb.bw), q, c);
        }
    }
    __syncthreads();
    const unsigned n = *n_list;
    for (unsigned i = (unsigned)tid; i < n; i += C::TB) {
        const unsigned j = list[i];
        long long q;
        unsigned c;
        unpack_sc(tb.sum[j], q, c);
        global_add(Rp, K, (long long)tb.key[j] - 1, q, c);
    }
}

// Sums over the block in a fixed tree order (double: loss) or any order
// (int64: full-image totals).
template <int TB, typename T>
__device__ __forceinline__ T block_sum(T* red, T v, int tid) {
    red[tid] = v;
    __syncthreads();
    for (int w = TB / 2; w > 0; w >>= 1) {
        if (tid < w) red[tid] = red[tid] + red[tid + w];
        __syncthreads();
    }
    return red[0];
}

// A pixel's target colour (image form: the loss gradient at it).
__device__ __forceinline__ void pixel_target(const TileJob& J, long long pix, float* t) {
    struct Rgb { float c[3]; };
    const Rgb v = gload((const Rgb*)(J.targets + 3 * pix));
#pragma unroll
    for (int c = 0; c < 3; ++c) t[c] = v.c[c];
}

// The loss difference's fixed-point code of a pixel from its two sides'
// colours; `note`: this lane reports its saturation.
__device__ __forceinline__ long long pixel_code(const TileJob& J, const float* P, const float* M, const float* target,
                                                bool note) {
    int flag;
    const long long q = quantize(pixel_delta(P, M, target, J.img), flag);
    if (flag && note) atomicAdd(&J.ras.stats[flag == 1 ? ST_SATURATIONS : ST_NONFINITE], 1ull);
    return q;
}

// MODE: 0 estimate (both signs, scatter), 1 render (write rgb/id/uv),
// 2 loss (per-tile sum of the per-pixel L2 error f_{w,h}), 3 full-image
// estimate (both signs, per-tile sum of the fixed-point differences); 4 is 3
// with a thread per pixel of a 32-pixel tile.
template <int TILE, int MODE>
struct TileShared {
    using C = TileCfg<TILE, MODE, 0>;
    static constexpr int KS = KeyRow<TILE, false>::N;
    alignas(16) unsigned long long key[C::NS * TILE * KS];
    // the raster's stage, then (estimate) the group table, or the sums
    union {
        RasterShared<TILE, C::NE, C::NW> ras;
        std::conditional_t<MODE == 0 || TILE <= 16, GroupMem<C>, NoGroups> g;
        double red[C::TB];
        long long qred[C::TB];
    } u;
    unsigned n_pairs;                    // distinct pairs of triangles (subdivision surface)
};

template <int TILE, int MODE, int SHADE>
__device__ __forceinline__ void tile_body(TileJob& J, TileShared<TILE, MODE>& S) {
    using C = TileCfg<TILE, MODE, 0>;
    constexpr int TB = C::TB, NS = C::NS, KS = TileShared<TILE, MODE>::KS;
    const int tid = threadIdx.x;
    const DScene& sc = *J.sc;
    const DView& vw = *J.vw;
    RasterJob& R = J.ras;
    const int px0 = R.tile % vw.tiles_x * TILE, py0 = R.tile / vw.tiles_x * TILE;
    R.px0 = px0;
    R.py0 = py0;
    R.cx1 = min(px0 + TILE - 1, vw.W - 1);
    R.cy1 = min(py0 + TILE - 1, vw.H - 1);
    if constexpr (NS == 2) {
        // no triangle of either render touches the tile: every pixel is
        // background in both, so the tile adds nothing (its bins are empty)
        if ((gload(&R.counts[0]) | gload(&R.counts[R.tstride])) == 0u) return;
    }
    for (int j = tid; j < NS * TILE * KS; j += TB) S.key[j] = ~0ull;
    raster_tile<TILE, 0, NS, TB, C::NE>(R, S.u.ras, S.key, 1);
    __syncthreads();                             // (a tile without triangles has only cleared its keys)
    if constexpr (MODE == 0) groups_clear<C>(S.u.g, tid);

    GroupTable tb{};
    double loss_acc = 0.0;
    long long qsum = 0;
    for (int local = tid; local < C::NPIX; local += TB) {
        const int lx = local % TILE, ly = local / TILE;
        const int x = px0 + lx, y = py0 + ly;
        const bool inpix = x < vw.W && y < vw.H;
        const int px = 256 * x + 128, py = 256 * y + 128;
        const long long pix = (long long)y * vw.W + x;
        // the target pixel's read is under way while the pixel is shaded
        float tgt[3] = {0.0f, 0.0f, 0.0f};
        if (MODE != 1 && inpix) pixel_target(J, pix, tgt);
        unsigned id[NS];
        float rgb[NS][3], uv[NS][2];
        FootBox f[NS];
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const unsigned long long k = inpix ? S.key[(s * TILE + ly) * KS + lx] : ~0ull;
            id[s] = (k == ~0ull) ? DRD_BG : (unsigned)k;
            rgb[s][0] = 0.0f; rgb[s][1] = 0.0f; rgb[s][2] = 0.0f;
            uv[s][0] = 0.0f; uv[s][1] = 0.0f;
            f[s] = {0xFFFFFFFFu, 0xFFFFFFFFu};
            if (id[s] != DRD_BG) {
                const TriR* rec = R.rec + (long long)s * sc.n_tris;
                const TriS* recS = J.recS + (long long)s * sc.n_tris;
                const TriG* recG = J.recG + (long long)s * sc.n_tris;
                const TriR r = gload(&rec[id[s]]);
                const TriS sh = gload(&recS[id[s]]);
                const CornerUV cu = load_cuv(sc, id[s]);
                float alpha;
                const unsigned flip = NS == 2 ? (s ? 0xFFFFFFFFu : 0u) : J.flip;
                shade_pixel<SHADE, false>(sc, vw, J.theta, J.sg, J.eps, flip, r, sh, recG + id[s], cu, px, py, rgb[s],
                                          uv[s], f[s], alpha);
            }
        }
        if constexpr (MODE == 2) {
            if (inpix) {
                float dr = rgb[0][0] - tgt[0], dg = rgb[0][1] - tgt[1], db = rgb[0][2] - tgt[2];
                loss_acc += (double)((dr * dr + dg * dg) + db * db);
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
            const bool act = inpix && (id[0] != DRD_BG || id[NS - 1] != DRD_BG) && (MODE >= 3 || J.any_act);
            long long q = 0;
            if (act) q = pixel_code(J, rgb[0], rgb[NS - 1], tgt, true);
            if constexpr (MODE >= 3) {
                qsum += q;
            } else {
                unsigned lo = 0xFFFFFFFFu, hi = 0u;
                if (act) {
#pragma unroll
                    for (int s = 0; s < 2; ++s)
                        if (id[s] != DRD_BG) {
                            lo = pk_min(lo, pk_min(f[s].a, f[s].b));
                            hi = pk_max(hi, pk_max(f[s].a, f[s].b));
                        }
                }
                static_assert(C::NPIX == TB, "the box is known when the pixel is scattered");
                tb = groups_open<C>(S.u.g, boxable(J), lo, hi, tid);
                // the + side's groups, and those of the - side that it does not hold
                if (J.act_pos && (sc.n_ctrl > 0 || full_launch<TB>())) {
                    static_assert(sizeof(S.key) >= C::NPIX * (sizeof(PairSlot) + 2), "pair table and list");
                    PairSlot* slots = reinterpret_cast<PairSlot*>(S.key);
                    unsigned short* pairs = reinterpret_cast<unsigned short*>(slots + C::NPIX);
                    slots[tid] = {0ull, 0ull};
                    if (tid == 0) S.n_pairs = 0u;
                    __syncthreads();
                    pair_add<C::NPIX>(slots, pairs, &S.n_pairs, act, id[0], id[1], q);
                    __syncthreads();
                    const int n = __builtin_amdgcn_readfirstlane((int)S.n_pairs);
                    if (sc.n_ctrl > 0) pair_expand<TB>(slots, pairs, n, tb, J.Rp, J.K, sc, tid);
                    else pair_verts<TB>(slots, pairs, n, tb, J.Rp, J.K, sc, tid);
                } else if (J.act_pos && act) {
                    Tri3 a = {{HASH_NONE, HASH_NONE, HASH_NONE}}, b = a;
                    if (id[0] != DRD_BG) a = gload((const Tri3*)(sc.tri + 3 * (long long)id[0]));
                    if (id[1] != DRD_BG && id[1] != id[0]) b = gload((const Tri3*)(sc.tri + 3 * (long long)id[1]));
                    unsigned g[6];
#pragma unroll
                    for (int i = 0; i < 3; ++i) {
                        g[i] = a.v[i];
                        g[3 + i] = (b.v[i] == a.v[0] || b.v[i] == a.v[1] || b.v[i] == a.v[2]) ? HASH_NONE : b.v[i];
                    }
                    table_add_all(tb, J.Rp, J.K, g, q);
                }
                if (act) {
                    for (int c = 0; c < sc.n_cls; ++c) {
                        if (!J.act_cls[c]) continue;
                        if (c > 0) {
#pragma unroll
                            for (int s = 0; s < 2; ++s)
                                if (id[s] != DRD_BG) f[s] = foot_box(sc, c, uv[s][0], uv[s][1]);
                        }
                        const bool boxed = c == 0 && tb.bw > 0;
                        foot_add(tb, boxed, J.Rp, J.K, sc, c, f[0], id[0] != DRD_BG ? foot_repeats(f[0]) : 0xFu, q);
                        foot_add(tb, boxed, J.Rp, J.K, sc, c, f[1],
                                 id[1] != DRD_BG ? foot_repeats(f[1]) | foot_shared(f[1], f[0]) : 0xFu, q);
                    }
                }
            }
        }
    }
    if constexpr (MODE == 2) {
        loss_acc = block_sum<TB>(S.u.red, loss_acc, tid);
        if (tid == 0) *J.partial = loss_acc;
    }
    if constexpr (MODE >= 3) {
        qsum = block_sum<TB>(S.u.qred, qsum, tid);
        if (tid == 0 && qsum != 0) atomicAdd((unsigned long long*)J.qtot, (unsigned long long)qsum);
    }
    if constexpr (MODE == 0) {
        __syncthreads();
        // the list of occupied slots takes the keys' place
        static_assert(sizeof(S.key) >= (2u << C::LOG2T), "slot list");
        groups_flush<C>(tb, reinterpret_cast<unsigned short*>(S.key), &S.u.g.n_list, J.Rp, J.K, sc, tid);
    }
}

// ------------------------------------------------- semi-transparent tile --
//
// Sec. 4.4 "Transparent geometry": the raster keeps, per pixel and sign,
// the L nearest fragments in front-to-back order (a deep ID buffer in LDS,
// built by the atomic-min cascade of insert_key), the shading pass
// composites them over black, C = sum_l T_l alpha_l c_l with
// T_{l+1} = T_l (1 - alpha_l), and the scatter credits the union over both
// renders and all listed layers of the layers' vertices and footprint
// texels, each group once per pixel.  Tiles are 8 or 16 pixels (a lane per
// pixel and side).

template <int TILE, int MODE, int LM>
struct DeepShared {
    using C = TileCfg<TILE, MODE, LM>;
    unsigned long long key[C::NS * C::NPIX * LM];
    float v[MODE == 0 ? C::NS * C::NPIX * LM : 1];      // the fragments' texture coordinate v
    // the raster's stage, then (estimate) the group table, or the sums
    union {
        RasterShared<TILE, C::NE, C::NW> ras;
        GroupMem<C> g;
        double red[C::TB];
        long long qred[C::TB];
    } u;
};

template <int TILE, int MODE, int LM, int SHADE>
__device__ __forceinline__ void tile_body_deep(TileJob& J, DeepShared<TILE, MODE, LM>& S) {
    using C = TileCfg<TILE, MODE, LM>;
    constexpr int TB = C::TB, NS = C::NS, NPIX = C::NPIX;
    const int tid = threadIdx.x, lane = tid & 63;
    const DScene& sc = *J.sc;
    const DView& vw = *J.vw;
    RasterJob& R = J.ras;
    const int px0 = R.tile % vw.tiles_x * TILE, py0 = R.tile / vw.tiles_x * TILE;
    R.px0 = px0;
    R.py0 = py0;
    R.cx1 = min(px0 + TILE - 1, vw.W - 1);
    R.cy1 = min(py0 + TILE - 1, vw.H - 1);
    if constexpr (NS == 2) {
        // no fragment in either render: the tile adds nothing
        if ((gload(&R.counts[0]) | gload(&R.counts[R.tstride])) == 0u) return;
    }
    for (int j = tid; j < NS * NPIX * LM; j += TB) S.key[j] = ~0ull;
    raster_tile<TILE, LM, NS, TB, C::NE>(R, S.u.ras, S.key, sc.layers);
    __syncthreads();
    const int L = sc.layers;
    if constexpr (MODE == 0) groups_clear<C>(S.u.g, tid);

    const int side = NS == 2 ? lane >> 5 : 0;
    const int local = NS == 2 ? (tid >> 6) * 32 + (lane & 31) : tid;
    const int lx = local % TILE, ly = local / TILE;
    const int x = px0 + lx, y = py0 + ly;
    const bool inpix = x < vw.W && y < vw.H;
    const int px = 256 * x + 128, py = 256 * y + 128;
    const long long pix = (long long)y * vw.W + x;
    float tgt[3] = {0.0f, 0.0f, 0.0f};
    if (MODE != 1 && inpix) pixel_target(J, pix, tgt);
    unsigned long long* mine = &S.key[(side * NPIX + local) * LM];   // this side's fragments
    float* mine_v = &S.v[MODE == 0 ? (side * NPIX + local) * LM : 0];
    // Lists fill from the front, so a list is empty when its first layer is.
    // The loop over layers stays rolled: one copy of the shading.  For the
    // scatter a fragment keeps its id and its texture coordinates (u over the
    // key's depth, v beside).
    float rgb[3] = {0.0f, 0.0f, 0.0f};
    bool any = false;
    float T = 1.0f;
    for (int l = 0; l < L; ++l) {
        const unsigned long long k = inpix ? mine[l] : ~0ull;
        const unsigned id = (k == ~0ull) ? DRD_BG : (unsigned)k;
        float uv[2] = {0.0f, 0.0f};
        if (id != DRD_BG) {
            any = true;
            const unsigned ti = id + (unsigned)side * (unsigned)sc.n_tris;
            const TriR r = gload(&R.rec[ti]);
            const TriS sh = gload(&J.recS[ti]);
            const CornerUV cu = load_cuv(sc, id);
            float c[3], al;
            const unsigned flip = NS == 2 ? (unsigned)-side : J.flip;
            FootBox fb;
            shade_pixel<SHADE, true>(sc, vw, J.theta, J.sg, J.eps, flip, r, sh, J.recG + ti, cu, px, py, c, uv, fb, al);
            const float wt = T * al;
            rgb[0] = rgb[0] + wt * c[0];
            rgb[1] = rgb[1] + wt * c[1];
            rgb[2] = rgb[2] + wt * c[2];
            T = T * (1.0f - al);
            if constexpr (MODE == 0) {
                mine[l] = ((unsigned long long)__float_as_uint(uv[0]) << 32) | id;
                mine_v[l] = uv[1];
            }
        }
        if constexpr (MODE == 1) {
            if (inpix) {
                const long long e = pix * L + l;
                if (J.out_id) J.out_id[e] = id;
                if (J.out_uv) {
                    J.out_uv[2 * e + 0] = uv[0];
                    J.out_uv[2 * e + 1] = uv[1];
                }
            }
        }
    }

    if constexpr (MODE == 1) {
        if (inpix && J.out_rgb) {
            J.out_rgb[3 * pix + 0] = rgb[0];
            J.out_rgb[3 * pix + 1] = rgb[1];
            J.out_rgb[3 * pix + 2] = rgb[2];
        }
        return;
    }
    if constexpr (MODE == 2) {
        double loss_acc = 0.0;
        if (inpix) {
            float dr = rgb[0] - tgt[0], dg = rgb[1] - tgt[1], db = rgb[2] - tgt[2];
            loss_acc = (double)((dr * dr + dg * dg) + db * db);
        }
        loss_acc = block_sum<TB>(S.u.red, loss_acc, tid);
        if (tid == 0) *J.partial = loss_acc;
        return;
    }
    if constexpr (MODE == 0 || MODE == 3) {
        unsigned anyP, anyM;
        float P[3], M[3];
        both_sides(any ? 1u : 0u, anyP, anyM);
#pragma unroll
        for (int c = 0; c < 3; ++c) both_sides(rgb[c], P[c], M[c]);
        const bool act = inpix && (anyP | anyM) != 0u && (MODE == 3 || J.any_act);
        long long q = 0;
        if (act) q = pixel_code(J, P, M, tgt, side == 0);
        if constexpr (MODE == 3) {
            q = block_sum<TB>(S.u.qred, side == 0 ? q : 0ll, tid);
            if (tid == 0 && q != 0) atomicAdd((unsigned long long*)J.qtot, (unsigned long long)q);
        } else {
            FootBox f[LM];
            const GroupTable tb = groups_open<C>(S.u.g, false, 0u, 0u, tid);
            // Each side adds its own fragments' groups, each by the first
            // fragment that holds it; the - side leaves out what the + side
            // holds.  Empty layers have all ones for a vertex or coordinate.
            if (J.act_pos) {
                Tri3 g[LM];
#pragma unroll
                for (int l = 0; l < LM; ++l) {
                    g[l] = {{DRD_BG, DRD_BG, DRD_BG}};
                    if (l < L && act && mine[l] != ~0ull)
                        g[l] = gload((const Tri3*)(sc.tri + 3 * (long long)(unsigned)mine[l]));
                }
                bool dup[LM][3];
#pragma unroll
                for (int l = 0; l < LM; ++l)
#pragma unroll
                    for (int i = 0; i < 3; ++i) {
                        dup[l][i] = g[l].v[i] == DRD_BG;
#pragma unroll
                        for (int o = 0; o < l; ++o)
                            dup[l][i] = dup[l][i] || g[l].v[i] == g[o].v[0] || g[l].v[i] == g[o].v[1] ||
                                        g[l].v[i] == g[o].v[2];
                    }
#pragma unroll
                for (int o = 0; o < LM; ++o) {
                    if (o >= L) break;
                    unsigned gp[3], gm;
#pragma unroll
                    for (int i = 0; i < 3; ++i) both_sides(g[o].v[i], gp[i], gm);
#pragma unroll
                    for (int l = 0; l < LM; ++l)
#pragma unroll
                        for (int i = 0; i < 3; ++i)
                            dup[l][i] = dup[l][i] || (side && (g[l].v[i] == gp[0] || g[l].v[i] == gp[1] ||
                                                               g[l].v[i] == gp[2]));
                }
#pragma unroll
                for (int l = 0; l < LM; ++l) {
                    if (l >= L) break;
                    const unsigned gl[3] = {dup[l][0] ? HASH_NONE : g[l].v[0], dup[l][1] ? HASH_NONE : g[l].v[1],
                                            dup[l][2] ? HASH_NONE : g[l].v[2]};
                    table_add_all(tb, J.Rp, J.K, gl, q);
                }
            }
            for (int c = 0; c < sc.n_cls; ++c) {
                if (!J.act_cls[c]) continue;
                unsigned skip[LM];
#pragma unroll
                for (int l = 0; l < LM; ++l) {
                    f[l] = {0xFFFFFFFFu, 0xFFFFFFFFu};
                    if (l < L && act && mine[l] != ~0ull)
                        f[l] = foot_box(sc, c, __uint_as_float((unsigned)(mine[l] >> 32)), mine_v[l]);
                    skip[l] = f[l].a == 0xFFFFFFFFu ? 0xFu : foot_repeats(f[l]);
                }
#pragma unroll
                for (int o = 0; o < LM; ++o) {
                    if (o >= L) break;
                    FootBox p;
                    unsigned other;
                    both_sides(f[o].a, p.a, other);
                    both_sides(f[o].b, p.b, other);
#pragma unroll
                    for (int l = 0; l < LM; ++l) {
                        if (l > o) skip[l] |= foot_shared(f[l], f[o]);
                        if (side) skip[l] |= foot_shared(f[l], p);
                    }
                }
#pragma unroll
                for (int l = 0; l < LM; ++l)
                    if (l < L && skip[l] != 0xFu) foot_add(tb, false, J.Rp, J.K, sc, c, f[l], skip[l], q);
            }
            __syncthreads();
            // the fragments are done with: the list of occupied slots takes their place
            static_assert(sizeof(S.key) >= (2u << C::LOG2T), "slot list");
            groups_flush<C>(tb, reinterpret_cast<unsigned short*>(S.key), &S.u.g.n_list, J.Rp, J.K, sc, tid);
        }
    }
}

// Constant memory: descriptors that no kernel writes while one runs.  A batch's
// tables are read as such, with scalar loads; through plain pointers they took
// vector loads that compete with the texel reads (12-scene batch 1406 -> 1277
// us).
#define DRD_CONST __attribute__((address_space(4)))

// The job of a tile of item li of a single-scene launch's layout.
template <int NS, int MODE>
__device__ __forceinline__ TileJob single_job(const TileArgs& a, int li, int pair, int view, int tile) {
    const DScene& sc = a.sc;
    const DView& vw = a.views.v[view];
    TileJob J;
    J.sc = &sc;
    J.vw = &vw;
    J.theta = a.theta;
    J.sg = a.pert.sg ? a.pert.sg + pair * sc.sg_stride : nullptr;
    J.eps = a.pert.eps;
    J.flip = a.sgn[0] > 0.0f ? 0u : 0xFFFFFFFFu;
    const long long slot = (long long)li * NS;
    const long long base = bin_base(a.whole, a.views, a.n_views, NS, a.max_tiles, li, 0) + tile;
    J.ras.rec = a.recR + slot * sc.n_tris;
    J.ras.n_tris = sc.n_tris;
    J.ras.counts = a.counts + base;
    J.ras.bins = a.bins + base * a.cap;
    J.ras.tstride = a.whole ? vw.tiles_x * vw.tiles_y : a.max_tiles;
    J.ras.cap = a.cap;
    J.ras.spn = a.spn + 2 * slot;
    J.ras.spill = a.spill + slot * SPILL_CAP;
    J.ras.tile = tile;
    J.ras.stats = a.stats;
    J.recS = a.recS + slot * sc.n_tris;
    J.recG = a.recG + (long long)(pair - a.item0 / a.n_views) * NS * sc.n_tris;
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
    J.qtot = (MODE >= 3) ? a.qtot + pair : nullptr;
    return J;
}

// The job of a tile of an item of a batch of several scenes.
__device__ __forceinline__ TileJob batch_job(const BatchArgs& b, int item, int tile) {
    const BItem& I = *(const BItem*)((const DRD_CONST BItem*)b.items + item);
    const BScene& Sc = *(const BScene*)((const DRD_CONST BScene*)b.scenes + I.scene);
    const DView& vw = *(const DView*)((const DRD_CONST DView*)b.views + I.view);
    const DScene& sc = Sc.sc;
    TileJob J;
    J.sc = &sc;
    J.vw = &vw;
    J.theta = Sc.theta;
    J.sg = Sc.sg + I.pair * sc.sg_stride;
    J.eps = Sc.eps;
    J.flip = 0u;
    J.ras.rec = b.recR + I.rec_off;
    J.ras.n_tris = sc.n_tris;
    J.ras.counts = b.counts + I.cnt_off + tile;
    J.ras.bins = b.bins + I.bin_off + (long long)tile * I.cap;
    J.ras.tstride = vw.tiles_x * vw.tiles_y;
    J.ras.cap = I.cap;
    J.ras.spn = b.spn + 2 * I.sp_off;
    J.ras.spill = b.spill + I.sp_off * SPILL_CAP;
    J.ras.tile = tile;
    J.ras.stats = b.stats;
    J.recS = b.recS + I.rec_off;
    J.recG = b.recG + I.g_off;
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
    return J;
}

// One (item, tile) of a single-scene launch: opaque or semi-transparent
// body, specialised for the scene's shading (kernels of 30 to 40 KB of code
// and 60 registers in place of one of 90 KB and 77: the instruction cache
// holds 64 KB).
//
// interleave: the grid walks the call's tile units in (view, tile, pair)
// order, so the pairs of one tile follow each other, run at about the same
// time on one XCD and share its L2 for what they have in common: the texels
// and target pixels of the tile.  Otherwise the grid is (tile, item).
// Measured at 1024 px, 46080 triangles, GGX, 32 items: 1989 -> 1586 us
// (specialised and interleaved; the interleaved general kernel 1640 us).
template <int TILE, int MODE, int LM, int SHADE>
__global__ void __launch_bounds__((TileCfg<TILE, MODE, LM>::TB), TILE > 16 ? 1 : TILE_MIN_WAVES)
k_tile(TileArgs a) {
    constexpr bool DEEP = LM > 0;
    using SH = std::conditional_t<DEEP, DeepShared<TILE, MODE, (DEEP ? LM : 1)>, TileShared<TILE, MODE>>;
    __shared__ SH S;
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
        li = a.first + blockIdx.y;
        const int item = a.item0 + li;
        pair = item / a.n_views;
        view = item - pair * a.n_views;
        tile = xcd_tile(blockIdx.x, gridDim.x);
    }
    if (tile >= a.views.v[view].tiles_x * a.views.v[view].tiles_y) return;
    TileJob J = single_job<TileCfg<TILE, MODE, LM>::NS, MODE>(a, li, pair, view, tile);
    if constexpr (DEEP) tile_body_deep<TILE, MODE, LM, SHADE>(J, S);
    else tile_body<TILE, MODE, SHADE>(J, S);
}

// Raster / shade / scatter of every (scene, pair, view, tile) unit of a
// batch of several scenes: one workgroup per unit, units in the XCD-aware
// order of xcd_tile(), items of the costliest scenes first.
template <int TILE, int SHADE>
__global__ void __launch_bounds__((TileCfg<TILE, 0, 0>::TB), TILE > 16 ? 1 : TILE_MIN_WAVES)
k_tile_b(BatchArgs b) {
    __shared__ TileShared<TILE, 0> S;
    const long long w = b.unit0 + xcd_tile(blockIdx.x, gridDim.x);
    if (w >= b.total_tiles) return;
    const int item = __builtin_amdgcn_readfirstlane(last_le((const char*)&b.items[0].tile0, sizeof(BItem), b.n_items, w));
    TileJob J = batch_job(b, item, (int)(w - b.items[item].tile0));
    tile_body<TILE, 0, SHADE>(J, S);
}

template <int TILE, int MODE, int LM, int SHADE>
static void launch_tile_kernel(hipStream_t st, const TileArgs& a, dim3 grid) {
    hipLaunchKernelGGL((k_tile<TILE, MODE, LM, SHADE>), grid, dim3(TileCfg<TILE, MODE, LM>::TB), 0, st, a);
}

// A full-image estimate of 32-pixel tiles takes 256 threads of four pixels each,
// since more, smaller blocks hide one another's chains, but a thread per pixel
// while all blocks of 1024 threads are in flight at once (two a CU).  Whole calls
// with 1024 / 256 threads (Lambert, two views): 128 blocks 144 / 168 us, 256 blocks
// 47 / 57, 352 blocks 52 / 62, 484 blocks 59 / 55, 1444 blocks 90 / 61, 2048 blocks
// 183 / 113, 32768 blocks 1163 / 549.  (With the group table's room, which this form
// does not use, 737 for the last.)
template <int TILE, int LM, int SHADE>
static void launch_tile_mode(hipStream_t st, const TileArgs& a, int mode, dim3 grid) {
    if constexpr (TILE == 32) {
        if (mode == 3 && (long long)grid.x * grid.y <= 512) return launch_tile_kernel<TILE, 4, LM, SHADE>(st, a, grid);
    }
    if (mode == 0) launch_tile_kernel<TILE, 0, LM, SHADE>(st, a, grid);
    else if (mode == 1) launch_tile_kernel<TILE, 1, LM, SHADE>(st, a, grid);
    else if (mode == 2) launch_tile_kernel<TILE, 2, LM, SHADE>(st, a, grid);
    else launch_tile_kernel<TILE, 3, LM, SHADE>(st, a, grid);
}

template <int TILE, int LM>
static hipError_t launch_tile_shade(hipStream_t st, const TileArgs& a, int mode, dim3 grid) {
    const int shade = scene_shade(a.sc);
    if (shade == 0) launch_tile_mode<TILE, LM, 0>(st, a, mode, grid);
    else if (shade == 1) launch_tile_mode<TILE, LM, 1>(st, a, mode, grid);
    else if (shade == 2) launch_tile_mode<TILE, LM, 2>(st, a, mode, grid);
    else launch_tile_mode<TILE, LM, SHADE_ANY>(st, a, mode, grid);
    return hipGetLastError();
}

template <int TILE>
hipError_t launch_tile_t(hipStream_t st, const TileArgs& a, int mode, dim3 grid) {
    return launch_tile_shade<TILE, 0>(st, a, mode, grid);
}

// Deep kernels for up to two layers and for up to four: half the keys and
// coordinates in LDS and in the unrolled unions of the scatter (512 px, two
// layers, 32 items 1144 -> 1124 us).
template <int TILE>
hipError_t launch_tile_deep_t(hipStream_t st, const TileArgs& a, int mode, dim3 grid) {
    return a.sc.layers <= 2 ? launch_tile_shade<TILE, 2>(st, a, mode, grid)
                            : launch_tile_shade<TILE, DRD_MAX_LAYERS>(st, a, mode, grid);
}

template <int TILE>
hipError_t launch_batch_tile_t(hipStream_t st, const BatchArgs& b, unsigned grid) {
    const dim3 block(TileCfg<TILE, 0, 0>::TB);
    if (b.shade == 0) hipLaunchKernelGGL((k_tile_b<TILE, 0>), dim3(grid), block, 0, st, b);
    else if (b.shade == 1) hipLaunchKernelGGL((k_tile_b<TILE, 1>), dim3(grid), block, 0, st, b);
    else if (b.shade == 2) hipLaunchKernelGGL((k_tile_b<TILE, 2>), dim3(grid), block, 0, st, b);
    else hipLaunchKernelGGL((k_tile_b<TILE, SHADE_ANY>), dim3(grid), block, 0, st, b);
    return hipGetLastError();
}
