// dr_kernels.hip -- HIP kernels of the per-pixel stochastic gradient
// estimator for gfx950 (MI355X).
//
// Pipeline of one estimate (Sec. 4.3, Alg. 1 and 2, Eq. 8-9):
//   signs      Philox sign bits of every pair                  (shader P)
//   subdiv     (subdivision surfaces only, Sec. 6.3) the tessellated
//              vertex positions of every (pair, sign)
//   setup      per (item, sign, triangle): perturb the three vertices,
//              project, snap, build the raster record and append the
//              triangle to the bins of the tiles its bbox touches
//   tile       per (item, tile): rasterise the + and - scenes into LDS
//              depth|id keys (64-bit atomic min; the L nearest keys for
//              semi-transparent scenes), shade (and composite), form the
//              per-pixel difference and scatter it to the union of the
//              pixel's contribution groups                  (R and G fused)
//   fold       Q_i += sum_n s_i^(n) R^(n)_g(i): the per-group sums of each
//              pair become per-parameter fixed-point sums
//   step       decode, per-parameter average, Adam / SGD    (shader D)
// An "item" is one (pair, view) of a scene.  The single-scene kernels take
// their descriptors as kernel arguments; the batch kernels read them from
// device memory and cover many scenes per launch (the tile launch of a
// one-scene batch takes the scene and its views as kernel arguments too).
// All share the bodies below, so they compute the same bits.
#include "dr_launch.h"
#include "dr_wave.h"


// ---------------------------------------------------------------- signs --

// Sign words of one pair: a Philox block holds 256 signs, 8 uint32 words.
__global__ void k_signs(unsigned long long seed, unsigned step, unsigned pair, unsigned scene, long long d, int words,
                        uint32_t* __restrict__ out) {
    const long long blk = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (blk >= ((d + 255) >> 8)) return;
    unsigned long long r[4];
    philox4x64_10((unsigned long long)blk, (unsigned long long)pair, step, scene, seed, 0ull, r);
#pragma unroll
    for (int w = 0; w < 8; ++w) {
        const long long word = blk * 8 + w;
        if (word < words) out[word] = (w & 1) ? (uint32_t)(r[w >> 1] >> 32) : (uint32_t)r[w >> 1];
    }
}

// Group sign bytes (DPert): a block makes those of up to SIGN_CH groups that
// lie in one segment (the vertices, or one texel class).  The signs are
// numbered by parameter, and a group's parameters lie in up to three ranges of
// them (one per texture of the class), so the block first forms the Philox
// blocks that its ranges touch in LDS (a range starts and ends within a block,
// so two of about a hundred are formed by a neighbour too) and then gathers
// each group's bits.  Writing bytes per group instead of the words in
// parameter order: the tile kernel reads a footprint's signs in all textures
// with two 16-bit loads per side (six 64-bit ones before) and the fold a byte
// per (pair, group) instead of a word per (pair, parameter).
// Bound by the Philox rounds' 64-bit products.
#define SIGN_CH 8192

struct SignShared {
    uint32_t bits[SIGN_CH / 4 + 64];             // at most 8 bits per group, a spare block per range
};

__host__ __device__ inline long long sign_chunks(long long n) { return (n + SIGN_CH - 1) / SIGN_CH; }

__device__ __forceinline__ void group_signs_block(SignShared& S, const DScene& sc, unsigned long long seed,
                                                  unsigned step, unsigned pair, unsigned scene, long long chunk,
                                                  uint8_t* __restrict__ sg) {
    // the segment: first group, its size, and its parameter ranges
    long long goff = 0, size = sc.n_vg, first[DRD_MAX_TEX] = {0, 0, 0};
    int C[DRD_MAX_TEX] = {3, 0, 0}, bit[DRD_MAX_TEX] = {0, 0, 0};
    long long left = chunk - sign_chunks(sc.n_vg);
    if (left >= 0) {
        int c = 0;
        while (c + 1 < sc.n_cls && left >= sign_chunks((long long)sc.cls_w[c] * sc.cls_h[c])) {
            left -= sign_chunks((long long)sc.cls_w[c] * sc.cls_h[c]);
            ++c;
        }
        chunk = left;
        goff = sc.cls_goff[c];
        size = (long long)sc.cls_w[c] * sc.cls_h[c];
#pragma unroll
        for (int t = 0; t < DRD_MAX_TEX; ++t) {
            C[t] = (t < sc.n_tex && sc.tex_cls[t] == c) ? sc.tex_c[t] : 0;
            first[t] = sc.tex_off[t];
            bit[t] = sc.tex_bit[t];
        }
    }
    const long long g0 = chunk * SIGN_CH;
    const int n = (int)min((long long)SIGN_CH, size - g0), tid = threadIdx.x;
    // Philox blocks of each range, end to end
    long long blk0[DRD_MAX_TEX];
    int at[DRD_MAX_TEX + 1];
    at[0] = 0;
#pragma unroll
    for (int t = 0; t < DRD_MAX_TEX; ++t) {
        const long long b0 = first[t] + g0 * C[t], b1 = b0 + (long long)n * C[t];
        blk0[t] = b0 >> 8;
        at[t + 1] = at[t] + (C[t] > 0 ? (int)(((b1 - 1) >> 8) - blk0[t]) + 1 : 0);
    }
    for (int i = tid; i < at[DRD_MAX_TEX]; i += (int)blockDim.x) {
        long long blk = blk0[0] + i;
#pragma unroll
        for (int t = 1; t < DRD_MAX_TEX; ++t)
            if (i >= at[t]) blk = blk0[t] + (i - at[t]);
        unsigned long long r[4];
        philox4x64_10((unsigned long long)blk, (unsigned long long)pair, step, scene, seed, 0ull, r);
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            S.bits[8 * i + 2 * w] = (uint32_t)r[w];
            S.bits[8 * i + 2 * w + 1] = (uint32_t)(r[w] >> 32);
        }
    }
    __syncthreads();
    // four groups at a time
    typedef uint32_t __attribute__((aligned(1))) u32a1;
    for (int q = 4 * tid; q < n; q += 4 * (int)blockDim.x) {
        uint32_t out = 0u;
#pragma unroll
        for (int t = 0; t < DRD_MAX_TEX; ++t) {
            if (C[t] == 0) continue;
            // the range's bits of these groups: at most 16, within two words
            const unsigned b = (unsigned)((first[t] + g0 * C[t]) & 255) + (unsigned)(q * C[t]);
            const uint32_t* w = &S.bits[8 * at[t] + (b >> 5)];
            const uint32_t x = __builtin_amdgcn_alignbit(w[1], w[0], b & 31u);
            const uint32_t m = (1u << C[t]) - 1u;
#pragma unroll
            for (int k = 0; k < 4; ++k) out |= ((x >> (k * C[t])) & m) << (8 * k + bit[t]);
        }
        uint8_t* p = sg + goff + g0 + q;
        if (q + 4 <= n) *(u32a1*)p = out;
        else
            for (int k = 0; k < n - q; ++k) p[k] = (uint8_t)(out >> (8 * k));
    }
}

__global__ void __launch_bounds__(256) k_group_signs(DScene sc, unsigned long long seed, unsigned step, unsigned pair0,
                                                     unsigned scene, uint8_t* __restrict__ sg) {
    __shared__ SignShared S;
    group_signs_block(S, sc, seed, step, pair0 + blockIdx.y, scene, blockIdx.x, sg + blockIdx.y * sc.sg_stride);
}

// ---------------------------------------------------------------- setup --

// The perturbed world positions of triangle t's corners (original order).
// fpos: the perturbed tessellated vertex positions of this (pair, sign) of a
// subdivision surface, or null (positions are the perturbed parameters).
__device__ __forceinline__ void tri_positions(const DScene& sc, const float* __restrict__ theta,
                                              const uint8_t* __restrict__ sg, float e0, float sgn, int t,
                                              const float* __restrict__ fpos, float* p) {
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const long long vid = sc.tri[3 * (long long)t + k];
        if (fpos) {
            p[3 * k + 0] = fpos[3 * vid + 0];
            p[3 * k + 1] = fpos[3 * vid + 1];
            p[3 * k + 2] = fpos[3 * vid + 2];
        } else {
            perturbed_vertex(theta, vid, e0, sg, sgn, p + 3 * k);
        }
    }
}

// Tiles a triangle's pixel box touches: [x0, x1] x [y0, y1], empty when
// x0 > x1.
struct TileRect {
    int x0, x1, y0, y1;
};

// What the views of one perturbation share of a face's shading, from its
// perturbed corners p: the Lambert shade (returned), or the GGX record
// (stored to G when it is given).
__device__ __forceinline__ float face_shade(const DScene& sc, const float* p, int t, TriG* __restrict__ G) {
    if (sc.shading == 0) return 0.0f;
    float nf[3];
    face_normal(p, nf);
    if (sc.shading == 1) {
        float ndl = dot3(nf, sc.light);
        if (!(ndl > 0.0f)) ndl = 0.0f;
        return sc.ambient + sc.diffuse * ndl;
    }
    if (G) {
        TriG g;
#pragma unroll
        for (int k = 0; k < 9; ++k) g.p[k] = p[k];
#pragma unroll
        for (int k = 0; k < 3; ++k) g.nf[k] = nf[k];
        const CornerUV cu = load_cuv(sc, (unsigned)t);
        face_tangent(p, cu.c, nf, g.T);
        g.pad = 0.0f;
        G[t] = g;
    }
    return 0.0f;
}

// Raster record of triangle t in one view from its perturbed corners p;
// returns the tiles its box touches (tile size 1 << lg pixels).
__device__ __forceinline__ TileRect setup_tri_at(const DView& vw, const float* p, int t, TriR* __restrict__ recR,
                                                 TriS* __restrict__ recS, float shade, int lg) {
    const TileRect none = {1, 0, 1, 0};
    Vtx v[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) v[k] = xform(vw, p[3 * k + 0], p[3 * k + 1], p[3 * k + 2]);
    TriR r;
    TriS sh;
    r.flags = 0u;
    r.ia = 0.0f;
    r.pad = 0;
    bool ok = v[0].valid && v[1].valid && v[2].valid;
    long long area2 = 0;
    if (ok) {
        area2 = (long long)(v[1].X - v[0].X) * (long long)(v[2].Y - v[0].Y) -
                (long long)(v[1].Y - v[0].Y) * (long long)(v[2].X - v[0].X);
        ok = area2 != 0;
    }
    if (!ok) {
        recR[t] = r;                 // flags 0: culled
        return none;
    }
    bool sw = area2 < 0;
    if (sw) {
        area2 = -area2;
        Vtx tmp = v[1]; v[1] = v[2]; v[2] = tmp;
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) { r.X[k] = v[k].X; r.Y[k] = v[k].Y; sh.iw[k] = v[k].iw; }
    unsigned fl = TRI_VALID | (sw ? TRI_SWAPPED : 0u);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        int ia = (k + 1) % 3, ib = (k + 2) % 3;
        int dx = r.X[ib] - r.X[ia], dy = r.Y[ib] - r.Y[ia];
        if ((dy < 0) || (dy == 0 && dx > 0)) fl |= (2u << k);
    }
    r.flags = fl;
    float d1 = v[1].z - v[0].z, d2 = v[2].z - v[0].z;
    float fX1 = (float)(r.X[1] - r.X[0]), fY1 = (float)(r.Y[1] - r.Y[0]);
    float fX2 = (float)(r.X[2] - r.X[0]), fY2 = (float)(r.Y[2] - r.Y[0]);
    float fa = (float)area2;
    r.z0 = v[0].z;
    r.zx = (d1 * fY2 - d2 * fY1) / fa;
    r.zy = (d2 * fX1 - d1 * fX2) / fa;
    r.ia = 1.0f / fa;
    int xmin = min(r.X[0], min(r.X[1], r.X[2])), xmax = max(r.X[0], max(r.X[1], r.X[2]));
    int ymin = min(r.Y[0], min(r.Y[1], r.Y[2])), ymax = max(r.Y[0], max(r.Y[1], r.Y[2]));
    if (xmax - xmin < 32000 && ymax - ymin < 32000) r.flags |= TRI_SMALL;
    // pixels whose centre 256 x + 128 lies in [min, max]
    int bx0 = max((xmin + 127) >> 8, 0), bx1 = min((xmax - 128) >> 8, vw.W - 1);
    int by0 = max((ymin + 127) >> 8, 0), by1 = min((ymax - 128) >> 8, vw.H - 1);
    sh.sh = shade;
    recR[t] = r;
    recS[t] = sh;
    if (bx0 > bx1 || by0 > by1) return none;    // no pixel centre in the bbox
    return {bx0 >> lg, bx1 >> lg, by0 >> lg, by1 >> lg};
}

// Binning of a block's 256 triangles (one per thread) in one view.
//
// A bin entry takes its place from the tile's counter.  Neighbouring
// triangles share tiles, so the block first counts its entries per tile in
// LDS, over the rectangle of tiles that its triangles touch, then adds each
// tile's total to the tile's counter with one global atomic (all tiles at
// once), and gives the entries their places by counting up from the returned
// bases.  Whatever the triangles' sizes, a block waits for one round of
// global atomics; a rectangle of more than BIN_SLOTS tiles takes one atomic
// per entry instead.  Threads walk their own triangle's tiles while none
// touches more than BIN_OWN of them; past that the block shares all entries
// evenly (prefix sums and a binary search for the owner), since a thread
// with hundreds of tiles would leave the others waiting.
//
// Bound by the latency of the chain index -> vertices -> counter -> entry
// where few blocks run, by the record writes where many do.  Measured against
// one counter round per tile of a wave's largest triangle: 2 renders of 20480
// triangles at 512 px 15.7 -> 8.6 us, 256 renders of a 10240-triangle soup
// 368 -> 133 us, 64 renders of 46080 triangles at 1024 px 130 -> 100 us, one
// render of 2420 triangles over 8 px tiles 222 -> 9 us.
#define SETUP_TB 256
#define BIN_SLOTS 4096
#define BIN_OWN 16

struct BinShared {
    unsigned tab[BIN_SLOTS];         // entries per tile of the block's rectangle, then places
    int red[SETUP_TB / 64][8];       // per-wave rectangle, largest and total entry count
    int incl[SETUP_TB];              // inclusive prefix sums of the entry counts (shared walk)
    int4 rect[SETUP_TB];
};

// The bins of one (item, sign): counters, entries and the spill list.
struct BinOut {
    unsigned* counts;
    unsigned* bins;
    int cap;
    unsigned* spn;
    unsigned long long* spill;
};

// Entry k of a tile's bin.  Entries past the capacity go to the render's
// spill list (the first of a tile also counts the tile as overflowing).
__device__ __forceinline__ void bin_put(const BinOut& o, int tile, unsigned k, unsigned t) {
    if (k < (unsigned)o.cap) {
        o.bins[(long long)tile * o.cap + k] = t;
        return;
    }
    if (!o.spill) return;
    const unsigned long long ms = __ballot(true);               // the lanes that spill together
    const int first = __ffsll((long long)ms) - 1;
    const unsigned below = __builtin_amdgcn_mbcnt_hi((unsigned)(ms >> 32),
                                                     __builtin_amdgcn_mbcnt_lo((unsigned)ms, 0u));
    unsigned j0 = 0u;
    if (below == 0u) j0 = atomicAdd(&o.spn[0], (unsigned)__popcll(ms));
    const unsigned j = __shfl(j0, first) + below;
    if (j < SPILL_CAP) o.spill[j] = ((unsigned long long)(unsigned)tile << 32) | t;
    if (k == (unsigned)o.cap) atomicAdd(&o.spn[1], 1u);
}

// r: the tiles of this thread's triangle t (x0 > x1: none); t0: the block's
// first triangle.  Called by every thread of the block.
__device__ __forceinline__ void bin_block(BinShared& S, const TileRect& r, int tiles_x, int t0, const BinOut& o) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const bool has = r.x0 <= r.x1;
    const int ntx = has ? r.x1 - r.x0 + 1 : 0;
    const int n = has ? ntx * (r.y1 - r.y0 + 1) : 0;
    const int big = 0x7fffffff;
    const int wx0 = -wave_max(has ? -r.x0 : -big), wx1 = wave_max(has ? r.x1 : -1);
    const int wy0 = -wave_max(has ? -r.y0 : -big), wy1 = wave_max(has ? r.y1 : -1);
    const int wn = wave_max(n);
    if (lane == 0) {
        int* q = S.red[wave];
        q[0] = wx0; q[1] = wx1; q[2] = wy0; q[3] = wy1; q[4] = wn;
    }
    __syncthreads();
    int x0 = big, x1 = -1, y0 = big, y1 = -1, nmax = 0;
#pragma unroll
    for (int w = 0; w < SETUP_TB / 64; ++w) {
        x0 = min(x0, S.red[w][0]); x1 = max(x1, S.red[w][1]);
        y0 = min(y0, S.red[w][2]); y1 = max(y1, S.red[w][3]);
        nmax = max(nmax, S.red[w][4]);
    }
    if (nmax == 0) return;                                      // (uniform)
    const int rw = x1 - x0 + 1;
    const long long area = (long long)rw * (y1 - y0 + 1);
    const bool local = area <= BIN_SLOTS;
    const bool own = nmax <= BIN_OWN;
    if (local)
        for (int j = tid; j < (int)area; j += SETUP_TB) S.tab[j] = 0u;
    if (!own) {
        // inclusive prefix sums of the entry counts over the block
        const int incl = wave_inclusive_sum(n);
        if (lane == 63) S.red[wave][5] = incl;
        S.rect[tid] = make_int4(r.x0, r.y0, ntx, 0);
        __syncthreads();
        int off = 0;
        for (int w = 0; w < wave; ++w) off += S.red[w][5];
        S.incl[tid] = off + incl;
    }
    __syncthreads();
    const int P = own ? 0 : S.incl[SETUP_TB - 1];
    // entry p of the block: its owner by binary search, its tile by its
    // place in the owner's rectangle
    auto entry = [&](int p, int& tx, int& ty) -> int {
        int lo = 0, hi = SETUP_TB - 1;                          // first owner whose sum exceeds p
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const int mid = (lo + hi) >> 1;
            if (S.incl[mid] > p) hi = mid;
            else lo = mid + 1;
        }
        const int4 q = S.rect[lo];
        const int i = p - (lo > 0 ? S.incl[lo - 1] : 0);
        const int iy = i / q.z;
        tx = q.x + (i - iy * q.z);
        ty = q.y + iy;
        return lo;
    };
    if (local) {
        if (own) {
            for (int ty = r.y0; ty <= r.y1; ++ty)
                for (int tx = r.x0; tx <= r.x1; ++tx) atomicAdd(&S.tab[(ty - y0) * rw + (tx - x0)], 1u);
        } else {
            for (int p = tid; p < P; p += SETUP_TB) {
                int tx, ty;
                (void)entry(p, tx, ty);
                atomicAdd(&S.tab[(ty - y0) * rw + (tx - x0)], 1u);
            }
        }
        __syncthreads();
        const float inv = 1.0f / (float)rw;
        for (int j = tid; j < (int)area; j += SETUP_TB) {
            const unsigned c = S.tab[j];
            if (c == 0u) continue;
            const int jy = (int)(((float)j + 0.5f) * inv);      // j / rw (exact: j < 4096)
            S.tab[j] = atomicAdd(&o.counts[(y0 + jy) * tiles_x + x0 + (j - jy * rw)], c);
        }
        __syncthreads();
    }
    if (own) {
        for (int ty = r.y0; ty <= r.y1; ++ty)
            for (int tx = r.x0; tx <= r.x1; ++tx) {
                const int tile = ty * tiles_x + tx;
                const unsigned k = local ? atomicAdd(&S.tab[(ty - y0) * rw + (tx - x0)], 1u)
                                         : atomicAdd(&o.counts[tile], 1u);
                bin_put(o, tile, k, (unsigned)(t0 + tid));
            }
    } else {
        for (int p = tid; p < P; p += SETUP_TB) {
            int tx, ty;
            const int w = entry(p, tx, ty);
            const int tile = ty * tiles_x + tx;
            const unsigned k = local ? atomicAdd(&S.tab[(ty - y0) * rw + (tx - x0)], 1u)
                                     : atomicAdd(&o.counts[tile], 1u);
            bin_put(o, tile, k, (unsigned)(t0 + w));
        }
    }
}

// Setup of a block's 256 triangles of one (pair, sign) in its views: the
// perturbed corners and what the views share of the shading are formed once,
// then each view's record and bin entries.  The launcher gives a block all
// views of a call when that leaves blocks enough to fill the chip, else one.
__global__ void __launch_bounds__(SETUP_TB) k_setup(SetupArgs a) {
    __shared__ BinShared S;
    const DScene& sc = a.sc;
    int y = blockIdx.y;                          // (local item, sign), or (pair, sign, views)
    int li, s, nv = 1;
    if (a.whole) {
        const int nvc = (a.n_views + a.vpb - 1) / a.vpb;
        const int vc = y % nvc;
        y /= nvc;
        s = y % a.nsign;
        li = (y / a.nsign) * a.n_views + vc * a.vpb;
        nv = min(a.vpb, a.n_views - vc * a.vpb);
    } else {
        s = y % a.nsign;
        li = y / a.nsign;
    }
    const int pair = (a.item0 + li) / a.n_views, pair0 = a.item0 / a.n_views;
    const int t0 = (int)blockIdx.x * SETUP_TB, t = t0 + (int)threadIdx.x;
    const int lg = 31 - __clz(a.tile);
    float p[9], shade = 0.0f;
    if (t < sc.n_tris) {
        const uint8_t* sg = a.pert.sg ? a.pert.sg + pair * sc.sg_stride : nullptr;
        const float* fpos = a.fpos ? a.fpos + ((long long)pair * a.nsign + s) * 3 * sc.n_verts : nullptr;
        tri_positions(sc, a.theta, sg, a.pert.eps[0], a.sgn[s], t, fpos, p);
        // the first view of the pair in this launch stores what all share
        const bool first = li == 0 || (a.item0 + li) - pair * a.n_views == 0;
        shade = face_shade(sc, p, t, first ? a.recG + (long long)((pair - pair0) * a.nsign + s) * sc.n_tris : nullptr);
    }
    for (int i = 0; i < nv; ++i, ++li) {
        const DView& vw = a.views.v[a.item0 + li - pair * a.n_views];
        const long long slot = (long long)li * a.nsign + s;
        const long long base = bin_base(a.whole, a.views, a.n_views, a.nsign, a.max_tiles, li, s);
        TileRect r = {1, 0, 1, 0};
        if (t < sc.n_tris) r = setup_tri_at(vw, p, t, a.recR + slot * sc.n_tris, a.recS + slot * sc.n_tris, shade, lg);
        if (i > 0) __syncthreads();              // the view before is done with the shared tables
        const BinOut o = {a.counts + base, a.bins + base * a.cap, a.cap, a.spn + 2 * slot, a.spill + slot * SPILL_CAP};
        bin_block(S, r, vw.tiles_x, t0, o);
    }
}

// Tessellated vertex positions of a subdivision surface for every (pair,
// sign) of a call: vertex j, coordinate c = the row's weights times the
// perturbed control coordinates, added in row order from zero.
__global__ void __launch_bounds__(256) k_subdiv(DScene sc, DPert pert, const float* __restrict__ theta, int nsign,
                                                float sgn0, float sgn1, float* __restrict__ fpos) {
    int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= sc.n_verts) return;
    int slot = blockIdx.y;                       // (pair, sign)
    int pair = slot / nsign, s = slot % nsign;
    const uint8_t* sg = pert.sg ? pert.sg + pair * sc.sg_stride : nullptr;
    float sgn = s == 0 ? sgn0 : sgn1;
    float e0 = pert.eps[0];
    int k0 = sc.sub_rowptr[j], k1 = sc.sub_rowptr[j + 1];
    float acc[3] = {0.0f, 0.0f, 0.0f};
    for (int k = k0; k < k1; ++k) {
        float w = sc.sub_w[k];
        float p[3];
        perturbed_vertex(theta, sc.sub_cols[k], e0, sg, sgn, p);
#pragma unroll
        for (int c = 0; c < 3; ++c) acc[c] = acc[c] + w * p[c];
    }
    float* out = fpos + ((long long)slot * sc.n_verts + j) * 3;
    out[0] = acc[0];
    out[1] = acc[1];
    out[2] = acc[2];
}

// Per-view loss: the tiles' partial sums added in tile order (one block per
// view, fixed-order reduction), so the value is reproducible run to run.
__global__ void __launch_bounds__(256) k_sum_tiles(const double* __restrict__ partials, int max_tiles,
                                                   DViews views, double* __restrict__ out) {
    __shared__ double red[256];
    int v = blockIdx.x, tid = threadIdx.x;
    int n = views.v[v].tiles_x * views.v[v].tiles_y;
    double acc = 0.0;
    for (int t = tid; t < n; t += 256) acc += partials[(long long)v * max_tiles + t];
    red[tid] = acc;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (tid < w) red[tid] = red[tid] + red[tid + w];
        __syncthreads();
    }
    if (tid == 0) out[v] = red[0];
}

// -------------------------------------------------------------- fold --

// Parameters of group g as vectors: calls fn(size, first param, block, first
// sign bit) for a vertex's three coordinates, or a texel's channels (1, 3 or 4)
// in each texture of its class.  One wide access per array and vector in place of strided
// single ones: the step at 7.3 M parameters 85 -> 43 us, the fold of 8 pairs 47 -> 37, both in one
// 61 -> 51.
template <typename Fn>
__device__ __forceinline__ void for_vectors(const DScene& sc, long long g, Fn fn) {
    if (g < sc.n_vg) {
        fn(std::integral_constant<int, 3>{}, 3 * g, 0, 0);
        return;
    }
    for (int c = 0; c < sc.n_cls; ++c) {
        const long long size = (long long)sc.cls_w[c] * sc.cls_h[c];
        const long long texel = g - sc.cls_goff[c];
        if (texel < 0 || texel >= size) continue;
        for (int t = 0; t < sc.n_tex; ++t) {
            if (sc.tex_cls[t] != c) continue;
            const int C = sc.tex_c[t], k = sc.tex_bit[t];
            const long long i = sc.tex_off[t] + texel * C;
            if (C == 1) fn(std::integral_constant<int, 1>{}, i, 1 + t, k);
            else if (C == 3) fn(std::integral_constant<int, 3>{}, i, 1 + t, k);
            else fn(std::integral_constant<int, 4>{}, i, 1 + t, k);
        }
    }
}

template <typename T, int C>
struct Vec {
    T c[C];
};

template <int C, typename T>
__device__ __forceinline__ Vec<T, C> vload(const T* p) {
    return gload((const Vec<T, C>*)p);
}

template <int C, typename T>
__device__ __forceinline__ void vstore(T* p, const Vec<T, C>& v) {
#pragma unroll
    for (int ch = 0; ch < C; ++ch) ((DRD_GLOBAL T*)p)[ch] = v.c[ch];
}

// v with sign -1 where bit k of b is set
__device__ __forceinline__ long long signed_by(long long v, unsigned b, int k) {
    const long long m = -(long long)((b >> k) & 1u);
    return (v ^ m) - m;
}

// Q_i += sum_n s_i^(n) R_g^(n) for the parameters of group g, then R_g = 0.
// Pairs are taken 8 at a time: the group's 8 sums and sign bytes are read
// once (not once per parameter), a chunk that is all zero (the group was not
// seen by those pairs) changes nothing, and only non-zero sums are cleared.
__device__ __forceinline__ void fold_group(const DScene& sc, long long g, long long* __restrict__ R,
                                           const uint8_t* __restrict__ sg, int n_pairs, const float* eps,
                                           long long* __restrict__ Q) {
    for (int n0 = 0; n0 < n_pairs; n0 += 8) {
        long long r[8];
        unsigned b[8];
        bool any = false;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const bool in = n0 + j < n_pairs;
            r[j] = in ? R[(long long)(n0 + j) * sc.G + g] : 0;
            b[j] = in ? sg[(n0 + j) * sc.sg_stride + g] : 0u;
            any = any || r[j] != 0;
        }
        if (!any) continue;
        for_vectors(sc, g, [&](auto size, long long i, int blk, int k) {
            constexpr int C = decltype(size)::value;
            if (eps[blk] == 0.0f) return;
            Vec<long long, C> q = vload<C>(Q + i);
#pragma unroll
            for (int ch = 0; ch < C; ++ch)
#pragma unroll
                for (int j = 0; j < 8; ++j) q.c[ch] += signed_by(r[j], b[j], k + ch);
            vstore<C>(Q + i, q);
        });
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (r[j] != 0) R[(long long)(n0 + j) * sc.G + g] = 0;
    }
}

// The last kernel of an estimate tells the host the largest bin seen so far.
__device__ __forceinline__ void tell_max_bin(const FoldArgs& a, long long g) {
    if (g == 0 && a.seen) __hip_atomic_store(a.seen, a.stats[ST_MAX_BIN], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Full-image estimate: every parameter of an active block gets
// s_i^(n) * T[n] for every pair n; every active group counts one
// contribution per (pair, view).  T is zeroed by k_zero64 before the call.
__global__ void __launch_bounds__(256) k_broadcast(FoldArgs a) {
    long long g = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const DScene& sc = a.sc;
    if (g >= sc.G) return;
    tell_max_bin(a, g);
    bool active = false;
    for_vectors(sc, g, [&](auto size, long long i, int b, int k) {
        constexpr int C = decltype(size)::value;
        if (a.eps[b] == 0.0f) return;
        active = true;
        Vec<long long, C> q = vload<C>(a.Q + i);
        // eight pairs' reads in flight together: a scene of few groups waits for
        // them (40960 groups, 128 pairs: 50 -> 17 us)
        for (int n0 = 0; n0 < a.n_pairs; n0 += 8) {
            long long r[8];
            unsigned sb[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int n = min(n0 + j, a.n_pairs - 1);
                r[j] = n0 + j < a.n_pairs ? a.qtot[n] : 0;
                sb[j] = gload(&a.sg[n * sc.sg_stride + g]);
            }
#pragma unroll
            for (int j = 0; j < 8; ++j)
#pragma unroll
                for (int ch = 0; ch < C; ++ch) q.c[ch] += signed_by(r[j], sb[j], k + ch);
        }
        vstore<C>(a.Q + i, q);
    });
    if (!active) return;
    a.K[g] += (unsigned)(a.n_pairs * a.n_views);
}

__global__ void k_zero64(long long* p, int n) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}

__global__ void __launch_bounds__(256) k_fold(FoldArgs a) {
    long long g = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= a.sc.G) return;
    tell_max_bin(a, g);
    fold_group(a.sc, g, a.R, a.sg, a.n_pairs, a.eps, a.Q);
}

// ------------------------------------------------------ step / decode --

// The decoded gradient of an accumulated sum (D: the divisor; 0: none).
__device__ __forceinline__ float decoded(long long q, float e, double D) {
    float gi = 0.0f;
    if (e != 0.0f && D != 0.0) gi = (float)(((double)q * (1.0 / 4294967296.0)) / (2.0 * (double)e * D));
    return gi;
}

// One optimiser step of C adjacent parameters with gradient gi; a parameter
// whose gradient is not finite stays as it is and is counted.
template <int C>
__device__ __forceinline__ void update(const OptimConst& oc, float l, float bc1, float bc2, const float (&gi)[C],
                                       float* __restrict__ theta, float* __restrict__ m, float* __restrict__ v,
                                       unsigned long long* __restrict__ stats) {
    Vec<float, C> th = vload<C>(theta), mo{}, vo{};
    if (oc.kind != 1) {
        mo = vload<C>(m);
        vo = vload<C>(v);
    }
#pragma unroll
    for (int ch = 0; ch < C; ++ch) {
        if (!(fabsf(gi[ch]) <= 3.402823466e38f)) {
            atomicAdd(&stats[ST_NONFINITE], 1ull);
            continue;
        }
        if (oc.kind == 1) {
            th.c[ch] = th.c[ch] - l * gi[ch];
        } else {
            float mi = oc.b1 * mo.c[ch] + oc.omb1 * gi[ch];
            float vi = oc.b2 * vo.c[ch] + oc.omb2 * (gi[ch] * gi[ch]);
            mo.c[ch] = mi;
            vo.c[ch] = vi;
            float mh = mi / bc1;
            float vh = vi / bc2;
            th.c[ch] = th.c[ch] - l * (mh / (sqrtf(vh) + oc.eps_hat));
        }
    }
    vstore<C>(theta, th);
    if (oc.kind != 1) {
        vstore<C>(m, mo);
        vstore<C>(v, vo);
    }
}

__device__ __forceinline__ void step_group(const DScene& sc, long long g, const float* eps, const float* lr,
                                           int n_pairs, const OptimConst& oc, float bc1, float bc2,
                                           int decode_only, float* __restrict__ theta, float* __restrict__ m,
                                           float* __restrict__ v, long long* __restrict__ Q,
                                           unsigned* __restrict__ K, float* __restrict__ grad,
                                           unsigned long long* __restrict__ stats) {
    unsigned kc = K[g];
    double D = (oc.averaging == 0) ? (double)kc : (double)n_pairs;
    for_vectors(sc, g, [&](auto size, long long i, int b, int) {
        constexpr int C = decltype(size)::value;
        const float e = eps[b];
        if (decode_only) {
            // no sums are read where there is no gradient (7.4 M parameters, 1024 px
            // GGX maps: none of the groups counted 14.1 -> 10.3 us, a tenth of them
            // 15.7 -> 13.1, all of them 16.4 either way)
            Vec<float, C> go{};
            if (e != 0.0f && D != 0.0) {
                const Vec<long long, C> q = vload<C>(Q + i);
#pragma unroll
                for (int ch = 0; ch < C; ++ch) go.c[ch] = decoded(q.c[ch], e, D);
            }
            vstore<C>(grad + i, go);
            return;
        }
        const Vec<long long, C> q = vload<C>(Q + i);
        float gi[C];
        bool some = false;
#pragma unroll
        for (int ch = 0; ch < C; ++ch) {
            gi[ch] = decoded(q.c[ch], e, D);
            some = some || q.c[ch] != 0;
        }
        if (some) vstore<C>(Q + i, Vec<long long, C>{});
        if (e == 0.0f) return;
        if (oc.averaging == 0 && kc == 0u) return;
        update<C>(oc, lr[b], bc1, bc2, gi, theta + i, m + i, v + i, stats);
    });
    if (!decode_only) K[g] = 0u;
}

__global__ void __launch_bounds__(256) k_step(StepArgs a) {
    long long g = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= a.sc.G) return;
    step_group(a.sc, g, a.eps, a.lr, a.n_pairs, a.oc, a.bc1, a.bc2, a.decode_only, a.theta, a.m, a.v, a.Q, a.K,
               a.grad, a.stats);
}

// -------------------------------------------------------- k_check_tri --

// Counts vertex indices outside [0, n_verts): run once when a context is
// created, so no later kernel can index outside the vertex array.
__global__ void k_check_tri(const int* __restrict__ tri, long long n, int n_verts,
                            unsigned long long* __restrict__ bad) {
    long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    int v = tri[i];
    if (v < 0 || v >= n_verts) atomicAdd(bad, 1ull);
}

// -------------------------------------------------------------- batch --

__global__ void k_batch_end(unsigned* step) { *step = *step + 1u; }

// Group sign bytes of every (scene, pair): the blocks of a scene are
// contiguous, sign_nblk per pair.
__global__ void __launch_bounds__(256) k_signs_b(BatchArgs b) {
    __shared__ SignShared SH;
    const long long blk = blockIdx.x;
    int si = last_le((const char*)&b.scenes[0].sign_blk0, sizeof(BScene), b.n_scenes, blk);
    si = __builtin_amdgcn_readfirstlane(si);
    const BScene& S = b.scenes[si];
    const long long local = blk - S.sign_blk0;
    const int pair = (int)(local / S.sign_nblk);
    group_signs_block(SH, S.sc, b.seed, *b.step, (unsigned)pair, (unsigned)S.scene_index, local - pair * S.sign_nblk,
                      S.sg + pair * S.sc.sg_stride);
}

// Setup of every (item, sign, triangle) of a batch of several scenes: each
// (item, sign) starts on a block boundary.
__global__ void __launch_bounds__(SETUP_TB) k_setup_b(BatchArgs b) {
    __shared__ BinShared SB;
    long long blk = b.unit0 + blockIdx.x;
    int it = last_le((const char*)&b.items[0].setup_blk0, sizeof(BItem), b.n_items, blk);
    it = __builtin_amdgcn_readfirstlane(it);
    const BItem& I = b.items[it];
    const BScene& S = b.scenes[I.scene];
    const DScene& sc = S.sc;
    long long per_sign = ((long long)sc.n_tris + 255) >> 8;
    long long local = blk - I.setup_blk0;
    int s = (int)(local / per_sign);
    const int t0 = (int)(local - s * per_sign) * SETUP_TB, t = t0 + (int)threadIdx.x;
    const DView& vw = b.views[I.view];
    const int tiles = vw.tiles_x * vw.tiles_y;
    TileRect r = {1, 0, 1, 0};
    if (t < sc.n_tris) {
        float p[9];
        tri_positions(sc, S.theta, S.sg + I.pair * sc.sg_stride, S.eps[0], s == 0 ? 1.0f : -1.0f, t, nullptr, p);
        // the items of a pair share its GGX records, stored by the first view's
        const float shade = face_shade(sc, p, t, I.view == S.view0 ? b.recG + I.g_off + (long long)s * sc.n_tris : nullptr);
        r = setup_tri_at(vw, p, t, b.recR + I.rec_off + (long long)s * sc.n_tris,
                         b.recS + I.rec_off + (long long)s * sc.n_tris, shade, 31 - __clz(b.tile));
    }
    const BinOut o = {b.counts + I.cnt_off + (long long)s * tiles, b.bins + I.bin_off + (long long)s * tiles * I.cap,
                      I.cap, b.spn + 2 * (I.sp_off + s), b.spill + (I.sp_off + s) * SPILL_CAP};
    bin_block(SB, r, vw.tiles_x, t0, o);
}

// Fold and step over the groups of every scene: each scene starts on a
// block boundary.
__global__ void __launch_bounds__(256) k_fold_b(BatchArgs b) {
    long long blk = blockIdx.x;
    int si = last_le((const char*)&b.scenes[0].group_blk0, sizeof(BScene), b.n_scenes, blk);
    si = __builtin_amdgcn_readfirstlane(si);
    const BScene& S = b.scenes[si];
    long long g = (blk - S.group_blk0) * 256 + threadIdx.x;
    if (g >= S.sc.G) return;
    fold_group(S.sc, g, S.R, S.sg, b.n_pairs, S.eps, S.Q);
}

__global__ void __launch_bounds__(256) k_step_b(BatchArgs b) {
    long long blk = blockIdx.x;
    int si = last_le((const char*)&b.scenes[0].group_blk0, sizeof(BScene), b.n_scenes, blk);
    si = __builtin_amdgcn_readfirstlane(si);
    const BScene& S = b.scenes[si];
    long long g = (blk - S.group_blk0) * 256 + threadIdx.x;
    if (g >= S.sc.G) return;
    unsigned t = *b.step;
    if (t < 1u) t = 1u;                      // Adam steps count from 1
    int ti = (int)min(t, (unsigned)b.n_bc) - 1;
    step_group(S.sc, g, S.eps, S.lr, b.n_pairs, b.oc, b.bc1[ti], b.bc2[ti], 0, (float*)S.theta, S.m, S.v, S.Q,
               S.K, nullptr, b.stats);
}

// Fold and step fused, for a descent over at most 8 pairs: each group's
// per-pair sums are read once and every parameter of the group goes from
// its sum straight to the update, so the fixed-point sums Q are not written
// and read back in between.  Q_i + sum_n s_i^(n) R_g^(n) is the value the
// fold would leave in Q; it is used as step_group uses Q, and Q, R and K are
// left zero as the two kernels leave them.
// q_zero: Q is known to be zero (not read).
__device__ __forceinline__ void fold_step_group(const DScene& sc, long long g, long long* __restrict__ R,
                                                const uint8_t* __restrict__ sg, int n_pairs, const float* eps,
                                                const float* lr, const OptimConst& oc, float bc1, float bc2,
                                                float* __restrict__ theta, float* __restrict__ m,
                                                float* __restrict__ v, long long* __restrict__ Q,
                                                unsigned* __restrict__ K, unsigned long long* __restrict__ stats,
                                                int q_zero) {
    long long r[8];
    unsigned sb[8];
    bool any = false;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        r[j] = (j < n_pairs) ? R[(long long)j * sc.G + g] : 0;
        sb[j] = (j < n_pairs) ? sg[j * sc.sg_stride + g] : 0u;
        any = any || r[j] != 0;
    }
    unsigned kc = K[g];
    double D = (oc.averaging == 0) ? (double)kc : (double)n_pairs;
    for_vectors(sc, g, [&](auto size, long long i, int b, int k) {
        constexpr int C = decltype(size)::value;
        const float e = eps[b];
        Vec<long long, C> q{};
        if (!q_zero) {
            q = vload<C>(Q + i);
            bool some = false;
#pragma unroll
            for (int ch = 0; ch < C; ++ch) some = some || q.c[ch] != 0;
            if (some) vstore<C>(Q + i, Vec<long long, C>{});
        }
        if (e == 0.0f) return;
        if (oc.averaging == 0 && kc == 0u) return;
        float gi[C];
#pragma unroll
        for (int ch = 0; ch < C; ++ch) {
            if (any) {
#pragma unroll
                for (int j = 0; j < 8; ++j) q.c[ch] += signed_by(r[j], sb[j], k + ch);
            }
            gi[ch] = decoded(q.c[ch], e, D);
        }
        update<C>(oc, lr[b], bc1, bc2, gi, theta + i, m + i, v + i, stats);
    });
#pragma unroll
    for (int j = 0; j < 8; ++j)
        if (r[j] != 0) R[(long long)j * sc.G + g] = 0;
    K[g] = 0u;
}

__global__ void __launch_bounds__(256) k_fold_step_b(BatchArgs b) {
    long long blk = blockIdx.x;
    int si = last_le((const char*)&b.scenes[0].group_blk0, sizeof(BScene), b.n_scenes, blk);
    si = __builtin_amdgcn_readfirstlane(si);
    const BScene& S = b.scenes[si];
    long long g = (blk - S.group_blk0) * 256 + threadIdx.x;
    if (g >= S.sc.G) return;
    unsigned t = *b.step;
    if (t < 1u) t = 1u;                      // Adam steps count from 1
    int ti = (int)min(t, (unsigned)b.n_bc) - 1;
    fold_step_group(S.sc, g, S.R, S.sg, b.n_pairs, S.eps, S.lr, b.oc, b.bc1[ti], b.bc2[ti], (float*)S.theta,
                    S.m, S.v, S.Q, S.K, b.stats, b.q_zero);
}

// --------------------------------------------------------- launchers --

hipError_t launch_signs(hipStream_t st, unsigned long long seed, unsigned step, unsigned pair, unsigned scene,
                        long long d, uint32_t* bits) {
    const long long nblk = (d + 255) >> 8;
    hipLaunchKernelGGL(k_signs, dim3((unsigned)((nblk + 255) / 256)), dim3(256), 0, st, seed, step, pair, scene, d,
                       (int)((d + 31) / 32), bits);
    return hipGetLastError();
}

long long group_sign_blocks(const DScene& sc) {
    long long n = sign_chunks(sc.n_vg);
    for (int c = 0; c < sc.n_cls; ++c) n += sign_chunks((long long)sc.cls_w[c] * sc.cls_h[c]);
    return n;
}

hipError_t launch_group_signs(hipStream_t st, const DScene& sc, unsigned long long seed, unsigned step, unsigned pair0,
                              unsigned scene, int n_pairs, uint8_t* sg) {
    dim3 grid((unsigned)group_sign_blocks(sc), (unsigned)n_pairs);
    hipLaunchKernelGGL(k_group_signs, grid, dim3(256), 0, st, sc, seed, step, pair0, scene, sg);
    return hipGetLastError();
}

// Blocks that fill the chip several times over: from here on a setup block
// takes all views of its (pair, sign) (256 CUs of 4 to 8 blocks).  With fewer
// the views run side by side instead (a 320-triangle mesh in 8 views: one
// block per view).
#define SETUP_FULL_BLOCKS 4096

hipError_t launch_setup(hipStream_t st, SetupArgs a) {
    const unsigned tb = (unsigned)((a.sc.n_tris + SETUP_TB - 1) / SETUP_TB);
    unsigned y = (unsigned)(a.n_items * a.nsign);
    a.vpb = 1;
    if (a.whole && (long long)tb * (y / a.n_views) >= SETUP_FULL_BLOCKS) {
        a.vpb = a.n_views;
        y /= (unsigned)a.n_views;
    }
    hipLaunchKernelGGL(k_setup, dim3(tb, y), dim3(SETUP_TB), 0, st, a);
    return hipGetLastError();
}

// The shading that a scene's kernels are specialised for: its own when its
// textures have at most 2^24 texels each (their byte offsets are 24-bit
// products then), else the general kernels.
int scene_shade(const DScene& sc) {
    for (int t = 0; t < sc.n_tex; ++t)
        if ((long long)sc.tex_w[t] * sc.tex_h[t] > (1ll << 24)) return SHADE_ANY;
    return sc.shading;
}

hipError_t launch_tile(hipStream_t st, TileArgs a, int tile, int mode) {
    // the interleaved order needs the call's units in one grid dimension
    const long long units = (long long)(a.n_items / a.n_views) * a.views.tsum[a.n_views];
    const bool all = a.whole && (long long)a.n_items == (long long)a.views.n_pairs * a.n_views;
    a.interleave = all && units * 1024 < (1ll << 32);
    dim3 grid((unsigned)a.max_tiles, (unsigned)a.n_items);
    if (a.interleave) grid = dim3((unsigned)units);
    if (a.sc.layers > 0) {
        if (tile == 8) return launch_tile_deep_t<8>(st, a, mode, grid);
        if (tile == 16) return launch_tile_deep_t<16>(st, a, mode, grid);
        return hipErrorInvalidValue;                // deep buffers fit LDS for tiles <= 16
    }
    if (tile == 8) return launch_tile_t<8>(st, a, mode, grid);
    if (tile == 16) return launch_tile_t<16>(st, a, mode, grid);
    return launch_tile_t<32>(st, a, mode, grid);
}

hipError_t launch_subdiv(hipStream_t st, const DScene& sc, const DPert& pert, const float* theta, int n_pairs,
                         int nsign, float sgn0, float sgn1, float* fpos) {
    dim3 grid((unsigned)((sc.n_verts + 255) / 256), (unsigned)(n_pairs * nsign));
    hipLaunchKernelGGL(k_subdiv, grid, dim3(256), 0, st, sc, pert, theta, nsign, sgn0, sgn1, fpos);
    return hipGetLastError();
}

hipError_t launch_sum_tiles(hipStream_t st, const double* partials, int max_tiles, const DViews& views,
                            int n_views, double* out) {
    hipLaunchKernelGGL(k_sum_tiles, dim3((unsigned)n_views), dim3(256), 0, st, partials, max_tiles, views, out);
    return hipGetLastError();
}

hipError_t launch_check_tri(hipStream_t st, const int* tri, long long n, int n_verts, unsigned long long* bad) {
    dim3 grid((unsigned)((n + 255) / 256));
    hipLaunchKernelGGL(k_check_tri, grid, dim3(256), 0, st, tri, n, n_verts, bad);
    return hipGetLastError();
}

hipError_t launch_broadcast(hipStream_t st, const FoldArgs& a) {
    dim3 grid((unsigned)((a.sc.G + 255) / 256));
    hipLaunchKernelGGL(k_broadcast, grid, dim3(256), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_zero64(hipStream_t st, long long* p, int n) {
    hipLaunchKernelGGL(k_zero64, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, p, n);
    return hipGetLastError();
}

hipError_t launch_fold(hipStream_t st, const FoldArgs& a) {
    dim3 grid((unsigned)((a.sc.G + 255) / 256));
    hipLaunchKernelGGL(k_fold, grid, dim3(256), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_step(hipStream_t st, const StepArgs& a) {
    dim3 grid((unsigned)((a.sc.G + 255) / 256));
    hipLaunchKernelGGL(k_step, grid, dim3(256), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_batch_signs(hipStream_t st, const BatchArgs& b) {
    hipLaunchKernelGGL(k_signs_b, dim3((unsigned)b.sign_blocks), dim3(256), 0, st, b);
    return hipGetLastError();
}

hipError_t launch_batch_setup(hipStream_t st, const BatchArgs& b, long long blk0, long long nblk) {
    if (nblk <= 0) return hipSuccess;
    BatchArgs a = b;
    a.unit0 = blk0;
    hipLaunchKernelGGL(k_setup_b, dim3((unsigned)nblk), dim3(SETUP_TB), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_batch_tile(hipStream_t st, const BatchArgs& b, long long w0, long long n) {
    BatchArgs a = b;
    const long long most = 1ll << 21;               // a grid dimension holds 2^32 threads
    for (a.unit0 = w0; a.unit0 < w0 + n; a.unit0 += most) {
        const unsigned grid = (unsigned)(w0 + n - a.unit0 < most ? w0 + n - a.unit0 : most);
        hipError_t e = a.tile == 8 ? launch_batch_tile_t<8>(st, a, grid)
                     : a.tile == 16 ? launch_batch_tile_t<16>(st, a, grid) : launch_batch_tile_t<32>(st, a, grid);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_batch_fold(hipStream_t st, const BatchArgs& b) {
    hipLaunchKernelGGL(k_fold_b, dim3((unsigned)b.group_blocks), dim3(256), 0, st, b);
    return hipGetLastError();
}

hipError_t launch_batch_fold_step(hipStream_t st, const BatchArgs& b) {
    hipLaunchKernelGGL(k_fold_step_b, dim3((unsigned)b.group_blocks), dim3(256), 0, st, b);
    return hipGetLastError();
}

hipError_t launch_batch_step(hipStream_t st, const BatchArgs& b) {
    hipLaunchKernelGGL(k_step_b, dim3((unsigned)b.group_blocks), dim3(256), 0, st, b);
    return hipGetLastError();
}

hipError_t launch_batch_end(hipStream_t st, const BatchArgs& b) {
    hipLaunchKernelGGL(k_batch_end, dim3(1), dim3(1), 0, st, (unsigned*)b.step);
    return hipGetLastError();
}
