// dr_device.h -- device-side data layout and per-pixel arithmetic of the
// per-pixel stochastic gradient estimator (gfx950).
//
// Every floating-point expression is written with explicit parentheses
// and compiled with -ffp-contract=off, so each result is the correctly
// rounded fp32 value of the stated operation sequence; divisions and square
// roots are the correctly rounded ones.  This fixed operation order is what
// makes the triangle IDs, the loss differences and hence the fixed-point
// gradient sums reproducible bit for bit.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#define DRD_BG 0xFFFFFFFFu
#define DRD_MAX_TEX 3
#define DRD_MAX_LAYERS 4
#define DRD_MAX_VIEWS 16
#define DRD_PI 3.14159265f
#define DRD_INV_PI 0.318309886f

// Scene constants, passed by value to every kernel.
struct DScene {
    int n_verts, n_tris;
    const int* tri;             // [F,3]
    const float* cuv;           // [F,3,2]
    int n_tex;
    int tex_w[DRD_MAX_TEX], tex_h[DRD_MAX_TEX], tex_c[DRD_MAX_TEX];
    long long tex_off[DRD_MAX_TEX];      // first parameter of each texture
    int tex_cls[DRD_MAX_TEX];            // texel class of each texture
    int tex_bit[DRD_MAX_TEX];            // first sign bit of the texture in its class's group bytes
    int n_cls;
    int cls_w[DRD_MAX_TEX], cls_h[DRD_MAX_TEX];
    long long cls_goff[DRD_MAX_TEX];     // first group of each class
    int shading, tex_mode;
    int layers;                          // 0 opaque; 1..4 composited fragments
    // subdivision surface: n_ctrl > 0 control vertices are the position
    // parameters; tessellated vertex j = sum_k sub_w[k] ctrl[sub_cols[k]],
    // and tessellated triangle t credits the control vertices
    // tri_cols[tri_rowptr[t] .. tri_rowptr[t+1]) (the union of its corners')
    int n_vg;                            // position groups: n_ctrl, else n_verts
    int n_ctrl;
    const int* sub_rowptr;
    const int* sub_cols;
    const float* sub_w;
    const int* tri_rowptr;
    const int* tri_cols;
    float light[3], light_rgb[3], ambient, diffuse;
    long long d, G;
    long long sg_stride;                 // group sign bytes per pair (G and room to read on)
};

struct DView {
    int W, H;
    float M[16];
    float cam[3];
    float near_w;
    int tiles_x, tiles_y;
    long long tgt_off;                   // first float of this view's target
};

struct DViews {
    DView v[DRD_MAX_VIEWS];
    int n, n_pairs;                      // of the call
    int tsum[DRD_MAX_VIEWS + 1];         // tiles of the views before v
};

// Perturbation of one launch: per-block eps and the signs of the pairs, a
// byte per group: bit k is set where the group's k-th parameter has sign -1 (a
// vertex's x, y, z; a texel's channels in every texture of its class, in
// texture order: at most 8).  A texel's signs in all its textures thus come
// with one byte, those of two adjacent texels with one 16-bit read.
struct DPert {
    const uint8_t* sg;                   // [pairs, sg_stride] or null (no perturbation)
    float eps[1 + DRD_MAX_TEX];
};

// Raster half of a triangle record (48 B): snapped vertices in normalised
// (positive-area) order, flags, 1 / area and the depth plane.  The first
// 32 B hold all that the shading reads from it; the pixel box is recomputed
// from the corners where it is needed (tri_box).
struct __align__(16) TriR {
    int X[3], Y[3];
    unsigned flags;                      // bit0 valid, bit1+k top-left edge k, bit4 swapped
    float ia;                            // 1 / area2
    float z0, zx, zy;
    int pad;
};

// Shading half (16 B): 1/w in normalised order and, for Lambert shading, the
// face's shade (ambient + diffuse n.l), which is the same for all its pixels.
struct __align__(16) TriS {
    float iw[3];
    float sh;
};

// GGX shading: what a face's pixels share in every view of one perturbation
// (64 B): the perturbed world positions in the original corner order, the
// unit face normal and the unit tangent of the face's UV map.  Formed once
// per triangle and perturbation by the setup instead of once per pixel (two
// of a pixel's five normalisations), and kept once for all views, so the
// setup writes less than with positions in every view's record (paper step:
// 236 MB against 283 MB).
struct __align__(16) TriG {
    float p[9];
    float nf[3];
    float T[3];
    float pad;
};

static_assert(sizeof(TriR) == 48, "TriR layout");
static_assert(sizeof(TriS) == 16, "TriS layout");
static_assert(sizeof(TriG) == 64, "TriG layout");

#define TRI_VALID 1u
#define TRI_SWAPPED 16u
#define TRI_SMALL 32u          // bbox spans < 32000 subpixels: 32-bit edge functions are exact

// ---------------------------------------------------------------- signs --

__device__ __forceinline__ void philox4x64_10(unsigned long long c0, unsigned long long c1,
                                              unsigned long long c2, unsigned long long c3,
                                              unsigned long long k0, unsigned long long k1,
                                              unsigned long long out[4]) {
    const unsigned long long M0 = 0xD2E7470EE14C6C93ull, M1 = 0xCA5A826395121157ull;
    const unsigned long long W0 = 0x9E3779B97F4A7C15ull, W1 = 0xBB67AE8584CAA73Bull;
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        if (r > 0) { k0 += W0; k1 += W1; }
        unsigned long long hi0 = __umul64hi(M0, c0), lo0 = M0 * c0;
        unsigned long long hi1 = __umul64hi(M1, c2), lo1 = M1 * c2;
        unsigned long long n0 = hi1 ^ c1 ^ k0, n2 = hi0 ^ c3 ^ k1;
        c0 = n0; c1 = lo1; c2 = n2; c3 = lo0;
    }
    out[0] = c0; out[1] = c1; out[2] = c2; out[3] = c3;
}

// x perturbed by sgn * s * e (one fp32 add or subtract), s = -1 where `neg`.
__device__ __forceinline__ float perturbed(float x, float e, bool neg, float sgn) {
    float se = neg ? -e : e;
    return (sgn > 0.0f) ? (x + se) : (x - se);
}

// The perturbed coordinates of (control) vertex v.
__device__ __forceinline__ void perturbed_vertex(const float* __restrict__ th, long long v, float e,
                                                 const uint8_t* __restrict__ sg, float sgn, float* p) {
#pragma unroll
    for (int c = 0; c < 3; ++c) p[c] = th[3 * v + c];
    if (sg == nullptr || e == 0.0f) return;
    const unsigned b = sg[v];
#pragma unroll
    for (int c = 0; c < 3; ++c) p[c] = perturbed(p[c], e, (b >> c) & 1u, sgn);
}

// ------------------------------------------------------------ geometry --

struct Vtx {
    int valid;
    int X, Y;
    float z, iw;
};

__device__ __forceinline__ Vtx xform(const DView& v, float x, float y, float z) {
    const float* M = v.M;
    float cx = ((M[0] * x + M[1] * y) + M[2] * z) + M[3];
    float cy = ((M[4] * x + M[5] * y) + M[6] * z) + M[7];
    float cz = ((M[8] * x + M[9] * y) + M[10] * z) + M[11];
    float cw = ((M[12] * x + M[13] * y) + M[14] * z) + M[15];
    Vtx o;
    o.valid = 0; o.X = 0; o.Y = 0; o.z = 0.0f; o.iw = 0.0f;
    if (!(cw >= v.near_w)) return o;
    float nx = cx / cw, ny = cy / cw, nz = cz / cw;
    float sx = (nx * 0.5f + 0.5f) * (float)v.W;
    float sy = (0.5f - ny * 0.5f) * (float)v.H;
    float fx = sx * 256.0f, fy = sy * 256.0f;
    if (!(fabsf(fx) <= 4194304.0f) || !(fabsf(fy) <= 4194304.0f)) return o;
    o.valid = 1;
    o.X = (int)rintf(fx);
    o.Y = (int)rintf(fy);
    o.z = nz * 0.5f + 0.5f;
    o.iw = 1.0f / cw;
    return o;
}

// Edge k of a normalised triangle runs from vertex k+1 to vertex k+2.
__device__ __forceinline__ long long edge_at(int xa, int ya, int xb, int yb, int px, int py) {
    return (long long)(xb - xa) * (long long)(py - ya) - (long long)(yb - ya) * (long long)(px - xa);
}

__device__ __forceinline__ bool inside(const TriR& r, int px, int py, long long& e0, long long& e1,
                                       long long& e2) {
    e0 = edge_at(r.X[1], r.Y[1], r.X[2], r.Y[2], px, py);
    e1 = edge_at(r.X[2], r.Y[2], r.X[0], r.Y[0], px, py);
    e2 = edge_at(r.X[0], r.Y[0], r.X[1], r.Y[1], px, py);
    bool ok0 = (e0 > 0) || (e0 == 0 && (r.flags & 2u));
    bool ok1 = (e1 > 0) || (e1 == 0 && (r.flags & 4u));
    bool ok2 = (e2 > 0) || (e2 == 0 && (r.flags & 8u));
    return ok0 && ok1 && ok2;
}

// Pixel box of a triangle clipped to [px0, cx1] x [py0, cy1] (px0, py0 >= 0):
// the pixels whose centre 256 x + 128 lies within the snapped corners'
// bounds.  Empty when x0 > x1 or y0 > y1.
__device__ __forceinline__ void tri_box(const TriR& r, int px0, int py0, int cx1, int cy1, int& x0, int& x1,
                                        int& y0, int& y1) {
    int xmin = min(r.X[0], min(r.X[1], r.X[2])), xmax = max(r.X[0], max(r.X[1], r.X[2]));
    int ymin = min(r.Y[0], min(r.Y[1], r.Y[2])), ymax = max(r.Y[0], max(r.Y[1], r.Y[2]));
    x0 = max((xmin + 127) >> 8, px0);
    x1 = min((xmax - 128) >> 8, cx1);
    y0 = max((ymin + 127) >> 8, py0);
    y1 = min((ymax - 128) >> 8, cy1);
}

__device__ __forceinline__ float depth_at(const TriR& r, int px, int py) {
    float z = (r.z0 + r.zx * (float)(px - r.X[0])) + r.zy * (float)(py - r.Y[0]);
    if (!(z > 0.0f)) z = 0.0f;
    return z;
}

// ------------------------------------------------------------- sampling --

struct Foot {
    int xa, xb, ya, yb;
    float fx, fy;
};

__device__ __forceinline__ Foot footprint(float u, float v, int W, int H) {
    Foot f;
    float x = u * (float)W - 0.5f;
    float y = v * (float)H - 0.5f;
    if (!(fabsf(x) < 16777216.0f)) x = 0.0f;
    if (!(fabsf(y) < 16777216.0f)) y = 0.0f;
    float x0f = floorf(x), y0f = floorf(y);
    f.fx = x - x0f;
    f.fy = y - y0f;
    const int x0 = (int)x0f, y0 = (int)y0f;
    // x0 mod W (non-negative).  Of x0, x0 - W and x0 + W as unsigned numbers
    // the least lies in [0, W) when x0 is within a period of it; UVs further
    // out take the division.
    unsigned xa = min((unsigned)x0, min((unsigned)x0 - (unsigned)W, (unsigned)x0 + (unsigned)W));
    if (xa >= (unsigned)W) {
        int m = x0 % W;
        xa = (unsigned)(m < 0 ? m + W : m);
    }
    f.xa = (int)xa;
    f.xb = (f.xa + 1 == W) ? 0 : f.xa + 1;
    f.ya = max(0, min(y0, H - 1));
    f.yb = max(0, min(y0 + 1, H - 1));
    return f;
}

// Global-memory views of device pointers (address space 1).  Loads and
// atomics through them compile to global_* instructions instead of flat_*
// ones, so the compiler can wait on each request by itself instead of on
// all outstanding memory and LDS traffic together.
#define DRD_GLOBAL __attribute__((address_space(1)))

template <class T>
__device__ __forceinline__ T gload(const T* p) {
#if defined(__HIP_DEVICE_COMPILE__)
    return *(const DRD_GLOBAL T*)p;
#else
    return *p;             // host pass: parsed, never run
#endif
}

// A footprint: its first texel (row ya, column xa) and its last (yb, xb),
// column in the low half, row in the high one (texture sides are at most 2^15,
// so all ones matches no texel).  Nearest mode: both the nearest texel.
struct FootBox {
    unsigned a, b;
};

__device__ __forceinline__ FootBox foot_corners(const DScene& sc, const Foot& f) {
    int xa = f.xa, xb = f.xb, ya = f.ya, yb = f.yb;
    if (sc.tex_mode == 1) {
        xa = xb = (f.fx >= 0.5f) ? f.xb : f.xa;
        ya = yb = (f.fy >= 0.5f) ? f.yb : f.ya;
    }
    return {(unsigned)xa | ((unsigned)ya << 16), (unsigned)xb | ((unsigned)yb << 16)};
}

__device__ __forceinline__ FootBox foot_box(const DScene& sc, int c, float u, float v) {
    return foot_corners(sc, footprint(u, v, sc.cls_w[c], sc.cls_h[c]));
}

// Signs of a footprint's four texels: sg is the class's first group byte.
// w[row] holds the row's two bytes in its upper half, complemented (flip) for
// the minus render.  The two texels of a row are adjacent unless the row
// wraps.
struct FootSigns {
    unsigned w[2];
};

__device__ __forceinline__ FootSigns foot_signs(const DRD_GLOBAL uint8_t* sg, int W, unsigned flip, const Foot& f) {
    typedef uint16_t __attribute__((aligned(1))) u16a1;
    FootSigns s;
#pragma unroll
    for (int row = 0; row < 2; ++row) {
        const unsigned o = __umul24((unsigned)(row ? f.yb : f.ya), (unsigned)W) + (unsigned)f.xa;      // < 2^30
        unsigned w = *(const DRD_GLOBAL u16a1*)(sg + o);
        if (f.xb != f.xa + 1) w = (w & 0xFFu) | ((unsigned)sg[o - (unsigned)f.xa + (unsigned)f.xb] << 8);
        s.w[row] = (w << 16) ^ flip;
    }
    return s;
}

// Bilinear sample of texture t (C channels) of the perturbed scene
// (theta + sgn s eps) over a precomputed footprint and its signs (null
// perturbation: pert false).  The perturbed value is x + (s_i ? -es : es) with
// es = +-eps by the render's sign: x - y and x + (-y) are the same IEEE
// operation, so this equals perturbed()'s result.  The weighted sum keeps its
// order ((w00 t00 + w10 t10) + w01 t01) + w11 t11.
//
// COMPACT: the texture has at most 2^24 texels, so a texel's byte offset is
// one 24-bit product and fits in 32 bits; the loads then take the texture's
// uniform base and a 32-bit offset instead of a 64-bit address per lane.
template <int C, bool COMPACT>
__device__ __forceinline__ void sample_tex(const DScene& sc, const float* __restrict__ th, bool pert, float e, int t,
                                           const Foot& f, const FootSigns& sig, float* out) {
    typedef float __attribute__((ext_vector_type(C == 1 ? 2 : C), aligned(4))) texel_t;
    const DRD_GLOBAL float* tt = (const DRD_GLOBAL float*)th + sc.tex_off[t];
    const unsigned eb = __float_as_uint(e);
    const float wx[2] = {1.0f - f.fx, f.fx};
    const bool adj = f.xb == f.xa + 1;
    float acc[C];
#pragma unroll
    for (int row = 0; row < 2; ++row) {
        const float wy = row ? f.fy : 1.0f - f.fy;
        // texel indices within the texture: W, H <= 32768 keep them below 2^30
        unsigned o[2];
        const unsigned ro = __umul24((unsigned)(row ? f.yb : f.ya), (unsigned)sc.tex_w[t]);
        o[0] = (ro + (unsigned)f.xa) * C;
        o[1] = (ro + (unsigned)f.xb) * C;
        float x[2][C];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const DRD_GLOBAL float* a;
            if constexpr (COMPACT) {
                a = (const DRD_GLOBAL float*)((const DRD_GLOBAL char*)tt + (o[k] << 2));
            } else {
                a = tt + (unsigned long long)o[k];
            }
            if constexpr (C == 1) {
                // the row's two single-channel texels are adjacent: one 8 B read
                if (k == 0 && adj) {
                    texel_t v = *(const DRD_GLOBAL texel_t*)a;
                    x[0][0] = v.x;
                    x[1][0] = v.y;
                } else if (k == 0 || !adj) {
                    x[k][0] = a[0];
                }
            } else {
                texel_t v = *(const DRD_GLOBAL texel_t*)a;
#pragma unroll
                for (int c = 0; c < C; ++c) x[k][c] = v[c];
            }
        }
        if (pert) {
            // the sign of texel k's channel c is bit 16 + 8 k + c of w: moved
            // to the top, it is the sign bit of the offset
            const unsigned w = sig.w[row] >> sc.tex_bit[t];
#pragma unroll
            for (int k = 0; k < 2; ++k)
#pragma unroll
                for (int c = 0; c < C; ++c)
                    x[k][c] = x[k][c] + __uint_as_float(((w << (15 - 8 * k - c)) & 0x80000000u) | eb);
        }
#pragma unroll
        for (int c = 0; c < C; ++c) {
            float t0 = (wx[0] * wy) * x[0][c], t1 = (wx[1] * wy) * x[1][c];
            acc[c] = row ? ((acc[c] + t0) + t1) : (t0 + t1);
        }
    }
#pragma unroll
    for (int c = 0; c < C; ++c) out[c] = acc[c];
}

// Correctly rounded square root and reciprocal for operands in a normal
// range, in fewer instructions than the general sequences.
// sqrt_rn: for x in [2^-96, 2^126] the hardware square root (within 1 ulp)
// corrected by the residuals of its two neighbours -- the correction the
// compiler's sqrtf applies, without its scaling of tiny inputs and its
// handling of 0, inf and NaN.  rcp_rn: for |y| in [2^-125, 2^125] the
// hardware reciprocal refined by one Newton step with fused multiply-adds.
// Both are checked against sqrtf and 1.0f / y for every operand of those
// ranges (dr_probe_math); operands outside them take sqrtf and division.
#define DRD_SQRT_LO 0x0F800000u        // 2^-96
#define DRD_SQRT_HI 0x7E800000u        // 2^126
#define DRD_RCP_LO 0x01000000u         // 2^-125
#define DRD_RCP_HI 0x7E000000u         // 2^125

__device__ __forceinline__ float sqrt_rn_fast(float x) {
    float s = __builtin_amdgcn_sqrtf(x);
    float sm = __uint_as_float(__float_as_uint(s) - 1u), sp = __uint_as_float(__float_as_uint(s) + 1u);
    float rm = __builtin_fmaf(-sm, s, x), rp = __builtin_fmaf(-sp, s, x);
    s = (rm <= 0.0f) ? sm : s;
    return (rp > 0.0f) ? sp : s;
}

__device__ __forceinline__ float rcp_rn_fast(float y) {
    float r = __builtin_amdgcn_rcpf(y);
    float e = __builtin_fmaf(-y, r, 1.0f);
    return __builtin_fmaf(e, r, r);
}

__device__ __forceinline__ bool sqrt_fast_ok(float x) {
    unsigned b = __float_as_uint(x);
    return b >= DRD_SQRT_LO && b <= DRD_SQRT_HI;            // positive, in range
}

__device__ __forceinline__ bool rcp_fast_ok(float y) {
    unsigned b = __float_as_uint(y) & 0x7FFFFFFFu;
    return b >= DRD_RCP_LO && b <= DRD_RCP_HI;
}

// sqrtf(x), correctly rounded
__device__ __forceinline__ float sqrt_rn(float x) { return sqrt_fast_ok(x) ? sqrt_rn_fast(x) : sqrtf(x); }

// 1.0f / y, correctly rounded
__device__ __forceinline__ float rcp_rn(float y) { return rcp_fast_ok(y) ? rcp_rn_fast(y) : 1.0f / y; }

// x / |x| (0 for 0): 1 / sqrt(l2) with each operation correctly rounded.  One
// range test serves both short sequences: the root of an operand in
// [2^-96, 2^126] lies in [2^-48, 2^63], within the reciprocal's range.
__device__ __forceinline__ void nrm3(float* x) {
    const float l2 = (x[0] * x[0] + x[1] * x[1]) + x[2] * x[2];
    float inv;
    if (sqrt_fast_ok(l2)) {
        inv = rcp_rn_fast(sqrt_rn_fast(l2));
    } else if (l2 > 0.0f) {
        inv = 1.0f / sqrtf(l2);
    } else {
        x[0] = 0.0f; x[1] = 0.0f; x[2] = 0.0f;
        return;
    }
    x[0] = x[0] * inv; x[1] = x[1] * inv; x[2] = x[2] * inv;
}

__device__ __forceinline__ float dot3(const float* a, const float* b) {
    return (a[0] * b[0] + a[1] * b[1]) + a[2] * b[2];
}

__device__ __forceinline__ void cross3(const float* a, const float* b, float* o) {
    o[0] = a[1] * b[2] - a[2] * b[1];
    o[1] = a[2] * b[0] - a[0] * b[2];
    o[2] = a[0] * b[1] - a[1] * b[0];
}

// A triangle's corner UVs (original corner order).
struct CornerUV {
    float c[6];
};

__device__ __forceinline__ CornerUV load_cuv(const DScene& sc, unsigned t) {
    return gload((const CornerUV*)(sc.cuv + 6 * (long long)t));
}

// Unit face normal of a triangle with perturbed corners p (original order).
__device__ __forceinline__ void face_normal(const float* p, float* nf) {
    float e1v[3], e2v[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) { e1v[c] = p[3 + c] - p[c]; e2v[c] = p[6 + c] - p[c]; }
    cross3(e1v, e2v, nf);
    nrm3(nf);
}

// Unit tangent of the face's UV map (the bitangent is nf x T).
__device__ __forceinline__ void face_tangent(const float* p, const float* cuv, const float* nf, float* T) {
    float e1v[3], e2v[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) { e1v[c] = p[3 + c] - p[c]; e2v[c] = p[6 + c] - p[c]; }
    float du1 = cuv[2] - cuv[0], dv1 = cuv[3] - cuv[1], du2 = cuv[4] - cuv[0], dv2 = cuv[5] - cuv[1];
    float rr = du1 * dv2 - du2 * dv1;
#pragma unroll
    for (int c = 0; c < 3; ++c) T[c] = e1v[c] * dv2 - e2v[c] * dv1;
    if (rr < 0.0f) { T[0] = -T[0]; T[1] = -T[1]; T[2] = -T[2]; }
    float nt = dot3(nf, T);
#pragma unroll
    for (int c = 0; c < 3; ++c) T[c] = T[c] - nf[c] * nt;
    nrm3(T);
}

// Perspective-correct attributes of pixel (px,py) on triangle t: the
// 1/w-weighted barycentrics, the reciprocal of their sum and the UV.
struct Attr {
    float pc0, pc1, pc2, iS, u, v;
};

__device__ __forceinline__ Attr frag_attr(const DScene& sc, const TriR& r, const TriS& s, const CornerUV& cu, int px,
                                          int py) {
    // edge functions as floats; for a TRI_SMALL triangle they fit in 32 bits
    // and convert in one instruction, to the same values
    float f0, f1, f2;
    if (r.flags & TRI_SMALL) {
        int e0 = __mul24(r.X[2] - r.X[1], py - r.Y[1]) - __mul24(r.Y[2] - r.Y[1], px - r.X[1]);
        int e1 = __mul24(r.X[0] - r.X[2], py - r.Y[2]) - __mul24(r.Y[0] - r.Y[2], px - r.X[2]);
        int e2 = __mul24(r.X[1] - r.X[0], py - r.Y[0]) - __mul24(r.Y[1] - r.Y[0], px - r.X[0]);
        f0 = (float)e0; f1 = (float)e1; f2 = (float)e2;
    } else {
        long long e0, e1, e2;
        (void)inside(r, px, py, e0, e1, e2);
        f0 = (float)e0; f1 = (float)e1; f2 = (float)e2;
    }
    float b0 = f0 * r.ia, b1 = f1 * r.ia, b2 = f2 * r.ia;
    float pc0 = b0 * s.iw[0], pc1 = b1 * s.iw[1], pc2 = b2 * s.iw[2];
    float S = (pc0 + pc1) + pc2;
    float iS = rcp_rn(S);
    bool sw = (r.flags & TRI_SWAPPED) != 0u;
    const float* cuv = cu.c;
    float cu0 = cuv[0], cv0 = cuv[1], cu1 = cuv[2], cv1 = cuv[3], cu2 = cuv[4], cv2 = cuv[5];
    float un1 = sw ? cu2 : cu1, vn1 = sw ? cv2 : cv1, un2 = sw ? cu1 : cu2, vn2 = sw ? cv1 : cv2;
    Attr a;
    a.pc0 = pc0; a.pc1 = pc1; a.pc2 = pc2; a.iS = iS;
    a.u = ((pc0 * cu0 + pc1 * un1) + pc2 * un2) * iS;
    a.v = ((pc0 * cv0 + pc1 * vn1) + pc2 * vn2) * iS;
    return a;
}

// Colour, opacity and UV of pixel (px,py) (subpixel sample coordinates)
// covered by triangle t: perspective-correct attributes, then unlit /
// Lambert / GGX.  opacity: the albedo's fourth channel clamped to [0, 1]
// (DEEP only).
//
// SHADE is the scene's shading, fixed at compile time, for scenes whose
// textures are compact (sample_texels); SHADE_ANY reads the shading from the
// scene and takes textures of any size.  DEEP: the albedo has four channels.
// G: the face's GGX record (read for GGX only).
// fb: the footprint of texel class 0 (foot_box's value).
#define SHADE_ANY 3

template <int SHADE, bool DEEP>
__device__ __forceinline__ void shade_pixel(const DScene& sc, const DView& vw, const float* __restrict__ th,
                                            const uint8_t* __restrict__ sg, const float* eps, unsigned flip,
                                            const TriR& r, const TriS& s, const TriG* __restrict__ G,
                                            const CornerUV& cu, int px, int py, float* rgb, float* uvo,
                                            FootBox& fb, float& opacity) {
    constexpr bool COMPACT = SHADE != SHADE_ANY;
    const int shading = SHADE != SHADE_ANY ? SHADE : sc.shading;
    Attr a = frag_attr(sc, r, s, cu, px, py);
    float pc0 = a.pc0, pc1 = a.pc1, pc2 = a.pc2, iS = a.iS, u = a.u, v = a.v;
    bool sw = (r.flags & TRI_SWAPPED) != 0u;
    uvo[0] = u;
    uvo[1] = v;
    float alb[4] = {0.0f, 0.0f, 0.0f, 1.0f};
    // footprint and signs of texel class 0; a texture of another class has its own
    const bool pert = sg != nullptr;
    const DRD_GLOBAL uint8_t* gsg = (const DRD_GLOBAL uint8_t*)sg;
    Foot foot0;
    FootSigns sig0 = {{0u, 0u}};
    if (sc.n_tex > 0) {
        foot0 = footprint(u, v, sc.cls_w[0], sc.cls_h[0]);
        fb = foot_corners(sc, foot0);
        if (pert) sig0 = foot_signs(gsg + sc.cls_goff[0], sc.cls_w[0], flip, foot0);
        sample_tex<DEEP ? 4 : 3, COMPACT>(sc, th, pert && eps[1] != 0.0f, eps[1], 0, foot0, sig0, alb);
    }
    if constexpr (DEEP) {
        float al = alb[3];
        if (!(al > 0.0f)) al = 0.0f;
        if (al > 1.0f) al = 1.0f;
        opacity = al;
    }
    if (shading == 0) {
        rgb[0] = alb[0]; rgb[1] = alb[1]; rgb[2] = alb[2];
        return;
    }
    if (shading == 1) {
#pragma unroll
        for (int c = 0; c < 3; ++c) rgb[c] = alb[c] * (s.sh * sc.light_rgb[c]);
        return;
    }
    // GGX with a tangent-space normal map in the face's UV frame
    float nm[4] = {0.5f, 0.5f, 1.0f, 0.0f};
    if (sc.n_tex > 1) {
        const int c1 = sc.tex_cls[1];
        Foot f1 = foot0;
        FootSigns s1 = sig0;
        if (c1 != 0) {
            f1 = footprint(u, v, sc.cls_w[c1], sc.cls_h[c1]);
            if (pert) s1 = foot_signs(gsg + sc.cls_goff[c1], sc.cls_w[c1], flip, f1);
        }
        sample_tex<3, COMPACT>(sc, th, pert && eps[2] != 0.0f, eps[2], 1, f1, s1, nm);
    }
    float tn[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) tn[c] = 2.0f * nm[c] - 1.0f;
    const TriG g = gload(G);
    float n[3], B[3];
    cross3(g.nf, g.T, B);
#pragma unroll
    for (int c = 0; c < 3; ++c) n[c] = (g.T[c] * tn[0] + B[c] * tn[1]) + g.nf[c] * tn[2];
    nrm3(n);
    float rough4[4] = {0.5f, 0.0f, 0.0f, 0.0f};
    if (sc.n_tex > 2) {
        const int c2 = sc.tex_cls[2];
        Foot f2 = foot0;
        FootSigns s2 = sig0;
        if (c2 != 0) {
            f2 = footprint(u, v, sc.cls_w[c2], sc.cls_h[c2]);
            if (pert) s2 = foot_signs(gsg + sc.cls_goff[c2], sc.cls_w[c2], flip, f2);
        }
        sample_tex<1, COMPACT>(sc, th, pert && eps[3] != 0.0f, eps[3], 2, f2, s2, rough4);
    }
    float P[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        float q0 = g.p[c], q1 = sw ? g.p[6 + c] : g.p[3 + c], q2 = sw ? g.p[3 + c] : g.p[6 + c];
        P[c] = ((pc0 * q0 + pc1 * q1) + pc2 * q2) * iS;
    }
    float V[3] = {vw.cam[0] - P[0], vw.cam[1] - P[1], vw.cam[2] - P[2]};
    nrm3(V);
    const float* L = sc.light;
    float Hh[3] = {L[0] + V[0], L[1] + V[1], L[2] + V[2]};
    nrm3(Hh);
    float ndl = dot3(n, L), ndv = dot3(n, V), ndh = dot3(n, Hh), vdh = dot3(V, Hh);
    if (!(ndl > 0.0f)) ndl = 0.0f;
    if (!(ndv > 0.0f)) ndv = 0.0f;
    if (!(ndh > 0.0f)) ndh = 0.0f;
    if (!(vdh > 0.0f)) vdh = 0.0f;
    float alpha = rough4[0] * rough4[0];
    if (!(alpha > 0.002f)) alpha = 0.002f;
    float a2 = alpha * alpha;
    // D G F / (4 n.l n.v) with D = a2 / (pi dd^2) and Smith-Schlick
    // G = n.l / gl * n.v / gv: n.l n.v cancel, leaving one division
    float dd = (ndh * ndh) * (a2 - 1.0f) + 1.0f;
    float k = alpha * 0.5f;
    float gl = ndl * (1.0f - k) + k;
    float gv = ndv * (1.0f - k) + k;
    float om = 1.0f - vdh;
    float om5 = ((om * om) * (om * om)) * om;
    float F = 0.04f + 0.96f * om5;
    float spec = 0.0f;
    if (ndl > 0.0f && ndv > 0.0f) spec = (a2 * F) / ((((4.0f * DRD_PI) * dd) * dd) * (gl * gv));
#pragma unroll
    for (int c = 0; c < 3; ++c)
        rgb[c] = ((alb[c] * DRD_INV_PI + spec) * sc.light_rgb[c]) * ndl + sc.ambient * alb[c];
}

// Fixed-point code of a loss difference: round-half-even(delta * 2^32),
// clamped to +-2^37; NaN gives 0.  flag: 1 saturated, 2 NaN.
__device__ __forceinline__ long long quantize(float delta, int& flag) {
    flag = 0;
    if (delta != delta) { flag = 2; return 0; }
    if (fabsf(delta) > 32.0f) {
        flag = 1;
        return delta > 0.0f ? (1ll << 37) : -(1ll << 37);
    }
    return (long long)rintf(delta * 4294967296.0f);
}

// The per-pixel difference that Eq. 8 scatters, from the colours of the two
// renders.  Loss form (img == 0): f+ - f- with f the L2 error against the
// target t (Table 1).  Image form (img != 0): t is the gradient g of a
// downstream loss with respect to the pixel's colour and the difference is
// <g, I+ - I->, the first-order change of that loss, so that the estimator
// approximates the vector-Jacobian product of the render.
__device__ __forceinline__ float pixel_delta(const float* p, const float* m, const float* t, int img) {
    float t0 = t[0], t1 = t[1], t2 = t[2];
    if (img) {
        float d0 = p[0] - m[0], d1 = p[1] - m[1], d2 = p[2] - m[2];
        return (t0 * d0 + t1 * d1) + t2 * d2;
    }
    float dr0 = p[0] - t0, dg0 = p[1] - t1, db0 = p[2] - t2;
    float dr1 = m[0] - t0, dg1 = m[1] - t1, db1 = m[2] - t2;
    float fp = (dr0 * dr0 + dg0 * dg0) + db0 * db0;
    float fm = (dr1 * dr1 + dg1 * dg1) + db1 * db1;
    return fp - fm;
}
