// a7 on gfx950: joint bilateral upsampling of the disparity (Eq. 2), with an
// optional fused triangulation of every output pixel (Eq. 3).
//
// A 256-thread block owns 16 x 16 full-resolution pixels (16 x 32 with two rows
// per thread).  The low-resolution
// taps every pixel of the block can reach are staged once in LDS, one 16-byte
// record each: the guide sample I_q at scale*q + scale/2 as FP16 channel pairs
// (exact for 8-bit values), -|I_q|^2 and the tap's disparity as floats.  The
// weight of a tap is exp2 of a non-positive exponent, spatial + range: the
// spatial part is separable and depends only on the pixel's sub-pixel phase,
// so a per-block LDS table holds, for each of the block's 16 columns, the
// 2R+1 x exponents (each thread copies its column's row into registers) and,
// for each of its 16 rows, the 2R+1 exp2 factors of the y part, applied once
// per window row to that row's sums; the range part is
// -|I_p - I_q|^2 scaled by log2(e) / (2 sigma_r^2).  The squared distance is
// formed exactly by FP16 dot products accumulating in FP32 (every term is an
// integer below 2^24): 2 I_p.I_q - |I_q|^2 - 256 floor(|I_p|^2 / 256), the
// remaining low byte of |I_p|^2 entering through the x table.  Weights are
// taken relative to exponent 0; a pixel whose weights sum below 2^-60 (a guide
// colour far from every tap in its window) is evaluated again relative to its
// largest exponent, so no pixel loses its weights to underflow.
// ALU/transcendental bound: per output pixel and tap one or two dot products,
// one exp2 and three other vector operations.
#include <hip/hip_runtime.h>

#include "bp_internal.h"

namespace bpk {

constexpr int kTile = 16;
constexpr int kMaxTap = kTile + 1 + 2 * 8;   // low-res tile width for scale >= 1, R <= 8

template <int C>
__device__ __forceinline__ uint32_t guide_px(const uint8_t *__restrict__ g, int64_t stride, int x, int y)
{
    const uint8_t *p = g + (int64_t)y * stride + (int64_t)x * C;
    if constexpr (C == 1) return p[0];
    else return (uint32_t)p[0] | ((uint32_t)p[1] << 8) | ((uint32_t)p[2] << 16);
}

// Eq. 3 epilogue: the camera-frame point of a full-resolution pixel (u, v)
// with disparity d = s * D_p pixels is (B / d) [u - u0, (v - v0) dv / du, f / du]
// (the last entry from Eq. 3's projection, d = f B / (z du)); NaN where d <= 0.
struct PointArgs {
    float *xyz;                 // [hh][wh][3], or NULL
    float baseline, f_du, dv_du, u0, v0;
};

typedef _Float16 h2_t __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t h2_bits(float a, float b)
{
    const h2_t v = {(_Float16)a, (_Float16)b};
    return __builtin_bit_cast(uint32_t, v);
}

__device__ __forceinline__ h2_t bits_h2(uint32_t u) { return __builtin_bit_cast(h2_t, u); }

// floor(a / b) for 0 <= a < 2^20 and b >= 1 from a reciprocal rb of b within
// one ulp: (a + 0.5) / b lies at least 0.5 / b, four ulps of the quotient,
// from an integer, beyond the error of the product.
__device__ __forceinline__ int div_small(int a, float rb) { return (int)(((float)a + 0.5f) * rb); }

template <int R, int C, bool PTS, int NY>
__global__ void __launch_bounds__(256) k_jbu(const int32_t *__restrict__ disp, int wl, int hl,
                                            const uint8_t *__restrict__ guide, int wh, int hh, int64_t stride,
                                            int s, float rs, float ksp, float krg, float *__restrict__ out,
                                            PointArgs pa)
{
    // Per tap: FP16 (I_R, I_G), (I_B, 256) (grey: (I, 256), unused),
    // -|I_q|^2 and the disparity.  Outside the grid -|I_q|^2 is -inf, which
    // gives the tap zero weight.
    __shared__ uint4 t_q[kMaxTap * kMaxTap];
    constexpr int NT = 2 * R + 1;
    // Separable spatial terms of the block's 16 columns and 16 rows, per
    // window column / row: the x exponent, and exp2 of the y exponent.
    constexpr int ROWS = kTile * NY;
    __shared__ float t_sx[kTile * NT], t_wy[ROWS * NT];
    const int bx0 = blockIdx.x * kTile, by0 = blockIdx.y * ROWS;
    const int qx0 = bx0 / s - R, qy0 = by0 / s - R;
    const int tw = (bx0 + kTile - 1) / s - bx0 / s + 1 + 2 * R;
    const int th = (by0 + ROWS - 1) / s - by0 / s + 1 + 2 * R;
    const float rtw = __builtin_amdgcn_rcpf((float)tw);
    for (int i = threadIdx.x; i < tw * th; i += 256) {
        const int ty = div_small(i, rtw), tx = i - ty * tw;
        const int qx = qx0 + tx, qy = qy0 + ty;
        uint4 r = make_uint4(0u, 0u, __float_as_uint(-__builtin_huge_valf()), 0u);
        if (qx >= 0 && qx < wl && qy >= 0 && qy < hl) {
            const uint32_t g = guide_px<C>(guide, stride, s * qx + s / 2, s * qy + s / 2);
            const int n = (int)__builtin_amdgcn_udot4(g, g, 0u, false);
            if constexpr (C == 3) {
                r.x = h2_bits((float)(g & 255u), (float)((g >> 8) & 255u));
                r.y = h2_bits((float)(g >> 16), 256.0f);
            } else {
                r.x = h2_bits((float)g, 256.0f);
            }
            r.z = __float_as_uint(-(float)n);
            r.w = __float_as_uint((float)disp[(int64_t)qy * wl + qx]);
        }
        t_q[ty * kMaxTap + tx] = r;
    }
    // s * (p_lo - q) = phase + 0.5 - s/2 - s*dq for window offset dq = i - R.
    for (int i = threadIdx.x; i < (kTile + ROWS) * NT; i += 256) {
        const int y = i >= kTile * NT, e = i - y * (kTile * NT), c = e / NT, k = e - c * NT;
        const int p = (y ? by0 : bx0) + c;
        const float t = (float)(p - s * div_small(p, rs)) + 0.5f - 0.5f * (float)s - (float)(s * (k - R));
        const float v = -(t * t * ksp);
        if (y) t_wy[e] = __builtin_amdgcn_exp2f(v);
        else t_sx[e] = v;
    }
    __syncthreads();
    const int col = (int)(threadIdx.x % kTile), rowi = (int)(threadIdx.x / kTile) * NY;
    const int px = bx0 + col, py0 = by0 + rowi;
    if (px >= wh || py0 >= hh) return;                  // hh is a multiple of s, so of NY
    const int cx = div_small(px, rs), cy = div_small(py0, rs);
    const int ox = cx - R - qx0, oy = cy - R - qy0;     // tile coordinates of the window corner
    // Pixel side of the dot products: 2 I_p (exact in FP16 up to 510) and
    // -floor(|I_p|^2 / 256) (at most 762) against the tap's 256; and the x term
    // of the exponent: spatial x exponent less krg * the low byte of |I_p|^2.
    h2_t pa2[NY], pb2[NY];
    float ex[NY][NT];
#pragma unroll
    for (int k = 0; k < NY; ++k) {
        const uint32_t ip = guide_px<C>(guide, stride, px, py0 + k);
        const int np = (int)__builtin_amdgcn_udot4(ip, ip, 0u, false);
        if constexpr (C == 3) {
            pa2[k] = bits_h2(h2_bits(2.0f * (float)(ip & 255u), 2.0f * (float)((ip >> 8) & 255u)));
            pb2[k] = bits_h2(h2_bits(2.0f * (float)(ip >> 16), -(float)(np >> 8)));
        } else {
            pa2[k] = bits_h2(h2_bits(2.0f * (float)ip, -(float)(np >> 8)));
            pb2[k] = pa2[k];
        }
        const float np_lo = krg * (float)(np & 255);
#pragma unroll
        for (int i = 0; i < NT; ++i) ex[k][i] = t_sx[col * NT + i] - np_lo;
    }
    // Range part of a tap's exponent before scaling, from its record:
    // 2 I_p.I_q - |I_q|^2 - 256 floor(|I_p|^2 / 256), an exact integer (-inf
    // outside the grid).
    auto range = [&](int k, const uint4 &q) {
        float r = __builtin_amdgcn_fdot2(pa2[k], bits_h2(q.x), __uint_as_float(q.z), false);
        if constexpr (C == 3) r = __builtin_amdgcn_fdot2(pb2[k], bits_h2(q.y), r, false);
        return r;
    };
    float num[NY], den[NY];
#pragma unroll
    for (int k = 0; k < NY; ++k) num[k] = den[k] = 0.0f;
#pragma unroll
    for (int dy = 0; dy < NT; ++dy) {
        float rn[NY], rd[NY];
#pragma unroll
        for (int k = 0; k < NY; ++k) rn[k] = rd[k] = 0.0f;
#pragma unroll
        for (int dx = 0; dx < NT; ++dx) {
            const uint4 q = t_q[(oy + dy) * kMaxTap + ox + dx];
#pragma unroll
            for (int k = 0; k < NY; ++k) {
                const float w = __builtin_amdgcn_exp2f(fmaf(range(k, q), krg, ex[k][dx]));
                rn[k] = fmaf(w, __uint_as_float(q.w), rn[k]);
                rd[k] += w;
            }
        }
#pragma unroll
        for (int k = 0; k < NY; ++k) {
            const float wy = t_wy[(rowi + k) * NT + dy];
            num[k] = fmaf(wy, rn[k], num[k]);
            den[k] = fmaf(wy, rd[k], den[k]);
        }
    }
    if constexpr (NY > 1) {
        // Both rows need the second evaluation below somewhere in the wavefront:
        // in one pass over the records then, whose loads' latency bounds it with
        // half as many wavefronts (1600 x 904, s = 8, R 4, RGB, a noisy guide: 44.0
        // us one row after the other, 34.5 together, 35.7 with one row per thread).
        // Together also where one row needs it: 3 to 5% slower there.
        const bool low[2] = {!(den[0] >= 0x1p-60f), !(den[1] >= 0x1p-60f)};
        static_assert(NY == 2, "rows of a cell per thread");
        if ((low[0] || low[1]) && __any(low[0]) && __any(low[1])) {
            const float fx = (float)(px - s * cx) + 0.5f - 0.5f * (float)s;
            float fy[NY], emax[NY], rm[NY], sm[NY], n2[NY], d2[NY];
#pragma unroll
            for (int k = 0; k < NY; ++k) {
                fy[k] = (float)(py0 + k - s * cy) + 0.5f - 0.5f * (float)s;
                emax[k] = -__builtin_huge_valf();
                rm[k] = sm[k] = n2[k] = d2[k] = 0.0f;
            }
#pragma unroll 1
            for (int dy = 0; dy < NT; ++dy) {
                float sy[NY];
#pragma unroll
                for (int k = 0; k < NY; ++k) {
                    const float ty = fy[k] - (float)(s * (dy - R));
                    sy[k] = -(ty * ty * ksp);
                }
#pragma unroll 1
                for (int dx = 0; dx < NT; ++dx) {
                    const float tx = fx - (float)(s * (dx - R));
                    const uint4 q = t_q[(oy + dy) * kMaxTap + ox + dx];
#pragma unroll
                    for (int k = 0; k < NY; ++k) {
                        const float sp = sy[k] - tx * tx * ksp, r = range(k, q), e = fmaf(r, krg, sp);
                        const bool more = e > emax[k];
                        emax[k] = more ? e : emax[k];
                        rm[k] = more ? r : rm[k];
                        sm[k] = more ? sp : sm[k];
                    }
                }
            }
#pragma unroll 1
            for (int dy = 0; dy < NT; ++dy) {
                float sy[NY];
#pragma unroll
                for (int k = 0; k < NY; ++k) {
                    const float ty = fy[k] - (float)(s * (dy - R));
                    sy[k] = -(ty * ty * ksp);
                }
#pragma unroll 1
                for (int dx = 0; dx < NT; ++dx) {
                    const float tx = fx - (float)(s * (dx - R));
                    const uint4 q = t_q[(oy + dy) * kMaxTap + ox + dx];
#pragma unroll
                    for (int k = 0; k < NY; ++k) {
                        const float sp = sy[k] - tx * tx * ksp;
                        const float w = __builtin_amdgcn_exp2f(fmaf(range(k, q) - rm[k], krg, sp - sm[k]));
                        n2[k] = fmaf(w, __uint_as_float(q.w), n2[k]);
                        d2[k] += w;
                    }
                }
            }
#pragma unroll
            for (int k = 0; k < NY; ++k) {
                num[k] = low[k] ? n2[k] : num[k];
                den[k] = low[k] ? d2[k] : den[k];
            }
        }
    }
#pragma unroll
    for (int k = 0; k < NY; ++k) {
        const int py = py0 + k;
        if (!(den[k] >= 0x1p-60f)) {
            // Every weight is tiny: the same sums relative to the tap of largest
            // exponent (finite, since the pixel's own cell is in the grid), with
            // the range difference to it taken exactly before scaling so that
            // exponents far below zero keep their precision.
            // Separable spatial exponents: s * (p_lo - q) = phase + 0.5 - s/2 - s*dq.
            const float fx = (float)(px - s * cx) + 0.5f - 0.5f * (float)s;
            const float fy = (float)(py - s * cy) + 0.5f - 0.5f * (float)s;
            float emax = -__builtin_huge_valf(), rm = 0.0f, sm = 0.0f;
#pragma unroll 1
            for (int dy = 0; dy < NT; ++dy) {
                const float ty = fy - (float)(s * (dy - R)), sy = -(ty * ty * ksp);
#pragma unroll 1
                for (int dx = 0; dx < NT; ++dx) {
                    const float tx = fx - (float)(s * (dx - R)), sp = sy - tx * tx * ksp;
                    const float r = range(k, t_q[(oy + dy) * kMaxTap + ox + dx]), e = fmaf(r, krg, sp);
                    if (e > emax) {
                        emax = e;
                        rm = r;
                        sm = sp;
                    }
                }
            }
            num[k] = 0.0f;
            den[k] = 0.0f;
#pragma unroll 1
            for (int dy = 0; dy < NT; ++dy) {
                const float ty = fy - (float)(s * (dy - R)), sy = -(ty * ty * ksp);
#pragma unroll 1
                for (int dx = 0; dx < NT; ++dx) {
                    const float tx = fx - (float)(s * (dx - R)), sp = sy - tx * tx * ksp;
                    const uint4 q = t_q[(oy + dy) * kMaxTap + ox + dx];
                    const float w = __builtin_amdgcn_exp2f(fmaf(range(k, q) - rm, krg, sp - sm));
                    num[k] = fmaf(w, __uint_as_float(q.w), num[k]);
                    den[k] += w;
                }
            }
        }
        // den >= 2^-60 here (>= 1 after the second pass): a normal number.
        const float dp = num[k] * __builtin_amdgcn_rcpf(den[k]);
        if (out) out[(int64_t)py * wh + px] = dp;
        if constexpr (PTS) {
            const float d = (float)s * dp;
            float x = __builtin_nanf(""), y = x, z = x;
            if (d > 0.0f) {
                const float b = pa.baseline / d;
                x = b * ((float)px - pa.u0);
                y = b * ((float)py - pa.v0) * pa.dv_du;
                z = b * pa.f_du;
            }
            float *o = pa.xyz + ((int64_t)py * wh + px) * 3;
            o[0] = x;
            o[1] = y;
            o[2] = z;
        }
    }
}

template <int R, int C, int NY>
static void launch_jbu(const int32_t *disp_lo, int wl, int hl, const uint8_t *guide, int wh, int hh, int64_t stride,
                       float ksp, float krg, float *out, const PointArgs &pa, hipStream_t st)
{
    const int s = wh / wl;
    const float rs = 1.0f / (float)s;
    const dim3 grid((unsigned)((wh + kTile - 1) / kTile), (unsigned)((hh + kTile * NY - 1) / (kTile * NY)));
    if (pa.xyz) k_jbu<R, C, true, NY><<<grid, 256, 0, st>>>(disp_lo, wl, hl, guide, wh, hh, stride, s, rs, ksp, krg, out, pa);
    else k_jbu<R, C, false, NY><<<grid, 256, 0, st>>>(disp_lo, wl, hl, guide, wh, hh, stride, s, rs, ksp, krg, out, pa);
}

// Pixels per thread (NY): two rows of a cell share their taps' records and the
// setup, which is a quarter of the issue slots at R = 4 (RGB, s = 4, one / two
// rows: 2704 x 1520 R 4 79.2 / 72.3 us, R 2 33.5 / 29.4, R 1 22.7 / 18.4; 1600 x
// 900 R 4 31.7 / 30.7).  Small outputs need the threads (1000 x 560 R 4 15.8 /
// 16.6), and with one channel a wide window's sums outweigh the setup (2704 x
// 1520 R 4 62.3 / 62.5, R 2 28.9 / 25.6).  Four rows: 77.7, no better anywhere.
constexpr int kRowsRadius = 4, kRowsRadiusGrey = 2;
constexpr int64_t kRowsPixels = 1200000;

bp_status launch_upsample(const int32_t *disp_lo, int wl, int hl, const uint8_t *guide, int wh, int hh, int ch,
                          int64_t stride, float sigma_s, float sigma_r, int radius, float *out, const bp_camera *cam,
                          float *xyz, hipStream_t st)
{
    const float log2e = 1.4426950408889634f;
    const float ksp = log2e / (2.0f * sigma_s * sigma_s);
    const float krg = log2e / (2.0f * sigma_r * sigma_r);
    PointArgs pa{xyz, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
    if (cam) {
        pa.baseline = cam->baseline;
        pa.f_du = cam->focal / cam->du;
        pa.dv_du = cam->dv / cam->du;
        pa.u0 = cam->u0;
        pa.v0 = cam->v0;
    }
    const bool two = (wh / wl) % 2 == 0 && (int64_t)wh * hh >= kRowsPixels;
#define BP_JBU(RV, CV)                                                                                       \
    if (RV <= (CV == 1 ? kRowsRadiusGrey : kRowsRadius) && two)                                              \
        launch_jbu<RV, CV, (RV <= (CV == 1 ? kRowsRadiusGrey : kRowsRadius) ? 2 : 1)>(                       \
            disp_lo, wl, hl, guide, wh, hh, stride, ksp, krg, out, pa, st);                                  \
    else launch_jbu<RV, CV, 1>(disp_lo, wl, hl, guide, wh, hh, stride, ksp, krg, out, pa, st);
#define BP_JBU_CASE(RV)                                                                                      \
    case RV:                                                                                                 \
        if (ch == 1) { BP_JBU(RV, 1) }                                                                       \
        else { BP_JBU(RV, 3) }                                                                               \
        break;
    switch (radius) {
        BP_JBU_CASE(0)
        BP_JBU_CASE(1)
        BP_JBU_CASE(2)
        BP_JBU_CASE(3)
        BP_JBU_CASE(4)
        BP_JBU_CASE(5)
        BP_JBU_CASE(6)
        BP_JBU_CASE(7)
        BP_JBU_CASE(8)
    default: return BP_ERR_UNSUPPORTED;
    }
#undef BP_JBU_CASE
#undef BP_JBU
    return launch_status();
}

}  // namespace bpk
