// Undistortion of a frame under a radial-only lens model (Sec. 2.1: the
// calibrated intrinsics with radial distortion only; every frame is
// undistorted and remapped before matching).
//
// Output pixel (u, v) samples the distorted frame at
//   xn = (u - cx) / fx, yn = (v - cy) / fy, r2 = xn^2 + yn^2,
//   g = 1 + r2 (k1 + r2 (k2 + r2 k3)),  (us, vs) = (cx + (u - cx) g, cy + (v - cy) g)
// (the pinhole projection of the radially scaled normalised point, written so
// that g = 1 maps each pixel onto itself), with bilinear interpolation per
// channel rounded half up to u8, and 0 where (us, vs) leaves [0, W-1] x [0, H-1].
// The source position is computed per pixel, so no map is stored or read.
// Every operation is rounded on its own (no contraction into fused
// multiply-adds): the u8 result is decided in FP32 by a fixed sequence of
// operations.
//
// A thread takes four pixels of a column, so that a wave's gathers are those
// of 64 neighbouring pixels; the two source samples of a row are one unaligned
// load (8 bytes for RGB, 2 for grey).  The results change hands through LDS,
// so that they leave as one unaligned store of four pixels (12 or 4 bytes).
// Bound by instruction issue and the gathers together (about 90 vector
// operations per RGB pixel, 9 us of issue at 2704 x 1520, ahead of its 24.6 MB
// of HBM traffic).  Measured per call there: three aligned words per sample
// pair and three byte stores per pixel 18.4 us; four pixels of a row per
// thread 11.5; this mapping 11.2.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "bp_device.h"
#include "bp_internal.h"

namespace bpk {

constexpr int kUndistortPx = 4;   // pixels per thread

// Samples x0 and x0 + 1 of a row, `off` bytes into the frame of `total` bytes;
// what the load holds beyond the row's last pixel only meets a zero weight.
// Near the frame's end (END) the load is moved back so that it does not pass
// it, and the bytes are shifted.  TINY: frames shorter than one load, byte by
// byte.
enum { SAMPLE_FREE = 0, SAMPLE_END = 1, SAMPLE_TINY = 2 };

template <int C, int MODE, typename Off>
__device__ __forceinline__ void sample_row(const uint8_t *__restrict__ in, Off off, Off total, float (&p0)[C],
                                           float (&p1)[C])
{
    constexpr uint32_t N = C == 3 ? 8 : 2;
    if constexpr (MODE == SAMPLE_TINY) {
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const Off o1 = off + (Off)(C + c);
            p0[c] = in[off + (Off)c];
            p1[c] = in[o1 < total ? o1 : off];
        }
        return;
    }
    const Off at = MODE == SAMPLE_FREE || off < total - N ? off : total - N;
    const uint32_t sh = 8u * (uint32_t)(off - at);
    if constexpr (C == 3) {
        uint64_t w;
        __builtin_memcpy(&w, in + at, 8);
        if (MODE == SAMPLE_END) w >>= sh;
        const uint32_t lo = (uint32_t)w, hi = (uint32_t)(w >> 32);
        p0[0] = (float)(lo & 0xffu);
        p0[1] = (float)((lo >> 8) & 0xffu);
        p0[2] = (float)((lo >> 16) & 0xffu);
        p1[0] = (float)(lo >> 24);
        p1[1] = (float)(hi & 0xffu);
        p1[2] = (float)((hi >> 8) & 0xffu);
    } else {
        uint16_t h;
        __builtin_memcpy(&h, in + at, 2);
        const uint32_t w = MODE == SAMPLE_END ? (uint32_t)h >> sh : h;
        p0[0] = (float)(w & 0xffu);
        p1[0] = (float)((w >> 8) & 0xffu);
    }
}

// y * stride + x * C; with 32-bit offsets and sides and strides below 2^24
// (the host's condition) as a full-rate 24-bit multiply.
template <int C>
__device__ __forceinline__ uint32_t pixel_offset(int x, int y, uint32_t stride)
{
    return __umul24((uint32_t)y, stride) + (uint32_t)x * C;
}
template <int C>
__device__ __forceinline__ uint64_t pixel_offset(int x, int y, uint64_t stride)
{
    return (uint64_t)y * stride + (uint64_t)x * C;
}

// Off: 32-bit byte offsets where the frame has fewer than 2^32 bytes.
template <int C, bool TINY, typename Off>
__global__ void __launch_bounds__(256) k_undistort(const uint8_t *__restrict__ in, int w, int h, int64_t in_stride,
                                                  float fx_inv, float fy_inv, float cx, float cy, float k1, float k2,
                                                  float k3, uint8_t *__restrict__ out, int64_t out_stride)
{
#pragma clang fp contract(off)
    constexpr int N = kUndistortPx;
    // Wave t / 64 takes rows [v0, v0 + 4) of the block's 64 columns.
    __shared__ uint32_t s_px[4][N][64];
    const int lane = (int)threadIdx.x & 63, wv = (int)threadIdx.x >> 6;
    const int u = (int)blockIdx.x * 64 + lane, v0 = (int)blockIdx.y * 16 + wv * N;
    const Off stride = (Off)in_stride, total = (Off)(h - 1) * stride + (Off)w * C;
    const float du = (float)u - cx, xn = du * fx_inv, xx = xn * xn;
    const float xm = (float)(w - 1), ym = (float)(h - 1);
    float ax[N], ay[N];
    Off top_off[N], bot_off[N], last = 0;
    bool inside[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const float dv = (float)(v0 + i) - cy;
        const float yn = dv * fy_inv;
        const float r2 = xx + yn * yn;
        const float g = 1.0f + r2 * (k1 + r2 * (k2 + r2 * k3));
        const float us = cx + du * g, vs = cy + dv * g;
        inside[i] = us >= 0.0f && vs >= 0.0f && us <= xm && vs <= ym;
        const float xf = inside[i] ? __builtin_floorf(us) : 0.0f, yf = inside[i] ? __builtin_floorf(vs) : 0.0f;
        ax[i] = us - xf;
        ay[i] = vs - yf;
        const int y0 = (int)yf;
        top_off[i] = pixel_offset<C>((int)xf, y0, stride);
        // On the last row and column the weights of what lies beyond are zero.
        bot_off[i] = y0 + 1 < h ? top_off[i] + stride : top_off[i];
        last = bot_off[i] > last ? bot_off[i] : last;
    }
    auto blend = [&](auto mode) __attribute__((always_inline)) {
        constexpr int MODE = decltype(mode)::value;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            float p00[C], p10[C], p01[C], p11[C];
            sample_row<C, MODE, Off>(in, top_off[i], total, p00, p10);
            sample_row<C, MODE, Off>(in, bot_off[i], total, p01, p11);
            uint32_t px = 0u;
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const float top = p00[c] + ax[i] * (p10[c] - p00[c]);
                const float bot = p01[c] + ax[i] * (p11[c] - p01[c]);
                const float val = top + ay[i] * (bot - top);
                // A mean of bytes rounded half up: val + 0.5 lies in [0, 256),
                // so truncation is the floor and nothing is clamped.
                px |= (uint32_t)(val + 0.5f) << (8 * c);
            }
            s_px[wv][i][lane] = inside[i] ? px : 0u;
        }
    };
    if constexpr (TINY) {
        blend(std::integral_constant<int, SAMPLE_TINY>{});
    } else {
        // Few wavefronts sample the frame's last bytes.
        if (__any(last + 8 > total)) blend(std::integral_constant<int, SAMPLE_END>{});
        else blend(std::integral_constant<int, SAMPLE_FREE>{});
    }
    __syncthreads();
    // Four neighbouring pixels of row v0 + lane / 16.
    const int j = lane & 15, uo = (int)blockIdx.x * 64 + j * N, v = v0 + (lane >> 4);
    if (uo >= w || v >= h) return;
    uint32_t word[C] = {};
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const uint32_t px = s_px[wv][lane >> 4][j * N + i];
#pragma unroll
        for (int c = 0; c < C; ++c)
            word[(i * C + c) / 4] |= ((px >> (8 * c)) & 0xffu) << (8 * ((i * C + c) % 4));
    }
    uint8_t *o = out + (int64_t)v * out_stride + (int64_t)uo * C;
    if (uo + N <= w) {
        __builtin_memcpy(o, word, N * C);
    } else {
#pragma unroll
        for (int i = 0; i < N * C; ++i)
            if (uo + i / C < w) o[i] = (uint8_t)(word[i / 4] >> (8 * (i % 4)));
    }
}

template <int C>
static void undistort(const uint8_t *in, int w, int h, int64_t in_stride, const bp_intrinsics &K, uint8_t *out,
                      int64_t out_stride, hipStream_t st)
{
    const float fx_inv = 1.0f / K.fx, fy_inv = 1.0f / K.fy;
    const dim3 grid(((unsigned)w + 63) / 64, ((unsigned)h + 15) / 16);
    const int64_t total = (int64_t)(h - 1) * in_stride + (int64_t)w * C;
    if (total < 8)
        k_undistort<C, true, uint32_t><<<grid, 256, 0, st>>>(in, w, h, in_stride, fx_inv, fy_inv, K.cx, K.cy, K.k1,
                                                            K.k2, K.k3, out, out_stride);
    else if (total + in_stride < (1ll << 32) && w < (1 << 24) && h < (1 << 24) && in_stride < (1 << 24))
        k_undistort<C, false, uint32_t><<<grid, 256, 0, st>>>(in, w, h, in_stride, fx_inv, fy_inv, K.cx, K.cy, K.k1,
                                                             K.k2, K.k3, out, out_stride);
    else
        k_undistort<C, false, uint64_t><<<grid, 256, 0, st>>>(in, w, h, in_stride, fx_inv, fy_inv, K.cx, K.cy, K.k1,
                                                             K.k2, K.k3, out, out_stride);
}

bp_status launch_undistort(const uint8_t *in, int w, int h, int ch, int64_t in_stride, const bp_intrinsics &K,
                           uint8_t *out, int64_t out_stride, hipStream_t st)
{
    if (ch == 1) undistort<1>(in, w, h, in_stride, K, out, out_stride, st);
    else undistort<3>(in, w, h, in_stride, K, out, out_stride, st);
    return launch_status();
}

}  // namespace bpk
