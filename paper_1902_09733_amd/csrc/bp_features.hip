// The pose front end's data-parallel part (Sec. 2.3): Harris response
// (Eq. 4-5), per-cell corner selection (a g x g grid of cells with a hard
// threshold, as in the experiments), and ZSSD patch matching within a search
// range.  Everything is exact integer arithmetic:
//   A = I(x+1, y) - I(x-1, y), B = I(x, y+1) - I(x, y-1)   (central differences)
//   M = sum w [A^2, AB; AB, B^2], w = (1 4 6 4 1)^T (1 4 6 4 1)   (binomial window)
//   25 R = 25 det M - tr(M)^2   (Eq. 5 with k = 1/25), 0 within 3 of the border
//   n ZSSD = n sum (a - b)^2 - (sum a - sum b)^2   (n patch pixels)
// so selections (largest response, smallest cost) are decided without
// rounding.  Ties: first in row-major order.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "bp_internal.h"

namespace bpk {

typedef short s16x2 __attribute__((ext_vector_type(2)));

// Two bytes of (hi:lo) at positions I and J as 16-bit lanes.
template <int I, int J>
__device__ __forceinline__ s16x2 byte_pair(uint32_t lo, uint32_t hi)
{
    return __builtin_bit_cast(s16x2, __builtin_amdgcn_perm(hi, lo, 0x0c000c00u | (uint32_t)I | ((uint32_t)J << 16)));
}

// A thread takes one column of kHRows rows and slides down it: per image row
// one unaligned 8-byte load (columns x - 3 .. x + 4) gives the row's
// derivatives as 16-bit pairs, 16-bit dot products the horizontal window sums
// (weight times derivative is at most 6 * 255), and a ring of five rows of them
// the vertical ones.  No LDS: neighbouring columns' loads overlap in the
// vector cache.  Bound by instruction issue (about 90 operations per row and
// wavefront, 64-bit products among them) ahead of the 33 MB written: 19.7 us at
// 2704 x 1520, against 27.1 with 16 x 16 tiles staged in LDS.
// TINY: frames narrower than one load, byte by byte.
constexpr int kHRows = 16;

template <bool TINY>
__global__ void __launch_bounds__(256) k_harris_response(const uint8_t *__restrict__ img, int w, int h, int64_t stride,
                                                        int64_t *__restrict__ r25)
{
    const int x = (int)blockIdx.x * 64 + ((int)threadIdx.x & 63);
    const int y0 = ((int)blockIdx.y * 4 + ((int)threadIdx.x >> 6)) * kHRows;
    if (x >= w || y0 >= h) return;
    // Columns within 3 of the border respond 0 whatever is loaded for them.
    const bool in_x = x >= 3 && x <= w - 4;
    const int at = min(max(x - 3, 0), w - 8);
    const uint32_t sh = !TINY && in_x ? 8u * (uint32_t)(x - 3 - at) : 0u;
    auto load = [&](int y, uint32_t &lo, uint32_t &hi) __attribute__((always_inline)) {
        const uint8_t *row = img + (int64_t)min(max(y, 0), h - 1) * stride;
        uint64_t v = 0;
        if constexpr (TINY) {
#pragma unroll
            for (int k = 0; k < 8; ++k) v |= (uint64_t)row[min(max(x - 3 + k, 0), w - 1)] << (8 * k);
        } else {
            __builtin_memcpy(&v, row + at, 8);
        }
        lo = (uint32_t)v;
        hi = (uint32_t)(v >> 32);
    };
    const s16x2 w0 = {1, 4}, w1 = {6, 4}, w2 = {1, 0};
    // Of the rows above: derivatives A of the last row, 16-bit columns
    // x - 2 .. x + 3 of the last two rows.
    s16x2 a0{}, a1{}, a2{}, p0[2]{}, p1[2]{}, p2[2]{};
    int32_t xx[5]{}, yy[5]{}, xy[5]{};
    uint32_t los[kHRows + 6], his[kHRows + 6];   // every row's load is under way before the first is used
#pragma unroll
    for (int i = 0; i < kHRows + 6; ++i) load(y0 - 3 + i, los[i], his[i]);
    // Branch-free stores where the strip is whole: a store that may be skipped
    // makes the waits for later rows' loads wait for earlier stores.
    const int64_t keep = in_x ? -1 : 0;
    auto rows = [&](auto whole) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < kHRows + 6; ++i) {
        // Image row r = y0 - 3 + i completes the derivatives of row r - 1 and
        // the window centred on row r - 3.
        const uint64_t row8 = (((uint64_t)his[i] << 32) | los[i]) >> sh;
        const uint32_t lo = (uint32_t)row8, hi = (uint32_t)(row8 >> 32);
        const s16x2 c0 = byte_pair<1, 2>(lo, hi), c1 = byte_pair<3, 4>(lo, hi), c2 = byte_pair<5, 6>(lo, hi);
        if (i >= 2) {
            const s16x2 b0 = c0 - p0[1], b1 = c1 - p1[1], b2 = c2 - p2[1];
            const s16x2 wa0 = a0 * w0, wa1 = a1 * w1, wa2 = a2 * w2, wb0 = b0 * w0, wb1 = b1 * w1, wb2 = b2 * w2;
            auto dot3 = [](s16x2 u0, s16x2 u1, s16x2 u2, s16x2 v0, s16x2 v1, s16x2 v2) __attribute__((always_inline)) {
                return __builtin_amdgcn_sdot2(u0, v0, __builtin_amdgcn_sdot2(u1, v1, __builtin_amdgcn_sdot2(u2, v2, 0, false),
                                                                            false), false);
            };
            const int k = (i - 2) % 5;
            xx[k] = dot3(wa0, wa1, wa2, a0, a1, a2);
            yy[k] = dot3(wb0, wb1, wb2, b0, b1, b2);
            xy[k] = dot3(wa0, wa1, wa2, b0, b1, b2);
        }
        if (i >= 6) {
            const int y = y0 + i - 6;
            if (!decltype(whole)::value && y >= h) return;
            auto column = [&](const int32_t (&s)[5]) __attribute__((always_inline)) {
                const int k = (i - 2) % 5;   // newest of the five rows
                const int32_t mid = s[(k + 3) % 5];
                return s[(k + 1) % 5] + s[k] + ((s[(k + 2) % 5] + s[(k + 4) % 5] + mid) << 2) + (mid << 1);
            };
            // At most 65025 * 256 each.
            const int32_t sxx = column(xx), syy = column(yy), sxy = column(xy), tr = sxx + syy;
            const int64_t det = (int64_t)sxx * syy - (int64_t)sxy * sxy;
            const int64_t v = (det << 4) + ((det << 3) + det) - (int64_t)tr * tr;
            r25[(int64_t)y * w + x] = v & (y >= 3 && y <= h - 4 ? keep : 0);
        }
        a0 = byte_pair<2, 3>(lo, hi) - byte_pair<0, 1>(lo, hi);
        a1 = byte_pair<4, 5>(lo, hi) - byte_pair<2, 3>(lo, hi);
        a2 = byte_pair<6, 7>(lo, hi) - byte_pair<4, 5>(lo, hi);
        p0[1] = p0[0];
        p1[1] = p1[0];
        p2[1] = p2[0];
        p0[0] = c0;
        p1[0] = c1;
        p2[0] = c2;
    }
    };
    if (y0 + kHRows <= h) rows(std::true_type{});
    else rows(std::false_type{});
}

// One block per cell: the largest response above the threshold among the
// cell's 3 x 3 local maxima, first in row-major order on ties.  The block's
// threads share the cell's columns out (up to 256 at a time) and its rows into
// as many runs as there are threads for; a thread slides down its column with
// the maxima of the three columns around it in the last rows, so each response
// is read three times, once from memory (outside the frame: INT64_MIN, never
// larger).  Bound by the latency of its row loads (3.5 wavefronts per SIMD):
// 15 us for 900 cells of 2704 x 1520, against 24.7 with strips of every cell
// staged in LDS; a first pass for the cell's largest response with a search
// only where a neighbour outside the cell is larger took 27.1, the few cells
// searched deciding the launch's time.
constexpr int kSelRows = 4;             // rows loaded ahead

__device__ __forceinline__ void take_best(int64_t v, int64_t idx, int64_t &bv, int64_t &bi)
{
    if (bi < 0 || v > bv || (v == bv && idx < bi)) {
        bv = v;
        bi = idx;
    }
}

__global__ void __launch_bounds__(256) k_harris_select(const int64_t *__restrict__ r25, int w, int h, int g,
                                                      int64_t thr, bp_corner *__restrict__ out)
{
    __shared__ int64_t s_v[4], s_i[4];
    const int ci = blockIdx.x / g, cj = blockIdx.x - ci * g;
    const int x0 = (int)((int64_t)cj * w / g), x1 = (int)((int64_t)(cj + 1) * w / g);
    const int y0 = (int)((int64_t)ci * h / g), y1 = (int)((int64_t)(ci + 1) * h / g);
    const int cw = x1 - x0, ch = y1 - y0;
    int64_t bv = 0, bi = -1;       // best value and row-major index of its pixel
    const int cols = min(max(cw, 1), 256), runs = 256 / cols;
    const int run = (int)threadIdx.x / cols, len = (ch + runs - 1) / runs;
    const int ya = y0 + run * len, yb = run < runs ? min(y1, ya + len) : ya;
    for (int x = x0 + (int)threadIdx.x - run * cols; x < x1; x += cols) {
        // Row y's response and the maximum of it and its two neighbours.
        auto load = [&](int y, int64_t &c, int64_t &l, int64_t &r) __attribute__((always_inline)) {
            c = l = r = INT64_MIN;
            if (y >= 0 && y < h) {
                const int64_t *row = r25 + (int64_t)y * w + x;
                c = row[0];
                if (x > 0) l = row[-1];
                if (x + 1 < w) r = row[1];
            }
        };
        if (ya >= yb) continue;
        int64_t c, l, r;
        load(ya - 1, c, l, r);
        int64_t above = max(max(l, r), c);
        load(ya, c, l, r);
        int64_t mid = c, side = max(l, r);
        for (int y = ya; y < yb; y += kSelRows) {
            int64_t nc[kSelRows], nl[kSelRows], nr[kSelRows];
#pragma unroll
            for (int k = 0; k < kSelRows; ++k) load(y + 1 + k, nc[k], nl[k], nr[k]);
#pragma unroll
            for (int k = 0; k < kSelRows; ++k) {
                const int64_t nside = max(nl[k], nr[k]), below = max(nside, nc[k]);
                if (y + k < yb && mid > thr && mid >= above && mid >= side && mid >= below)
                    take_best(mid, (int64_t)(y + k) * w + x, bv, bi);
                above = max(side, mid);
                mid = nc[k];
                side = nside;
            }
        }
    }
    // Largest of the block, first in row-major order on ties.
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        const int64_t ov = __shfl_xor(bv, d), oi = __shfl_xor(bi, d);
        if (oi >= 0) take_best(ov, oi, bv, bi);
    }
    if ((threadIdx.x & 63) == 0) {
        s_v[threadIdx.x >> 6] = bv;
        s_i[threadIdx.x >> 6] = bi;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int k = 1; k < 4; ++k)
            if (s_i[k] >= 0) take_best(s_v[k], s_i[k], bv, bi);
        bp_corner c;
        c.y = bi < 0 ? -1 : (int32_t)(bi / w);
        c.x = bi < 0 ? -1 : (int32_t)(bi - (int64_t)c.y * w);
        c.response = bi < 0 ? 0 : bv;
        out[blockIdx.x] = c;
    }
}

// Words of a region row in LDS: the widest shift's first word and the patch's,
// an odd number so that rows spread over the banks.
__host__ __device__ inline int zssd_row_words(int pw, int sr) { return ((2 * sr) / 4 + pw) | 1; }

// One block per corner: every shift in [-sr, sr]^2 whose patch lies inside
// frame b.  With sum (a - b)^2 = sum a^2 - 2 sum ab + sum b^2, all three (and the
// plain sums) are byte dot products of four pixels at a time: the patch of
// frame a is staged in LDS as words (PW per row, zero beyond the patch), the
// search region of frame b four times, copy c starting c bytes later, so that
// every shift's rows are whole words of one copy.  A thread takes one
// horizontal shift and kZD vertical ones, so that each of its region rows is
// read once for all of them.  The smallest n ZSSD wins, the first shift in
// row-major order on ties.  Bound by the latency of staging and of the LDS
// reads: 14.3 us for 900 corners, 33 x 33 shifts and 11 x 11 pixels, against
// 47.6 with one byte product per pixel and shift.
constexpr int kZD = 5;

template <int PW>
__global__ void __launch_bounds__(256) k_zssd(const uint8_t *__restrict__ a, const uint8_t *__restrict__ b, int w,
                                             int h, int64_t stride, const bp_corner *__restrict__ corners, int pr,
                                             int sr, bp_match *__restrict__ out)
{
    extern __shared__ uint32_t s_mem[];
    __shared__ int64_t s_c[4];
    __shared__ int32_t s_k[4];
    const bp_corner c = corners[blockIdx.x];
    const int P = 2 * pr + 1, S = 2 * sr + 1, G = P + 2 * sr;
    const bool ok = c.x >= pr && c.y >= pr && c.x + pr < w && c.y + pr < h;
    if (!ok) {
        if (threadIdx.x == 0) out[blockIdx.x] = bp_match{-1, -1, 0};
        return;
    }
    const int RW = zssd_row_words(PW, sr), CS = G * RW;     // words of a region row and of a copy
    uint32_t *const s_b = s_mem, *const s_a = s_mem + 4 * CS;
    // Word at pixel (x, y) of a frame, zero outside it.
    auto word = [&](const uint8_t *f, int x, int y) __attribute__((always_inline)) {
        uint32_t v = 0u;
        if (y >= 0 && y < h) {
            const uint8_t *row = f + (int64_t)y * stride;
            if (x >= 0 && x + 3 < w) {
                __builtin_memcpy(&v, row + x, 4);
            } else {
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if (x + k >= 0 && x + k < w) v |= (uint32_t)row[x + k] << (8 * k);
            }
        }
        return v;
    };
    const uint32_t tail = P % 4 ? (1u << (8 * (P % 4))) - 1u : ~0u;   // bytes of a row's last word inside the patch
    for (int i = threadIdx.x; i < P * PW; i += 256) {
        const int j = i / PW, k = i - j * PW;
        const uint32_t v = word(a, c.x - pr + 4 * k, c.y - pr + j);
        s_a[i] = k == PW - 1 ? v & tail : v;
    }
    for (int i = threadIdx.x; i < CS; i += 256) {
        const int j = i / RW, k = i - j * RW;
        const int x = c.x - sr - pr + 4 * k, y = c.y - sr - pr + j;
        const uint32_t lo = word(b, x, y), hi = word(b, x + 4, y);
        s_b[i] = lo;
        s_b[CS + i] = __builtin_amdgcn_alignbyte(hi, lo, 1);
        s_b[2 * CS + i] = __builtin_amdgcn_alignbyte(hi, lo, 2);
        s_b[3 * CS + i] = __builtin_amdgcn_alignbyte(hi, lo, 3);
    }
    __syncthreads();
    // 32-bit sums: at most 31^2 pixels, so sums of squares stay below 2^26.
    uint32_t sa = 0u, saa = 0u;
    for (int i = 0; i < P * PW; ++i) {
        sa = __builtin_amdgcn_udot4(s_a[i], 0x01010101u, sa, false);
        saa = __builtin_amdgcn_udot4(s_a[i], s_a[i], saa, false);
    }
    const int64_t np = (int64_t)P * P;
    int64_t best = -1;
    int bk = -1;
    const int groups = (S + kZD - 1) / kZD;
    for (int item = threadIdx.x; item < S * groups; item += 256) {
        const int gy = item / S, kx = item - gy * S, ky0 = gy * kZD;
        const uint32_t *col = s_b + (kx & 3) * CS + (kx >> 2) + ky0 * RW;
        uint32_t ab[kZD] = {}, sb[kZD] = {}, sbb[kZD] = {};
        const int rows = min(P + kZD - 1, G - ky0);
        for (int r = 0; r < rows; ++r) {
            uint32_t v[PW], hb = 0u, hbb = 0u;
#pragma unroll
            for (int k = 0; k < PW; ++k) v[k] = col[r * RW + k];
            v[PW - 1] &= tail;
#pragma unroll
            for (int k = 0; k < PW; ++k) {
                hb = __builtin_amdgcn_udot4(v[k], 0x01010101u, hb, false);
                hbb = __builtin_amdgcn_udot4(v[k], v[k], hbb, false);
            }
#pragma unroll
            for (int d = 0; d < kZD; ++d) {
                const int j = r - d;           // patch row that vertical shift ky0 + d lays on this row
                if (j < 0 || j >= P) continue;
                sb[d] += hb;
                sbb[d] += hbb;
#pragma unroll
                for (int k = 0; k < PW; ++k) ab[d] = __builtin_amdgcn_udot4(s_a[j * PW + k], v[k], ab[d], false);
            }
        }
        for (int d = 0; d < kZD; ++d) {
            const int ky = ky0 + d, qx = c.x + kx - sr, qy = c.y + ky - sr, s = ky * S + kx;
            if (ky >= S || qx < pr || qy < pr || qx + pr >= w || qy + pr >= h) continue;
            const int64_t sd = (int64_t)saa + sbb[d] - 2 * (int64_t)ab[d], ds = (int64_t)sa - (int64_t)sb[d];
            const int64_t cost = np * sd - ds * ds;
            if (bk < 0 || cost < best || (cost == best && s < bk)) {
                best = cost;
                bk = s;
            }
        }
    }
    auto take = [](int64_t oc, int ok2, int64_t &mc, int &mk) {
        if (ok2 >= 0 && (mk < 0 || oc < mc || (oc == mc && ok2 < mk))) {
            mc = oc;
            mk = ok2;
        }
    };
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        const int64_t oc = __shfl_xor(best, d);
        const int ok2 = __shfl_xor(bk, d);
        take(oc, ok2, best, bk);
    }
    if ((threadIdx.x & 63) == 0) {
        s_c[threadIdx.x >> 6] = best;
        s_k[threadIdx.x >> 6] = bk;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int k = 1; k < 4; ++k) take(s_c[k], s_k[k], best, bk);
        out[blockIdx.x] = bk < 0 ? bp_match{-1, -1, 0} : bp_match{c.x + (bk % S - sr), c.y + (bk / S - sr), best};
    }
}

bp_status launch_harris(const uint8_t *img, int w, int h, int64_t stride, int g, int64_t thr, int64_t *r25,
                        bp_corner *corners, hipStream_t st)
{
    const dim3 grid(((unsigned)w + 63) / 64, ((unsigned)h + 4 * kHRows - 1) / (4 * kHRows));
    if (w < 8) k_harris_response<true><<<grid, 256, 0, st>>>(img, w, h, stride, r25);
    else k_harris_response<false><<<grid, 256, 0, st>>>(img, w, h, stride, r25);
    bp_status s = launch_status();
    if (s != BP_OK) return s;
    k_harris_select<<<(unsigned)(g * g), 256, 0, st>>>(r25, w, h, g, thr, corners);
    return launch_status();
}

bp_status launch_zssd(const uint8_t *a, const uint8_t *b, int w, int h, int64_t stride, const bp_corner *corners,
                      int n, int pr, int sr, bp_match *out, hipStream_t st)
{
    if (n == 0) return BP_OK;
    const int P = 2 * pr + 1, pw = (P + 3) / 4;
    const size_t lds = ((size_t)4 * (P + 2 * sr) * zssd_row_words(pw, sr) + (size_t)P * pw) * 4;
    switch (pw) {
#define BP_ZSSD(PW) \
    case PW: k_zssd<PW><<<(unsigned)n, 256, lds, st>>>(a, b, w, h, stride, corners, pr, sr, out); break;
        BP_ZSSD(1) BP_ZSSD(2) BP_ZSSD(3) BP_ZSSD(4) BP_ZSSD(5) BP_ZSSD(6) BP_ZSSD(7) BP_ZSSD(8)
#undef BP_ZSSD
    default: return BP_ERR_UNSUPPORTED;
    }
    return launch_status();
}

}  // namespace bpk
