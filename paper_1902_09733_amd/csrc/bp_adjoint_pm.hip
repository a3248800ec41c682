// a8 on pixel-major states: the reverse half-sweep with the labels of a
// pixel spread over lanes, as in the forward pixel-major kernels (a sender
// pixel owns SEG lanes, R labels per lane, and handles its four outgoing
// messages k in turn, sharing the loads of its cost, incoming rows and
// adjoints and the partial sums of h).
//
// Per message the forward arithmetic is repeated exactly (same sums, same
// lane-local passes and cross-lane carries), now carrying the winner label
// along every minimum:
//   forward pass  A(f) = min(h(f), A(f-1) + lambda), the later label on ties
//                 (larger winner across lanes);
//   backward pass B(f) = min(A(f), B(f+1) + lambda), the current value on
//                 ties (smaller winner across lanes);
//   truncation    applies only when min h + lambda tau < B(f) strictly.
// Given the receiver slot's adjoint mb(f), h-bar(winner(f)) += mb(f) and
// h-bar(gmin) -= mb(f) for untruncated f, with the lambda / tau partials as
// in the label-major reverse step.  The scatter is deterministic in two
// phases through LDS: every lane posts (winner, mb) of its labels, then
// every lane adds, for each of its labels g, the posted mb of the labels f
// with winner g in increasing f.  An untruncated winner lies within tau of f
// (h(g) + lambda |f - g| <= min h + lambda tau), so f only ranges over a
// window of `win` labels around g (all labels when lambda = 0).
//
// A window of at most kNear labels (tau < 3) reaches no further than the next
// lane.  Then the scans need only that lane's values (what comes from further
// off exceeds min h + lambda tau whatever it is, and so does everything that
// depends on it), and phase 2 takes the next lanes' posts through DPP: no LDS,
// and the adds of a label in the same order.  At eight 320 x 240 x 64 problems
// (1.18 GB moved per reverse step) the general form issues about 2460 VALU
// instructions per wavefront and runs 239 us, issue bound; the near one 1480
// and 210 us, 5.6 TB/s: memory bound.
#include <hip/hip_runtime.h>

#include "bp_device.h"
#include "bp_internal.h"
#include "bp_pm_core.h"

namespace bpk {

// Level-0 geometry of a pixel-major level, passed by value to kernels.
struct PmDesc {
    int w, h, wh;
    int64_t blk, lp;
};

static PmDesc pm_desc(const Level &v) { return PmDesc{v.w, v.h, v.wh, v.blk, (int64_t)v.lp}; }

struct BwdPmArgs {
    const float *cost;      // level-0 cost, pixel-major
    uint32_t cost_bytes;
    const uint8_t *msg;     // state M_t, pixel-major float32
    uint32_t msg_bytes;
    float *mbar;            // adjoint of the message state, same layout
    uint32_t mbar_bytes;
    float *gcost;           // adjoint of the cost, pixel-major like `cost`
    float *partial;         // per-block (lambda, tau) partial sums
    int w, h, wh;
    uint32_t blk, lp;
    int colour, L, ncomp, win;
    int first;              // 1 for the first reverse step (t = K - 1)
    float lambda, tau, lt;
};

// Value and winner of lane (s - N) of the segment, or (inf, -1) below it.
template <int SEG, int N>
__device__ __forceinline__ void pair_from_lower(float v, int i, int s, float &ov, int &oi)
{
    ov = dpp_f<0x110 + N>(__builtin_huge_valf(), v);
    oi = dpp_i<0x110 + N>(-1, i);
    if constexpr (SEG < 16) {
        if (s < N) {
            ov = __builtin_huge_valf();
            oi = -1;
        }
    }
}

// Value and winner of lane (s + N) of the segment, or (inf, -1) above it.
template <int SEG, int N>
__device__ __forceinline__ void pair_from_upper(float v, int i, int s, float &ov, int &oi)
{
    ov = dpp_f<0x100 + N>(__builtin_huge_valf(), v);
    oi = dpp_i<0x100 + N>(-1, i);
    if constexpr (SEG < 16) {
        if (s + N >= SEG) {
            ov = __builtin_huge_valf();
            oi = -1;
        }
    }
}

// Exclusive prefix minimum over lanes 0..s-1 with its winner (ties: the
// larger winner, i.e. the nearer lane).
template <int SEG>
__device__ __forceinline__ void pair_prefix_excl(float u, int ui, int s, float &pv, int &pi)
{
    pair_from_lower<SEG, 1>(u, ui, s, pv, pi);
    auto step = [&](float ov, int oi) {
        if (ov < pv || (ov == pv && oi > pi)) {
            pv = ov;
            pi = oi;
        }
    };
    float ov;
    int oi;
    if constexpr (SEG > 1) {
        pair_from_lower<SEG, 1>(pv, pi, s, ov, oi);
        step(ov, oi);
    }
    if constexpr (SEG > 2) {
        pair_from_lower<SEG, 2>(pv, pi, s, ov, oi);
        step(ov, oi);
    }
    if constexpr (SEG > 4) {
        pair_from_lower<SEG, 4>(pv, pi, s, ov, oi);
        step(ov, oi);
    }
    if constexpr (SEG > 8) {
        pair_from_lower<SEG, 8>(pv, pi, s, ov, oi);
        step(ov, oi);
    }
}

// Exclusive suffix minimum over lanes s+1..SEG-1 with its winner (ties: the
// smaller winner, i.e. the nearer lane).
template <int SEG>
__device__ __forceinline__ void pair_suffix_excl(float v, int vi, int s, float &qv, int &qi)
{
    pair_from_upper<SEG, 1>(v, vi, s, qv, qi);
    auto step = [&](float ov, int oi) {
        if (ov < qv || (ov == qv && oi >= 0 && (qi < 0 || oi < qi))) {
            qv = ov;
            qi = oi;
        }
    };
    float ov;
    int oi;
    if constexpr (SEG > 1) {
        pair_from_upper<SEG, 1>(qv, qi, s, ov, oi);
        step(ov, oi);
    }
    if constexpr (SEG > 2) {
        pair_from_upper<SEG, 2>(qv, qi, s, ov, oi);
        step(ov, oi);
    }
    if constexpr (SEG > 4) {
        pair_from_upper<SEG, 4>(qv, qi, s, ov, oi);
        step(ov, oi);
    }
    if constexpr (SEG > 8) {
        pair_from_upper<SEG, 8>(qv, qi, s, ov, oi);
        step(ov, oi);
    }
}

// Window, in labels, of the near form (kNear <= R).
constexpr int kNear = 4;

// Byte offset past every row: loads there return zero, stores are dropped.
constexpr uint32_t kNoRow = 0xffffff00u;

template <int SEG, int R, bool NEAR>
__device__ __forceinline__ void bwd_step_pm(const BwdPmArgs &a, uint32_t block)
{
    // The forward arithmetic is repeated exactly as the half-sweep kernels
    // do it: products rounded before they are added (bp_pm_core.h).
#pragma clang fp contract(off)
    constexpr int LP = SEG * R;           // labels stored per pixel
    constexpr int PPB = 256 / SEG;        // pixels per block
    // Posted mb and winner (a byte: labels are fewer than 128 here): per
    // pixel its four messages' rows of LP labels, each row preceded and
    // followed by PAD entries that post nothing (winner -1), so that a window
    // of up to PAD labels around a lane's labels needs no clamping at the
    // row's ends.
    static_assert(LP <= kMaxBackwardLabels && kMaxBackwardLabels <= 128, "winners must fit a signed byte");
    static_assert(kNear <= R, "the near form reaches one lane");
    constexpr int PAD = 4;
    constexpr int PROW = 4 * (LP + PAD) + PAD;
    __shared__ float s_pv[NEAR ? 1 : PPB * PROW];
    __shared__ int8_t s_pw[NEAR ? 1 : PPB * PROW];
    __shared__ float s_part[4][2];
    const uint32_t gid = block * 256u + threadIdx.x;
    const int j = (int)(gid / SEG);
    const int s = (int)(gid % SEG);
    const int f0 = s * R;
    const int prow = (int)(threadIdx.x / SEG) * PROW;
    if constexpr (!NEAR) {
        for (int e = (int)threadIdx.x; e < PPB * 5 * PAD; e += 256) {
            const int px = e / (5 * PAD), q = e - px * (5 * PAD);
            const int at = px * PROW + (q / PAD) * (LP + PAD) + q % PAD;
            s_pv[at] = 0.0f;
            s_pw[at] = -1;
        }
    }
    const int y = j / a.wh, x = 2 * (j - y * a.wh) + ((y + a.colour) & 1);
    const bool live = j < a.ncomp && x < a.w;
    const bool has[4] = {live && x > 0, live && x < a.w - 1, live && y > 0, live && y < a.h - 1};
    const __amdgpu_buffer_rsrc_t rc = make_rsrc(a.cost, a.cost_bytes);
    const __amdgpu_buffer_rsrc_t rm = make_rsrc(a.msg, a.msg_bytes);
    const __amdgpu_buffer_rsrc_t rb = make_rsrc(a.mbar, a.mbar_bytes);
    const __amdgpu_buffer_rsrc_t rg = make_rsrc(a.gcost, a.cost_bytes);
    const float inf = __builtin_huge_valf();
    const float lam = a.lambda;
    const float lamR = lam * (float)R;
    const uint32_t base = (uint32_t)j * a.lp + (uint32_t)f0;
    const uint32_t cb = (uint32_t)a.colour * a.blk, mb4 = 4u * cb;   // the colour's blocks of cost and messages

    // The four receiver slots' adjoints (zeros for a missing neighbour), the
    // cost adjoint this pixel accumulates, the cost and the four incoming
    // rows, all loaded before any arithmetic.  At the first reverse step a
    // slot's adjoint is its pixel's readout adjoint, which the cost adjoint
    // holds.  The receiver slots are not cleared: every in-grid slot of the
    // receivers' colour is overwritten by the next reverse step's sender side
    // before anything reads it again.
    float mbv[4][R];
    const uint32_t other = a.blk - cb;                      // the other colour's block (colour 0 or 1)
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int nx = k == 0 ? x - 1 : k == 1 ? x + 1 : x, ny = k == 2 ? y - 1 : k == 3 ? y + 1 : y;
        const uint32_t row = (uint32_t)(ny * a.wh + (nx >> 1)) * a.lp + (uint32_t)f0;
        const uint32_t slot = a.first ? other : 4u * other + (uint32_t)(k ^ 1) * a.blk;
        ld_row<StoreF32, R>(a.first ? rg : rb, has[k] ? (slot + row) * 4u : kNoRow, mbv[k]);
    }
    const uint32_t goff = live ? (cb + base) * 4u : kNoRow;
    float gc[R];
    ld_row<StoreF32, R>(rg, goff, gc);
    // h of the four outgoing messages, summed as in the forward kernels.
    float h[4][R];
    {
        float c[R], m[4][R];
        ld_row<StoreF32, R>(rc, goff, c);
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
            ld_row<StoreF32, R>(rm, live ? (mb4 + (uint32_t)kk * a.blk + base) * 4u : kNoRow, m[kk]);
        pm_h4<R>(c, m, h);
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (f0 + r >= a.L) h[k][r] = inf;
    }

    // Phase 1, message by message: the transform with winners (label minus f0,
    // as floats: exact, and |f - winner| needs no conversion), then post
    // (winner, mb) of the receiver slot's adjoint.
    float lsum = 0.0f, tsum = 0.0f, nsum[4], hb[4][R];
    float gmin[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        // Lowest minimiser of h.
        float hmin = h[k][0];
#pragma unroll
        for (int r = 1; r < R; ++r) hmin = fminf(hmin, h[k][r]);
        hmin = seg_allmin<SEG>(hmin);
        float gm = (float)LP;
#pragma unroll
        for (int r = R - 1; r >= 0; --r) gm = h[k][r] == hmin ? (float)(f0 + r) : gm;
        gmin[k] = seg_allmin<SEG>(gm) - (float)f0;
        // Forward pass with winners.
        float A[R], wa[R];
        A[0] = h[k][0];
        wa[0] = 0.0f;
#pragma unroll
        for (int r = 1; r < R; ++r) {
            const float v = A[r - 1] + lam;
            const bool keep = h[k][r] <= v;
            A[r] = keep ? h[k][r] : v;
            wa[r] = keep ? (float)r : wa[r - 1];
        }
        {
            float pv, pi;
            const float u = A[R - 1] - lamR * (float)s;
            if constexpr (NEAR) {
                pv = seg_from_lower<SEG, 1>(u, inf, s);
                pi = seg_from_lower<SEG, 1>(wa[R - 1], 0.0f, s) - (float)R;
            } else {
                int i;
                pair_prefix_excl<SEG>(u, f0 + (int)wa[R - 1], s, pv, i);
                pi = (float)(i - f0);
            }
            const float carry = pv + lamR * (float)(s - 1);
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const float cand = carry + lam * (float)(r + 1);
                const bool take = cand < A[r];
                A[r] = take ? cand : A[r];
                wa[r] = take ? pi : wa[r];
            }
        }
        // Backward pass with winners.
        float B[R], wb[R];
        B[R - 1] = A[R - 1];
        wb[R - 1] = wa[R - 1];
#pragma unroll
        for (int r = R - 2; r >= 0; --r) {
            const float v = B[r + 1] + lam;
            const bool take = v < A[r];
            B[r] = take ? v : A[r];
            wb[r] = take ? wb[r + 1] : wa[r];
        }
        {
            float qv, qi;
            const float u = B[0] + lamR * (float)s;
            if constexpr (NEAR) {
                qv = seg_from_upper<SEG, 1>(u, inf, s);
                qi = seg_from_upper<SEG, 1>(wb[0], 0.0f, s) + (float)R;
            } else {
                int i;
                pair_suffix_excl<SEG>(u, f0 + (int)wb[0], s, qv, i);
                qi = (float)(i - f0);
            }
            const float carry = qv - lamR * (float)(s + 1);
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const float cand = carry + lam * (float)(R - r);
                const bool take = cand < B[r];
                B[r] = take ? cand : B[r];
                wb[r] = take ? qi : wb[r];
            }
        }
        const float cap = hmin + a.lt;
        float ns = 0.0f, post[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const float mb = f0 + r < a.L ? mbv[k][r] : 0.0f;
            const bool cut = cap < B[r];
            post[r] = cut ? 0.0f : mb;
            ns += post[r];
            lsum += mb * (cut ? a.tau : fabsf((float)r - wb[r]));
            tsum += cut ? mb * a.lambda : 0.0f;
            wb[r] = cut ? 1024.0f : wb[r];                  // no label
        }
        nsum[k] = ns;
        if constexpr (NEAR) {
            // Phase 2: h-bar of this lane's labels from the posts within kNear
            // labels of them, in increasing label.
#pragma unroll
            for (int r = 0; r < R; ++r) hb[k][r] = 0.0f;
#pragma unroll
            for (int i = R - kNear; i < R; ++i) {
                const float pv = seg_from_lower<SEG, 1>(post[i], 0.0f, s), w = seg_from_lower<SEG, 1>(wb[i], 0.0f, s);
#pragma unroll
                for (int r = 0; r <= i - (R - kNear); ++r) hb[k][r] += w == (float)(R + r) ? pv : 0.0f;
            }
#pragma unroll
            for (int i = 0; i < R; ++i)
#pragma unroll
                for (int r = 0; r < R; ++r)
                    if (i - r <= kNear && r - i <= kNear) hb[k][r] += wb[i] == (float)r ? post[i] : 0.0f;
#pragma unroll
            for (int i = 0; i < kNear; ++i) {
                const float pv = seg_from_upper<SEG, 1>(post[i], 0.0f, s), w = seg_from_upper<SEG, 1>(wb[i], 0.0f, s);
#pragma unroll
                for (int r = R - kNear + i; r < R; ++r) hb[k][r] += w == (float)(r - R) ? pv : 0.0f;
            }
        } else {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                s_pv[prow + PAD + k * (LP + PAD) + f0 + r] = post[r];
                s_pw[prow + PAD + k * (LP + PAD) + f0 + r] = wb[r] < 1024.0f ? (int8_t)(f0 + (int)wb[r]) : (int8_t)-1;
            }
        }
    }

    // Phase 2: h-bar of this lane's labels for each message.  One pass over
    // the posts that can reach them (winners lie within `win` of their
    // label); every h-bar(g) still adds its posts in increasing f.
    if constexpr (!NEAR) __syncthreads();
    const int lo = f0 - a.win > 0 ? f0 - a.win : 0;
    const int hi = f0 + R - 1 + a.win < LP - 1 ? f0 + R - 1 + a.win : LP - 1;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const float ntot = seg_allreduce<SEG>(nsum[k], [](float p, float q) { return p + q; });
        if constexpr (!NEAR) {
#pragma unroll
            for (int r = 0; r < R; ++r) hb[k][r] = 0.0f;
            const int row = prow + PAD + k * (LP + PAD);
            if (a.win <= PAD) {
                // Every lane the same count of posts, the pads past the row's
                // ends included (they match no label).
                const int n = R + 2 * a.win, p0 = row + f0 - a.win;
                for (int i = 0; i < n; ++i) {
                    const float pv = s_pv[p0 + i];
                    const int wv = s_pw[p0 + i];
#pragma unroll
                    for (int r = 0; r < R; ++r)
                        if (wv == f0 + r) hb[k][r] += pv;
                }
            } else {
                for (int f = lo; f <= hi; ++f) {
                    const float pv = s_pv[row + f];
                    const int d = (int)s_pw[row + f] - f0;
#pragma unroll
                    for (int r = 0; r < R; ++r)
                        if (d == r) hb[k][r] += pv;
                }
            }
        }
#pragma unroll
        for (int r = 0; r < R; ++r) hb[k][r] -= gmin[k] == (float)r ? ntot : 0.0f;
    }

    // Sender side: cost-bar += sum over messages; slot k's adjoint gets the
    // other three messages' h-bar, added to the readout adjoint at the first
    // reverse step and written over the consumed value afterwards.
    float tot[R];
#pragma unroll
    for (int r = 0; r < R; ++r) tot[r] = (hb[0][r] + hb[1][r]) + (hb[2][r] + hb[3][r]);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        float cur[R];
#pragma unroll
        for (int r = 0; r < R; ++r) cur[r] = tot[r] - hb[k][r];
        if (a.first) {
#pragma unroll
            for (int r = 0; r < R; ++r) cur[r] += gc[r];
        }
        st_row<StoreF32, R>(rb, has[k] ? (mb4 + (uint32_t)k * a.blk + base) * 4u : kNoRow, cur);
    }
#pragma unroll
    for (int r = 0; r < R; ++r) gc[r] += tot[r];
    st_row<StoreF32, R>(rg, goff, gc);

    // Block sums of the lambda and tau partials: per wavefront by shuffles,
    // then the four wavefronts in order.
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        lsum += __shfl_xor(lsum, o, 64);
        tsum += __shfl_xor(tsum, o, 64);
    }
    if (threadIdx.x % 64 == 0) {
        s_part[threadIdx.x / 64][0] = lsum;
        s_part[threadIdx.x / 64][1] = tsum;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        a.partial[2 * block] = ((s_part[0][0] + s_part[1][0]) + s_part[2][0]) + s_part[3][0];
        a.partial[2 * block + 1] = ((s_part[0][1] + s_part[1][1]) + s_part[2][1]) + s_part[3][1];
    }
}

struct BwdPmEntry {
    BwdPmArgs a;
    int block0;
    int pad[3];
};
constexpr int kBwdPmChunk = 16;
struct BwdPmChunk {
    BwdPmEntry e[kBwdPmChunk];
    int n;
};

// The reverse half-sweep of several problems (same lane split) in one
// launch, their arguments passed by value: block b belongs to the last entry
// whose first block is <= b.
template <int SEG, int R, bool NEAR>
__global__ void __launch_bounds__(256) k_bwd_step_pm_batch(const BwdPmChunk c)
{
    int i = 0;
    while (i + 1 < c.n && c.e[i + 1].block0 <= (int)blockIdx.x) ++i;
    bwd_step_pm<SEG, R, NEAR>(c.e[i].a, blockIdx.x - (uint32_t)c.e[i].block0);
}

// Readout adjoint on pixel-major states: b = cost + the four incoming rows
// (summed as the forward readout sums them), d = sum f p_f with p =
// softmax(-b / T); b-bar(f) = -(g / T) p_f (f - d).  Initialises the cost
// adjoint; every incoming slot's adjoint is its pixel's b-bar too, and the
// first reverse step reads it there (writing the eight slot rows per pixel
// pair as well: 34 against 23 us at 320 x 240 x 64).  Memory bound.  Grid
// (ncomp * SEG / 256, 2 colours).
template <int SEG, int R>
__global__ void __launch_bounds__(256) k_bwd_readout_pm(const float *__restrict__ cost, uint32_t cost_bytes,
                                                       const uint8_t *__restrict__ msg, uint32_t msg_bytes,
                                                       float *__restrict__ gcost,
                                                       const float *__restrict__ grad_soft, PmDesc d, int L,
                                                       float inv_t)
{
    const int c = blockIdx.y;
    const int gid = blockIdx.x * 256 + threadIdx.x;
    const int j = gid / SEG, s = gid % SEG;
    if (j >= d.h * d.wh) return;
    const int y = j / d.wh;
    const int x = 2 * (j - y * d.wh) + ((y + c) & 1);
    if (x >= d.w) return;
    const __amdgpu_buffer_rsrc_t rc = make_rsrc(cost, cost_bytes);
    const __amdgpu_buffer_rsrc_t rm = make_rsrc(msg, msg_bytes);
    const __amdgpu_buffer_rsrc_t rg = make_rsrc(gcost, cost_bytes);
    const int f0 = s * R;
    const uint32_t lp = (uint32_t)d.lp, blk = (uint32_t)d.blk;
    const uint32_t base = (uint32_t)j * lp + (uint32_t)f0;
    float b[R], m[4][R];
    ld_row<StoreF32, R>(rc, ((uint32_t)c * blk + base) * 4u, b);
#pragma unroll
    for (int k = 0; k < 4; ++k) ld_row<StoreF32, R>(rm, (((uint32_t)c * 4u + (uint32_t)k) * blk + base) * 4u, m[k]);
    const float inf = __builtin_huge_valf();
    float bmin = inf;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        b[r] = (((b[r] + m[0][r]) + m[1][r]) + m[2][r]) + m[3][r];
        if (f0 + r >= L) b[r] = inf;
        bmin = fminf(bmin, b[r]);
    }
    bmin = seg_allreduce<SEG>(bmin, [](float p, float q) { return fminf(p, q); });
    float wgt[R], num = 0.0f, den = 0.0f;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        wgt[r] = f0 + r < L ? expf(-(b[r] - bmin) * inv_t) : 0.0f;
        num += (float)(f0 + r) * wgt[r];
        den += wgt[r];
    }
    auto add = [](float p, float q) { return p + q; };
    num = seg_allreduce<SEG>(num, add);
    den = seg_allreduce<SEG>(den, add);
    const float dd = num / den;
    const float g = grad_soft[(int64_t)y * d.w + x];
    float bb[R];
#pragma unroll
    for (int r = 0; r < R; ++r) bb[r] = f0 + r < L ? -g * inv_t * (wgt[r] / den) * ((float)(f0 + r) - dd) : 0.0f;
    st_row<StoreF32, R>(rg, ((uint32_t)c * blk + base) * 4u, bb);
}

// Pixel-major cost adjoint -> planar [L][h][w] output with 16-byte accesses
// both ways: a block moves 64 pixels of one row x 64 labels through LDS,
// loading four consecutive labels of one pixel per lane (a pixel's labels are
// contiguous) and storing four consecutive pixels of one label.  ALIGNED:
// w % 4 == 0 and a 16-byte aligned output; else the stores are 4-byte aligned
// and a row's last pixels go one by one (319 x 240 x 64: 11.8 us against 18.9
// with 4-byte accesses).  Memory bound.  grid (w / 64, h, L / 64).
template <bool ALIGNED>
__global__ void __launch_bounds__(256) k_gcost_to_planar4(const float *__restrict__ gcost, PmDesc d, int L,
                                                         float *__restrict__ out)
{
    __shared__ float tile[64][65];
    const int x0 = blockIdx.x * 64, y = blockIdx.y, f0 = blockIdx.z * 64;
    const int t = threadIdx.x, q = t & 15, r = t >> 4;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int xl = r + 16 * i, x = x0 + xl, f = f0 + 4 * q;
        float4 v = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        if (x < d.w && f < L) {
            const int c = (x + y) & 1;
            v = *(const float4 *)(gcost + (int64_t)c * d.blk + ((int64_t)y * d.wh + (x >> 1)) * d.lp + f);
        }
        tile[4 * q][xl] = v.x;
        tile[4 * q + 1][xl] = v.y;
        tile[4 * q + 2][xl] = v.z;
        tile[4 * q + 3][xl] = v.w;
    }
    __syncthreads();
    const int64_t plane = (int64_t)d.h * d.w;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int fl = r + 16 * i, f = f0 + fl, x = x0 + 4 * q;
        const float4 v = make_float4(tile[fl][4 * q], tile[fl][4 * q + 1], tile[fl][4 * q + 2], tile[fl][4 * q + 3]);
        float *o = out + f * plane + (int64_t)y * d.w + x;
        if constexpr (ALIGNED) {
            if (f < L && x < d.w) *(float4 *)o = v;
        } else if (f < L && x + 3 < d.w) {
            __builtin_memcpy(o, &v, 16);
        } else if (f < L && x < d.w) {
            o[0] = v.x;
            if (x + 1 < d.w) o[1] = v.y;
            if (x + 2 < d.w) o[2] = v.z;
        }
    }
}

int bwd_pm_blocks(const Plan &p)
{
    int S, R;
    pm_split(p.L, &S, &R);
    return (int)(((int64_t)p.lv[0].h * p.lv[0].wh * S + 255) / 256);
}

bp_status launch_bwd_readout_pm(const Plan &p, const uint8_t *msg, float *gcost, const float *grad_soft, float temperature,
                                uint8_t *ws, hipStream_t s)
{
    const Level &v = p.lv[0];
    const int64_t ncomp = (int64_t)v.h * v.wh;
    int S, R;
    pm_split(p.L, &S, &R);
    const float *cost = (const float *)(ws + v.cost_off);
    const float inv_t = 1.0f / temperature;
#define BP_RPM(SV, RV)                                                                                             \
    if (S == SV && R == RV) {                                                                                      \
        k_bwd_readout_pm<SV, RV><<<dim3((unsigned)((ncomp * SV + 255) / 256), 2), 256, 0, s>>>(                    \
            cost, (uint32_t)v.cost_bytes, msg, (uint32_t)v.msg_bytes, gcost, grad_soft, pm_desc(v), p.L, inv_t); \
        return launch_status();                                                                                    \
    }
    BP_RPM(4, 4) BP_RPM(8, 4) BP_RPM(16, 4) BP_RPM(16, 6) BP_RPM(16, 8)
#undef BP_RPM
    return BP_ERR_UNSUPPORTED;
}

bp_status launch_gcost_to_planar(const Plan &p, const float *gcost, float *grad_cost, hipStream_t s)
{
    const Level &v = p.lv[0];
    const dim3 grid((unsigned)((v.w + 63) / 64), (unsigned)v.h, (unsigned)((p.L + 63) / 64));
    if (v.w % 4 == 0 && ((uintptr_t)grad_cost % 16) == 0)
        k_gcost_to_planar4<true><<<grid, 256, 0, s>>>(gcost, pm_desc(v), p.L, grad_cost);
    else
        k_gcost_to_planar4<false><<<grid, 256, 0, s>>>(gcost, pm_desc(v), p.L, grad_cost);
    return launch_status();
}

// The near form's condition: untruncated winners within kNear labels.
static bool bwd_near(float lambda, int win) { return lambda > 0.0f && win <= kNear; }

bp_status launch_bwd_step_pm_batch(const BwdPmProblem *probs, int count, int t, bool first_step, float lambda,
                                   float tau, hipStream_t s)
{
    bool *done = new bool[count]();
    bp_status st = BP_OK;
    // Launches of up to kBwdPmChunk problems of one lane split (the kernel's
    // template arguments) and window.
    for (int i = 0; i < count && st == BP_OK; ++i) {
        if (done[i]) continue;
        int S, R;
        pm_split(probs[i].plan->L, &S, &R);
        bool near = false;
        int blocks = 0;
        BwdPmChunk c;
        c.n = 0;
        for (int k = i; k < count && c.n < kBwdPmChunk; ++k) {
            int Sk, Rk;
            pm_split(probs[k].plan->L, &Sk, &Rk);
            if (done[k] || Sk != S || Rk != R) continue;
            done[k] = true;
            const Plan &p = *probs[k].plan;
            const Level &v = p.lv[0];
            BwdPmEntry &e = c.e[c.n++];
            BwdPmArgs &a = e.a;
            a.cost = (const float *)(probs[k].ws + v.cost_off);
            a.cost_bytes = (uint32_t)v.cost_bytes;
            a.msg = probs[k].state;
            a.msg_bytes = (uint32_t)v.msg_bytes;
            a.mbar = probs[k].mbar;
            a.mbar_bytes = (uint32_t)v.msg_bytes;
            a.gcost = probs[k].gcost;
            a.partial = probs[k].partial;
            a.w = v.w;
            a.h = v.h;
            a.wh = v.wh;
            a.blk = (uint32_t)v.blk;
            a.lp = (uint32_t)v.lp;
            a.colour = t & 1;
            a.L = p.L;
            a.ncomp = v.h * v.wh;
            // Untruncated winners lie within tau of their label; two labels of
            // margin cover rounding.  Without smoothness any label can win.
            a.win = lambda > 0.0f ? (int)std::min((float)(v.lp - 1), std::floor(tau) + 2.0f) : v.lp - 1;
            near = bwd_near(lambda, a.win);               // the same for a lane split
            a.first = first_step ? 1 : 0;
            a.lambda = lambda;
            a.tau = tau;
            a.lt = lambda * tau;
            e.block0 = blocks;
            blocks += bwd_pm_blocks(p);
        }
#define BP_BPM(SV, RV)                                                                                             \
    if (S == SV && R == RV) {                                                                                      \
        if (near) k_bwd_step_pm_batch<SV, RV, true><<<blocks, 256, 0, s>>>(c);                                     \
        else k_bwd_step_pm_batch<SV, RV, false><<<blocks, 256, 0, s>>>(c);                                         \
        st = launch_status();                                                                                      \
        continue;                                                                                                  \
    }
        BP_BPM(4, 4) BP_BPM(8, 4) BP_BPM(16, 4) BP_BPM(16, 6) BP_BPM(16, 8)
#undef BP_BPM
        st = BP_ERR_UNSUPPORTED;
    }
    delete[] done;
    return st;
}

}  // namespace bpk
