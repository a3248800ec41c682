// a5, pixel-major levels: T = 2P consecutive checkerboard half-sweeps
// (t .. t + T - 1, t even) in one launch, streaming down the rows of a strip.
//
// Half-sweep t + 1 reads only what half-sweep t wrote next to it, so a block
// that owns a strip of columns can run T half-sweeps ("stages" 1 .. T) over it
// in one pass down the rows, stage s two rows behind stage s - 1: at step n,
// stage s is at row n - 2 (s - 1) of the segment.  Memory then carries one
// colour-0 state in and one out per T half-sweeps (and the cost once per
// stage, which the caches serve after the first), against one in and out per
// two half-sweeps for the tiled pair (bp_iter_pm2_impl.h).
//
// A lane group (SEG lanes, R labels each) keeps one column.  At a step the
// columns of one parity have their odd stages' pixels in the current rows and
// those of the other parity their even stages'; a wave holds columns of one
// parity (every second column), so which stages it runs is uniform, and half
// the waves read memory (stage 1) while the other half write it (stage T).
// Messages up and down go to the same column, so they stay in registers
// between stages (`up` for the pixel above, handled at the next step; `dn` and
// the older `dd` for the one below, handled three steps on); messages left and
// right go to the neighbouring columns' lane groups through LDS, one row per
// stage boundary, column and side.  A row that stage s writes in step n is read
// by its owner at the end of step n + 1, for stage s + 1 in step n + 2, and
// written again in step n + 2.  One barrier closes each step, so the read of a
// row lies between two barriers with neither of its writes.
//
// Edges: with NS stages (T, and one more in a launch that reads out both
// colours) a strip's block carries NS - 1 more columns on each side and a
// segment NS - 1 more rows, and stage s covers the strip and segment plus
// NS - s; what lies beyond is garbage that no covered pixel reads.  Only stage
// T writes the state (none does where both colours are read out), and each
// slot of colour 0 has one writer.  As in the tiled
// pair colour 0's incoming rows are double-buffered (`src`, `dst`), the first
// launch of a level reads the parent level's state or zeros, and the launch
// that ends a level stores colour 1's incoming rows (write_c1), which stage T
// holds as its inputs.
//
// What bounds it, by counters (VALU instructions against the 614 G wavefront
// instructions a second of the nominal clock; HBM bytes): with four labels per
// lane instruction issue (676 x 380 x 64, byte costs: .72 to .74 of the slots, .82
// to .88 of those in the CUs' busy cycles, 2.7 to 2.9 TB/s; about 150 VALU
// instructions per visit of four pixels), with eight and 16-bit rows too (1352 x
// 760 x 128, five labels: .80 and .96, 3.7 TB/s); with eight and FP32 rows issue
// and memory together (.58 and .71, 4.6 TB/s; levels 1 and 2, FP32 costs, .32 to
// .51 and 4.8 to 6.1 TB/s).  A step's loads are issued two steps (stage 1) or one
// step (costs) ahead, without branches, so that the compiler's waits count
// just them; before that, waits for whole queues (stores included) took half
// the time (1352 x 760 x 128: 2.11 against 1.43 ms for its six pairs).
// Measured, level 0, FP32 rows, integer costs: 676 x 380 x 64, five pairs: 296
// (tiled) -> 162 us; 1352 x 760 x 128, six pairs: 2928 -> 1427 us; in bfloat16
// with the five-label form 2652 -> 1743 us.
//
// Messages are rounded to the storage format where the one-half-sweep kernel
// stores them, and the arithmetic per message is that kernel's variant 1
// (bp_pm_core.h), so results are equal bit for bit; with the five-label form
// above four labels per lane, whose results are the scans' while h stays below
// about 2^18 lambda (pm_transform_near2_scans), up to roundings of h beyond.
#pragma once

#include <hip/hip_runtime.h>

#include "bp_device.h"
#include "bp_internal.h"
#include "bp_iter_stream.h"
#include "bp_pm_core.h"

namespace bpk {

#define BP_INLINE __attribute__((always_inline))

// Words of a lane's R values as stored: messages (S) and cost (CF).
template <typename S, int R>
constexpr int msg_words = S::bytes == 4 ? R : R / 2;
template <int R, int CF>
constexpr int cost_words = CF == COST_U8 ? R / 4 : CF == COST_F16 ? R / 2 : R;

template <typename S, int R>
__device__ __forceinline__ void unpack_row(const uint32_t (&w)[msg_words<S, R>], float (&v)[R])
{
    if constexpr (S::bytes == 4) {
#pragma unroll
        for (int i = 0; i < R; ++i) v[i] = __builtin_bit_cast(float, w[i]);
    } else {
#pragma unroll
        for (int i = 0; i < R / 2; ++i) {
            v[2 * i] = S::decode((uint16_t)(w[i] & 0xffffu));
            v[2 * i + 1] = S::decode((uint16_t)(w[i] >> 16));
        }
    }
}

template <typename S, int R>
__device__ __forceinline__ void pack_row(const float (&v)[R], uint32_t (&w)[msg_words<S, R>])
{
    if constexpr (S::bytes == 4) {
#pragma unroll
        for (int i = 0; i < R; ++i) w[i] = __builtin_bit_cast(uint32_t, v[i]);
    } else {
#pragma unroll
        for (int i = 0; i < R / 2; ++i) w[i] = S::pack2(v[2 * i], v[2 * i + 1]);
    }
}

template <int R, int CF>
__device__ __forceinline__ void unpack_cost(const uint32_t (&w)[cost_words<R, CF>], float (&v)[R])
{
    if constexpr (CF == COST_U8) {
#pragma unroll
        for (int i = 0; i < R / 4; ++i)
#pragma unroll
            for (int b = 0; b < 4; ++b) v[4 * i + b] = (float)((w[i] >> (8 * b)) & 255u);
    } else if constexpr (CF == COST_F16) {
        unpack_row<StoreF16, R>(w, v);
    } else {
        unpack_row<StoreF32, R>(w, v);
    }
}

template <int R, int CF>
constexpr uint32_t cost_bytes_of = CF == COST_U8 ? 1u : CF == COST_F16 ? 2u : 4u;

// Exchange row of one lane group in LDS: chunk q (16, 8 or 4 bytes) of a
// lane's words next to the other lanes' chunk q, so that a wave's accesses are
// consecutive.
template <int W>
struct Chunk {
    typedef uint32_t type;
    static constexpr int words = 1;
};
template <>
struct Chunk<4> {
    typedef u32x4 type;
    static constexpr int words = 4;
};
template <>
struct Chunk<2> {
    typedef u32x2 type;
    static constexpr int words = 2;
};
template <int W>
using chunk_of = Chunk<(W % 4 == 0 ? 4 : W % 2 == 0 ? 2 : 1)>;

template <int SEG, int W>
__device__ __forceinline__ void lds_put(uint32_t *row, int s, const uint32_t (&w)[W])
{
    using C = chunk_of<W>;
    typename C::type *p = (typename C::type *)row + s;
#pragma unroll
    for (int q = 0; q < W / C::words; ++q) {
        if constexpr (C::words == 1) {
            p[q * SEG] = w[q];
        } else {
            typename C::type t;
#pragma unroll
            for (int e = 0; e < C::words; ++e) t[e] = w[q * C::words + e];
            p[q * SEG] = t;
        }
    }
}

template <int SEG, int W>
__device__ __forceinline__ void lds_get(const uint32_t *row, int s, uint32_t (&w)[W])
{
    using C = chunk_of<W>;
    const typename C::type *p = (const typename C::type *)row + s;
#pragma unroll
    for (int q = 0; q < W / C::words; ++q) {
        const typename C::type t = p[q * SEG];
        if constexpr (C::words == 1) {
            w[q] = t;
        } else {
#pragma unroll
            for (int e = 0; e < C::words; ++e) w[q * C::words + e] = t[e];
        }
    }
}

// Byte offset past every row: loads there return zero and stores are dropped,
// so that a step's memory operations need no branches (the compiler can then
// count them and wait for just the ones it needs).
constexpr uint32_t kNowhere = 0xffffff00u;

// END: 0 a launch inside a level; 1 its last one, which stores colour 1's
// incoming rows; 2 the finest level's last one, which reads out colour 1 (and
// stores its rows when asked); 3 the same where nothing reads the final state:
// it reads out colour 0 too, in one more stage, and stores labels only (a
// readout pass reads colour 0's state and costs: 21 us at 676 x 380 x 64 and
// 215 at 1352 x 760 x 128, in FP32).  The extra stage's registers spill a few in
// some forms (three pairs at 16 and 32 labels, FP32 costs at 128 labels with
// tau > 2) and it is the faster end there too: whole calls at 1352 x 760, two
// levels, against the pass, FP32 at 16 .. 128 labels and tau 2 .. 5 .78 to .95 of the
// time, bfloat16 .95 to 1.00.
template <int SEG, int R, typename S, int P, int NW, int CF, int NEAR, int END>
__global__ void __launch_bounds__(NW * 64) k_iter_stream(const PairArgs a)
{
    constexpr int T = 2 * P, NS = END == 3 ? T + 1 : T, H = NS - 1;   // half-sweeps, stages, columns repeated
    constexpr int PO = END == 3 ? P + 1 : P;             // odd stages
    constexpr int CPW = 64 / SEG, NC = NW * CPW;         // columns per wave and per block
    constexpr int MW = msg_words<S, R>, CW = cost_words<R, CF>;
    constexpr uint32_t CB = cost_bytes_of<R, CF>, MB = S::bytes;
    constexpr int ROW = SEG * MW;                        // words of an exchange row
    constexpr int BND = NC * 2 * ROW;                    // words of a boundary's exchange rows
    extern __shared__ __attribute__((aligned(16))) uint32_t xch[];                    // [NS - 1 boundaries][NC][2 sides][ROW]

    // Tile of the block: consecutive tiles per XCD (blocks b, b + 8, ... run
    // on one), strips fastest, so that neighbours' shared columns meet in
    // its L2.
    const int tile = ((int)blockIdx.x & 7) * a.per_xcd + ((int)blockIdx.x >> 3);
    if (tile >= a.ntiles) return;
    const int strip = tile % a.tiles_x, seg = tile / a.tiles_x;
    const int xs = strip * a.tx, xe = min(a.w, xs + a.tx);
    const int ya = seg * a.ty, yb = min(a.h, ya + a.ty);
    const int x0 = max(0, xs - H);
    const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int lane = (int)threadIdx.x & 63, s = lane % SEG, f0 = s * R;
    const int col = (wv >> 1) * (2 * CPW) + 2 * (lane / SEG) + (wv & 1);
    const int x = x0 + col;
    const bool in_x = x < a.w, out_x = x >= xs && x < xe;
    const bool has_l = x > 0 && in_x, has_r = x < a.w - 1;
    const uint32_t lp = a.lp;

    // Rows of stage st (1-based): the segment and NS - st more on each side.
    auto row_on = [&](int st, int y) BP_INLINE { return y >= max(0, ya - (NS - st)) && y < min(a.h, yb + (NS - st)); };

    // Bytes of a pixel row of one colour (and slot) of the cost, the level's
    // states and the source state, and of a colour-and-slot block of each.
    const uint32_t crow = (uint32_t)a.wh * a.lp * CB, mrow = (uint32_t)a.wh * a.lp * MB;
    const uint32_t srow = a.src_parent ? (uint32_t)a.src_wh * a.sps * MB : mrow;
    const uint32_t cblk = a.blk * CB, mblk = a.blk * MB, sblk = a.sblk * MB;
    // `on`: the row is there; otherwise a descriptor that no lane's offset is
    // inside.
    auto row_at = [&](const void *base, uint32_t off, uint32_t bytes, bool on) BP_INLINE {
        return make_rsrc((const uint8_t *)base + off, on ? bytes : 0u);
    };

    // Lane offsets in a row, kNowhere where the column has no such pixel.
    const uint32_t xoff = (uint32_t)(x >> 1) * a.lp + (uint32_t)f0;
    const uint32_t vcost = in_x ? xoff * CB : kNowhere;
    // Source rows: the pixel's own, or the parent pixel's, whose colour also
    // depends on the parent row's parity (index of rd_v).
    const uint32_t sx = (uint32_t)(x >> 1), pv = a.src_parent ? ((sx >> 1) * a.sps + (uint32_t)f0) * MB : xoff * MB;
    const uint32_t pblk = a.src_parent ? 4u * sblk : 0u;
    const uint32_t rd_v[2] = {pv + ((sx & 1u) ? pblk : 0u), pv + ((sx & 1u) ? 0u : pblk)};
    const uint32_t wr_c = out_x ? xoff * MB : kNowhere;
    const uint32_t wr_l = out_x && has_l ? ((uint32_t)((x - 1) >> 1) * a.lp + (uint32_t)f0) * MB : kNowhere;
    const uint32_t wr_r = out_x && has_r ? ((uint32_t)((x + 1) >> 1) * a.lp + (uint32_t)f0) * MB : kNowhere;
    // A row's offset as the compiler may not take apart: otherwise it forms
    // every word's offset on its own ahead of the loop, which splits the
    // 16-byte accesses.
    auto whole = [](uint32_t v) BP_INLINE {
        asm volatile("" : "+v"(v));
        return v;
    };

    // Cost row of the column's pixel at row y, colour c (stage st's).
    auto load_cost = [&](auto check, int c, int st, int y, uint32_t (&w)[CW]) BP_INLINE {
        const bool on = !decltype(check)::value || row_on(st, y);
        ld_words<CW>(row_at(a.cost, (uint32_t)c * cblk + (uint32_t)y * crow, crow, on), whole(vcost), w);
    };
    // Stage 1's inputs at row y: the cost row and the four incoming rows of
    // the source state.  Slots from outside the grid are zero and not read.
    auto load_stage1 = [&](auto check, int y, uint32_t (&cw)[CW], uint32_t (&mw)[4][MW]) BP_INLINE {
        constexpr bool CHECK = decltype(check)::value;
        load_cost(check, 0, 1, y, cw);
        const bool on = !a.src_zero && (!CHECK || row_on(1, y));
        const bool row_k[4] = {on, on, on && (!CHECK || y > 0), on && (!CHECK || y < a.h - 1)};
        const int sy = a.src_parent ? y >> 1 : y;
        const uint32_t v = rd_v[sy & 1];
        const uint32_t lanes[4] = {has_l ? v : kNowhere, has_r ? v : kNowhere, in_x ? v : kNowhere,
                                   in_x ? v : kNowhere};
#pragma unroll
        for (int k = 0; k < 4; ++k)
            ld_words<MW>(row_at(a.src, (uint32_t)k * sblk + (uint32_t)sy * srow, pblk + srow, row_k[k]),
                         whole(lanes[k]), mw[k]);
    };

    uint32_t *const my_row = xch + (col * 2) * ROW;      // + boundary * BND + side * ROW

    // Messages held between stages b + 1 and b + 2, as stored.
    uint32_t up[NS - 1][MW], dn[NS - 1][MW], dd[NS - 1][MW];
#pragma unroll
    for (int b = 0; b < NS - 1; ++b)
#pragma unroll
        for (int i = 0; i < MW; ++i) up[b][i] = dn[b][i] = dd[b][i] = 0u;

    // One pixel of stage ST: its four messages from its cost and incoming rows.
    auto visit = [&](auto st_tag, auto check, int y, const uint32_t (&cw)[CW], const uint32_t (&mw)[4][MW]) BP_INLINE {
        constexpr int ST = decltype(st_tag)::value;
        constexpr bool CHECK = decltype(check)::value;
        float c[R], m[4][R];
        unpack_cost<R, CF>(cw, c);
#pragma unroll
        for (int k = 0; k < 4; ++k) unpack_row<S, R>(mw[k], m[k]);
        const bool has_u = !CHECK || y > 0, has_d = !CHECK || y < a.h - 1;
        if constexpr (ST >= T && END >= 2) {
            // Labels of the row's columns (no label array, no row); lane 0 of
            // a column stores them.
            float bel[R], sv;
            int bi;
            pm_belief<R>(c, m, bel);
            pm_readout<SEG, R, true>(bel, f0, a.L, a.soft != nullptr, a.inv_t, bi, sv);
            const uint32_t row = ST == NS || (y >= ya && y < yb) ? (uint32_t)a.w * 4u : 0u;
            const uint32_t at = out_x && s == 0 ? (uint32_t)x * 4u : kNowhere;
            __builtin_amdgcn_raw_buffer_store_b32((uint32_t)bi, make_rsrc(a.disp + (size_t)y * a.w, a.disp ? row : 0u),
                                                  at, 0, 0);
            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, sv),
                                                  make_rsrc(a.soft + (size_t)y * a.w, a.soft ? row : 0u), at, 0, 0);
        }
        if constexpr (ST == NS && END == 3) return;
        if constexpr (ST == T && (END == 1 || END == 2)) {
            const uint32_t lanes[4] = {has_l ? wr_c : kNowhere, has_r ? wr_c : kNowhere, wr_c, wr_c};
            const bool has[4] = {true, true, has_u, has_d};
#pragma unroll
            for (int k = 0; k < 4; ++k)
                st_words<MW>(row_at(a.msg, (uint32_t)(4 + k) * mblk + (uint32_t)y * mrow, mrow, a.write_c1 && has[k]),
                             whole(lanes[k]), mw[k]);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            float h[R], o[R];
            uint32_t w[MW];
            pm_h<R>(c, m, k, h);
            pm_transform<SEG, R, true, NEAR>(h, s, f0, a.L, a.lambda, a.lt, o);
            pack_row<S, R>(o, w);
            if constexpr (ST == NS) {
                const int ny = k == 2 ? y - 1 : k == 3 ? y + 1 : y;
                const bool has = k == 2 ? has_u : k == 3 ? has_d : true;
                st_words<MW>(row_at(a.dst, (uint32_t)(k ^ 1) * mblk + (uint32_t)ny * mrow, mrow, has),
                             whole(k == 0 ? wr_l : k == 1 ? wr_r : wr_c), w);
            } else if (k == 0) {
                if (col > 0 && in_x) lds_put<SEG, MW>(my_row + (ST - 1) * BND - ROW, s, w);    // column - 1, side 1
            } else if (k == 1) {
                if (col < NC - 1) lds_put<SEG, MW>(my_row + (ST - 1) * BND + 2 * ROW, s, w);   // column + 1, side 0
            } else if (k == 2) {
#pragma unroll
                for (int i = 0; i < MW; ++i) up[ST - 1][i] = w[i];
            } else {
#pragma unroll
                for (int i = 0; i < MW; ++i) dn[ST - 1][i] = w[i];
            }
        }
    };

    // Stage 1's rows of the next odd step; the costs and the left and right
    // rows of the next step's later stages.
    uint32_t c1[CW], m1[4][MW], cn[PO][CW], l[PO][MW], r[PO][MW];

    // One step of the wave at row y1: odd stages (1, 3, ...) or even ones,
    // the later ones first, so that stage T's stores are long issued when
    // stage 1 waits for its loads.  CHECK: some row of the step or of its loads
    // ahead may lie outside its range or on the grid's first or last row.
    auto step = [&](auto odd_tag, auto check, int y1) BP_INLINE {
        constexpr bool ODD = decltype(odd_tag)::value, CHECK = decltype(check)::value;
        uint32_t cc[PO][CW];
#pragma unroll
        for (int q = 0; q < PO; ++q)
#pragma unroll
            for (int i = 0; i < CW; ++i) cc[q][i] = cn[q][i];
        // Costs of the next step's later stages.
#pragma unroll
        for (int q = ODD ? 0 : 1; q < (ODD ? P : PO); ++q)
            load_cost(check, ODD ? 1 : 0, ODD ? 2 * q + 2 : 2 * q + 1, y1 + 1 - (ODD ? 4 * q + 2 : 4 * q), cn[q]);
        // Stage 2q + 1 (odd steps) or 2q + 2.
        auto later = [&](auto q_tag) BP_INLINE {
            constexpr int q = decltype(q_tag)::value, ST = ODD ? 2 * q + 1 : 2 * q + 2, b = ST - 2;
            const int y = y1 - 2 * (ST - 1);
            if constexpr (ST < NS) {
#pragma unroll
                for (int i = 0; i < MW; ++i) dd[ST - 1][i] = dn[ST - 1][i];
            }
            if (CHECK && !row_on(ST, y)) return;
            // Left and right from LDS, up and down from the column's
            // registers; zero outside the grid (left and right: rows of LDS
            // that are cleared once and never written).
            uint32_t mw[4][MW];
#pragma unroll
            for (int i = 0; i < MW; ++i) {
                mw[0][i] = l[q][i];
                mw[1][i] = r[q][i];
                mw[2][i] = CHECK && y <= 0 ? 0u : dd[b][i];
                mw[3][i] = CHECK && y >= a.h - 1 ? 0u : up[b][i];
            }
            visit(std::integral_constant<int, ST>{}, check, y, cc[q], mw);
        };
        if constexpr (ODD && PO > P) later(std::integral_constant<int, P>{});
        if constexpr (P > 2) later(std::integral_constant<int, (P > 2 ? 2 : 1)>{});
        if constexpr (P > 1) later(std::integral_constant<int, (P > 1 ? 1 : 0)>{});
        if constexpr (ODD) {
#pragma unroll
            for (int i = 0; i < MW; ++i) dd[0][i] = dn[0][i];
            if (!CHECK || row_on(1, y1)) visit(std::integral_constant<int, 1>{}, check, y1, c1, m1);
            load_stage1(check, y1 + 2, c1, m1);
        } else {
            later(std::integral_constant<int, 0>{});
        }
        // Rows of the next step's later stages: written in the step before
        // this one, and written again only in the next one.
#pragma unroll
        for (int q = ODD ? 0 : 1; q < (ODD ? P : PO); ++q) {
            const uint32_t *row = my_row + (ODD ? 2 * q : 2 * q - 1) * BND;
            lds_get<SEG, MW>(row, s, l[q]);
            lds_get<SEG, MW>(row + ROW, s, r[q]);
        }
        __syncthreads();
    };
    using Odd = std::true_type;
    using Even = std::false_type;
    using Check = std::true_type;
    using Free = std::false_type;

    // Rows that no column writes (beyond the grid, and the block's first and
    // last column) read as zero.
    for (int i = (int)threadIdx.x; i < (NS - 1) * BND; i += NW * 64) xch[i] = 0u;
    __syncthreads();

    // Steps ybeg .. ybeg + n - 1 (n even), in twos of an odd and an even step;
    // the waves whose first step is an even one start and end with one alone.
    const int ybeg = max(0, ya - H);
    const int n = (yb - 1 + 2 * (NS - 1) - ybeg + 2) & ~1, yend = ybeg + n;
    const bool odd_first = (((x0 + (wv & 1)) + ybeg) & 1) == 0;
#pragma unroll
    for (int q = 0; q < PO; ++q)
#pragma unroll
        for (int i = 0; i < CW; ++i) cn[q][i] = 0u;
#pragma unroll
    for (int q = 0; q < PO; ++q)
#pragma unroll
        for (int i = 0; i < MW; ++i) l[q][i] = r[q][i] = 0u;
    int y1 = ybeg;
    load_stage1(Check{}, odd_first ? y1 : y1 + 1, c1, m1);
    if (!odd_first) step(Even{}, Check{}, y1++);
    // In steps [free_lo, free_hi) every stage's row, and stage 1's two steps
    // ahead, is in its range and inside the grid.
    const int free_lo = max(ya, 1) + 2 * (NS - 1), free_hi = min(a.h - 1, yb + H) - 2;
#pragma unroll 1
    while (y1 + 1 < yend && y1 < free_lo) {
        step(Odd{}, Check{}, y1);
        step(Even{}, Check{}, y1 + 1);
        y1 += 2;
    }
    __builtin_amdgcn_s_waitcnt(0);
#pragma unroll 1
    while (y1 + 1 < free_hi) {
        step(Odd{}, Free{}, y1);
        step(Even{}, Free{}, y1 + 1);
        y1 += 2;
    }
#pragma unroll 1
    while (y1 + 1 < yend) {
        step(Odd{}, Check{}, y1);
        step(Even{}, Check{}, y1 + 1);
        y1 += 2;
    }
    if (y1 < yend) step(Odd{}, Check{}, y1);
}

template <int SEG, int R, typename S, int P, int CF, int NEAR>
static bp_status launch_stream_pairs(const PairArgs &a, hipStream_t st)
{
    constexpr int NW = stream_waves(R), NC = NW * (64 / SEG);
    constexpr size_t row = (size_t)NC * 2 * SEG * msg_words<S, R> * 4, lds = (2 * P - 1) * row;
    static_assert(lds + row <= 160 * 1024, "exchange rows exceed the LDS");
    const unsigned grid = (unsigned)(8 * a.per_xcd);
    if (a.ro0) k_iter_stream<SEG, R, S, P, NW, CF, NEAR, 3><<<grid, NW * 64, lds + row, st>>>(a);
    else if (a.disp || a.soft) k_iter_stream<SEG, R, S, P, NW, CF, NEAR, 2><<<grid, NW * 64, lds, st>>>(a);
    else if (a.write_c1) k_iter_stream<SEG, R, S, P, NW, CF, NEAR, 1><<<grid, NW * 64, lds, st>>>(a);
    else k_iter_stream<SEG, R, S, P, NW, CF, NEAR, 0><<<grid, NW * 64, lds, st>>>(a);
    return launch_status();
}

template <int SEG, int R, typename S, int CF, int NEAR>
static bp_status launch_stream_near(const PairArgs &a, hipStream_t st)
{
    if (a.pairs == 2) return launch_stream_pairs<SEG, R, S, 2, CF, NEAR>(a, st);
    if constexpr (NEAR == 1 && stream_three(R, S::fmt))
        if (a.pairs == 3) return launch_stream_pairs<SEG, R, S, 3, CF, NEAR>(a, st);
    return BP_ERR_UNSUPPORTED;
}

template <int SEG, int R, typename S, int CF>
static bp_status launch_stream_cf(const PairArgs &a, hipStream_t st)
{
    if (a.near == 1) return launch_stream_near<SEG, R, S, CF, 1>(a, st);
    if (a.near == 2) return launch_stream_near<SEG, R, S, CF, 2>(a, st);
    return launch_stream_near<SEG, R, S, CF, 0>(a, st);
}

template <int SEG, int R, typename S>
static bp_status launch_stream_split(const PairArgs &a, hipStream_t st)
{
    if (a.cost_fmt == COST_F32) return launch_stream_cf<SEG, R, S, COST_F32>(a, st);
    if constexpr (R % 4 == 0) {
        if (a.cost_fmt == COST_U8) return launch_stream_cf<SEG, R, S, COST_U8>(a, st);
    } else {
        if (a.cost_fmt == COST_F16) return launch_stream_cf<SEG, R, S, COST_F16>(a, st);
    }
    return BP_ERR_UNSUPPORTED;
}

template <typename S>
bp_status stream_launch(const PairArgs &a, int SEGV, int R, hipStream_t st)
{
#define BP_STREAM(SV, RV) \
    if (SEGV == SV && R == RV) return launch_stream_split<SV, RV, S>(a, st);
    BP_STREAM(4, 4) BP_STREAM(8, 4) BP_STREAM(16, 4) BP_STREAM(16, 6) BP_STREAM(16, 8)
#undef BP_STREAM
    return BP_ERR_UNSUPPORTED;
}

}  // namespace bpk
