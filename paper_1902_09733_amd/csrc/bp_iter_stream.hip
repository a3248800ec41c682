// a5, pixel-major levels: host side of the streamed half-sweeps (the kernel is
// in bp_iter_stream_impl.h, compiled per message storage format in
// bp_iter_stream_f32.hip, _f16.hip and _bf16.hip): which levels use them, the
// strips and segments of a launch, and dispatch by storage format.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "bp_device.h"
#include "bp_internal.h"
#include "bp_iter_stream.h"

namespace bpk {

constexpr int kSlots = 256;   // blocks resident at a time: one per compute unit

// Strips of a w-wide level for blocks of `nc` columns that run `stages` stages
// (half-sweeps, and the readout of colour 0): tx columns with stages - 1 more
// on each side (none beyond the grid), as wide as the block allows.
static int strip_width(int w, int nc, int stages)
{
    const int H = stages - 1;
    for (int n = 1;; ++n) {
        const int t = (w + n - 1) / n;
        if ((n == 1 ? t : n == 2 ? t + H : t + 2 * H) <= nc) return t;
    }
}

// Rows of a segment: the count of segments with the least time in the model
//   rounds of resident blocks x steps of a block,
// where a block of t rows takes t + 3 (stages - 1) steps: short segments repeat
// the rows at their ends and fill the pipeline of stages anew, long ones leave
// compute units idle.
static int segment_rows(int h, int strips, int stages)
{
    const int H = stages - 1, most = std::max(1, std::min(h, 4 * kSlots / strips));
    int64_t best = -1;
    int ty = h;
    for (int k = 1; k <= most; ++k) {
        const int t = (h + k - 1) / k;
        const int64_t blocks = (int64_t)strips * ((h + t - 1) / t);
        const int64_t cost = (blocks + kSlots - 1) / kSlots * (t + 3 * H);
        if (best < 0 || cost < best) {
            best = cost;
            ty = t;
        }
    }
    return ty;
}

// Pairs of half-sweeps per launch for a level (1: the tiled pair).  Streaming
// needs enough pixels to fill the chip with strips of rows: a step of a block
// takes about 0.7 us however few blocks there are, and every segment repeats
// rows and fills its pipeline.  Measured per pair, tiled / two / three pairs
// per launch, FP32 rows, tau 2 (w x h x labels):
//   240 x 135 x 64   (2.1 M values)  10.4 / 11.8 / 12.5 us
//   338 x 190 x 64   (4.1 M)         16.9 / 14.3 / 15.3
//   676 x 380 x 16   (4.1 M)         17.8 / 14.3 / 15.1
//   676 x 380 x 32   (8.2 M)         27.5 / 20.4 / 21.1
//   676 x 380 x 64   (16.4 M)        60.6 / 33.1 / 31.3
//   1352 x 760 x 64  (65.8 M)         244 /  121 /  95
//   480 x 270 x 96   (12.4 M)        41.8 / 27.6 / 27.8
//   676 x 380 x 96   (24.7 M)         101 /   56 /  50
//   1352 x 760 x 128 (132 M)          488 /  258 / (434, spilling)
// with FP16 rows
//   240 x 135 x 128  (4.1 M)         15.4 / 16.8
//   338 x 190 x 64   (4.1 M)         17.5 / 16.0 / 16.6
//   676 x 380 x 64                   46.4 / 39.1 / 36.1
//   480 x 270 x 128  (16.6 M)        44.4 / 38.9 / 43.0
//   1352 x 760 x 128                  384 /  277 /  249
// What a call gains (two levels, K = 8, both cost formats, labels alone, with
// messages, and in batches of six; streamed over tiled, least and most):
//   values               4 M        6 M        8 M       12 M       16 M       32 M
//   tau 2    FP32     .82-1.00   .78-.93    .73-.90   .68-.90    .57-.82    .53-.79
//     FP16, R <= 4    .96-1.09   .91-1.04   .91-.97   .88-.97    .81-.91    .72-.83
//     FP16, R > 4    1.03-1.12   .98-1.05   .95-1.02  .93-.98    .88-.94    .78-.86
//   tau 2.6  FP32     .92-1.09   .84-1.02   .79-.96   .72-.95    .64-.85    .56-.79
//     FP16, R <= 4   1.00-1.17   .96-1.07   .96-1.02  .93-1.00   .86-.95    .75-.87
//     FP16, R > 4    1.02-1.17   .98-1.08   .95-1.05  .96-1.00   .91-.97    .81-.89
//   tau 5    FP32    1.02-1.23   .99-1.16   .92-1.06  .86-1.02   .74-.90    .66-.84
//     FP32, R > 4    1.03-1.14   .96-1.07   .90-1.01  .82-.96    .73-.86    .66-.81
//     FP16           1.06-1.31  1.03-1.17  1.03-1.14 1.00-1.10   .92-1.07   .81-.96
// so two pairs from where that is about 1 (FP16, tau 2, R <= 4: from 4 M values,
// .97-1.03, and 6 M where several problems of a batch share tiled launches,
// 1.02-1.09 at 4 M; R > 4: 353 x 236 x 96, 8.0 M, 141 -> 136 us, 340 x 213 x 96, 7.0
// M, 220 -> 223).  A level under a finer one starts with its state out of the
// caches and gains earlier in 16 bits above four labels per lane, from 6 M, with
// five labels from 8 M (1352 x 760 x 128, six levels, in bfloat16, tau 2.6, its
// 8.2 M level tiled / streamed: 2760 / 2724 us).  The more instructions a message
// takes, the less the memory traffic that streaming saves was what held the
// tiled pair back.  Three pairs, the three-label form alone (elsewhere they spill
// or wait more: 1352 x 760 x 128 in bfloat16, tau 2.6: 438 / 291 / 378 us per
// pair), from 16 M values, and 24 M above four labels per lane: three over two,
// 16 .. 130 M values, with five pairs (one + two + two against three + two) .78 ..
// .97 and with six (three launches against two) .87 .. 1.03, up to 1.08 from 16 to
// 24 M above four labels per lane.
// Label counts that fill the lanes only (16, 32, 64, 96, 128): the others are
// padded to these, and the masks that their padded labels need are not compiled
// into the streamed kernel; above 128 (12 and 16 labels per lane) its messages
// would not fit the registers.
static int stream_pairs(const Level &v, int L, float tau, bool finest, bool shared)
{
    int S, R;
    pm_split(L, &S, &R);
    const int nc = stream_columns(S, R), form = stream_form(R, tau);
    if (L != S * R || nc == 0 || v.layout != PIXEL_MAJOR) return 1;
    if (v.cost_fmt == COST_F16 && R % 4 == 0) return 1;   // those lanes hold byte costs
    const int64_t n = (int64_t)v.w * v.h * v.lp;
    const bool f32 = v.fmt == FMT_F32;
    const int64_t two = form == 1 ? (f32 ? 4000000 : R > 4 ? (finest ? 7500000 : 6000000) : finest && shared ? 6000000 : 4000000)
                      : form == 2 ? (f32 || R <= 4 || !finest ? 8000000 : 10000000)
                                  : (!f32 ? 32000000 : R <= 4 ? 12000000 : 8000000);
    if (v.w < 2 * nc || v.h < 64 || n < two) return 1;
    return form == 1 && stream_three(R, v.fmt) && n >= (R <= 4 ? 16000000 : 24000000) ? 3 : 2;
}

PairSchedule pair_schedule(const Plan &p, int l, int np, float tau, bool saves, bool even_count, bool shared)
{
    const int most = saves ? 1 : stream_pairs(p.lv[l], p.L, tau, l == 0, shared);
    PairSchedule s{0, 0, 0};
    if (most == 3 && np >= 2) {
        // As few launches as possible.
        const int launches = (np + 2) / 3;
        s.threes = np - 2 * launches;
        s.twos = launches - s.threes;
    } else if (most >= 2) {
        // A single pair comes first, where the incoming state is the parent
        // level's (a quarter of the rows to read) or zero.
        s.ones = np & 1;
        s.twos = np / 2;
    } else {
        s.ones = np;
    }
    if (even_count && (s.count() & 1)) {
        // One more launch: three pairs as one and two, or two as single ones.
        if (s.threes > 0) {
            --s.threes;
            ++s.twos;
            ++s.ones;
        } else if (s.twos > 0) {
            --s.twos;
            s.ones += 2;
        }
    }
    return s;
}

// The extra stage against colour 0's state stored and a readout pass over it,
// whole frames: 676 x 380 x 64 FP32 454 -> 431 us, 1352 x 760 x 128 FP32 2591 ->
// 2327, in bfloat16 with soft disparities 2823 -> 2758, eight frames in FP16
// 5368 -> 5267.  Over all splits, forms and costs at 1352 x 760: FP32 .78 to .95 of
// the time, also where its registers spill, bfloat16 .95 to 1.00.
bool stream_reads_out(const PairSchedule &s, bool exports, bool saves)
{
    return !exports && !saves && s.count() > 0 && s.pairs(s.count() - 1) > 1;
}

void stream_shape(PairArgs *a, int SEGV, int R)
{
    const int stages = 2 * a->pairs + (a->ro0 ? 1 : 0);
    a->tx = strip_width(a->w, stream_columns(SEGV, R), stages);
    a->tiles_x = (a->w + a->tx - 1) / a->tx;
    a->ty = segment_rows(a->h, a->tiles_x, stages);
    a->ntiles = a->tiles_x * ((a->h + a->ty - 1) / a->ty);
    a->per_xcd = (a->ntiles + 7) / 8;
}

bp_status dispatch_iter_stream(const PairArgs &a, int fmt, int SEGV, int R, hipStream_t st)
{
    switch (fmt) {
    case FMT_F16: return stream_launch<StoreF16>(a, SEGV, R, st);
    case FMT_BF16: return stream_launch<StoreBF16>(a, SEGV, R, st);
    default: return stream_launch<StoreF32>(a, SEGV, R, st);
    }
}

}  // namespace bpk
