// Shapes of the streamed half-sweeps, shared by their host side
// (bp_iter_stream.hip) and their kernels' translation units.
#pragma once

#include <hip/hip_runtime.h>

#include "bp_internal.h"

namespace bpk {

// Waves per block for R labels per lane: as many as their registers leave
// room for (about 100 to 165 VGPRs with four labels, 180 to 250 with eight),
// since a block's columns are its waves' and wide strips repeat fewer.
// Measured at 676 x 380 x 64 (five pairs, as 2 + 3): 8 waves 203 us, 10 185,
// 12 167, 16 (128 registers, spilling) 230.
constexpr int stream_waves(int R) { return R <= 4 ? 12 : 8; }

// Columns a block carries for a lane split (0: not streamed).
inline int stream_columns(int SEGV, int R)
{
    const bool ok = (SEGV == 4 && R == 4) || (SEGV == 8 && R == 4) || (SEGV == 16 && (R == 4 || R == 6 || R == 8));
    return ok ? stream_waves(R) * (64 / SEGV) : 0;
}

// Whether three pairs per launch are compiled for a lane split and storage:
// with eight labels per lane and FP32 rows their registers would spill (434
// against 257 us per pair at 1352 x 760 x 128).
constexpr bool stream_three(int R, int fmt) { return R <= 6 || fmt != FMT_F32; }

template <typename S>
bp_status stream_launch(const PairArgs &a, int SEGV, int R, hipStream_t st);

}  // namespace bpk
