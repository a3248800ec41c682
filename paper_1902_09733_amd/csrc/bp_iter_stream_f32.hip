// The streamed half-sweeps (bp_iter_stream_impl.h) with F32 message storage.
#include "bp_iter_stream_impl.h"

namespace bpk {

template bp_status stream_launch<StoreF32>(const PairArgs &, int, int, hipStream_t);

}  // namespace bpk
