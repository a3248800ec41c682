// The streamed half-sweeps (bp_iter_stream_impl.h) with F16 message storage.
#include "bp_iter_stream_impl.h"

namespace bpk {

template bp_status stream_launch<StoreF16>(const PairArgs &, int, int, hipStream_t);

}  // namespace bpk
