// The streamed half-sweeps (bp_iter_stream_impl.h) with BF16 message storage.
#include "bp_iter_stream_impl.h"

namespace bpk {

template bp_status stream_launch<StoreBF16>(const PairArgs &, int, int, hipStream_t);

}  // namespace bpk
