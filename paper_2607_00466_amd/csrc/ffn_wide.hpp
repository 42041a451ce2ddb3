// The expert FFN's kernel for batches whose buckets are large.
#pragma once

#include "ffn_common.hpp"

namespace eldr {

// Launches the wide kernel (and sets a.tiles).
template <int MODE, int FMT>
void launch_ffn_wide(FfnArgs a, int T, int K, int E, hipStream_t s);

}  // namespace eldr
