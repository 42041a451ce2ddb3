// The expert FFN's kernel for batches of a few tokens.
#pragma once

#include "ffn_common.hpp"

namespace eldr {

// Launches the one-wave kernel; ROUTED (up): the buckets are built from a.ids and written out.
template <int MODE, int FMT, bool ROUTED>
void launch_ffn_slim(const FfnArgs& args, int T, int K, int E, hipStream_t s);

}  // namespace eldr
