// The few-token stages (stream_mma.hip): linears of up to 64 tokens by the
// list's matrix-core stages, each in the first ws_bytes (what
// lb_forward_workspace_bytes says) of its own workspace; n (1 .. kFewMaxBatch)
// of one token tile count and one pair of dtypes at once.
#pragma once
#include "lb_internal.h"

namespace lb {

constexpr int kFewMaxBatch = 8;
bool few_tokens_supports(const ForwardArgs& a, size_t ws_bytes);
hipError_t launch_few_tokens(const ForwardArgs* a, const size_t* ws_bytes, int n, hipStream_t stream);

}  // namespace lb
