// The few-token stages (stream_mma.hip): linears of up to 64 tokens by the
// list's matrix-core stages, each in the first ws_bytes (what
// lb_forward_workspace_bytes says) of its own workspace, by the plan that
// few_tokens_plan made for it; n (1 .. kFewMaxBatch) of one token tile count and
// one pair of dtypes at once.
#pragma once
#include "lb_internal.h"

namespace lb {

constexpr int kFewMaxBatch = 8;
struct FewPlan {
  int tt, nmf;   // token and latent tiles of 16
  int ng, mt;    // groups of four waves the latent tiles are spread over, tiles per wave
  int bpr, s1d;  // 32-input blocks per run, runs
  int cls;       // tile class of stage 1
};
// whether the stages take a (its plan then in g)
bool few_tokens_plan(const ForwardArgs& a, size_t ws_bytes, FewPlan& g);
hipError_t launch_few_tokens(const ForwardArgs* a, const FewPlan* g, int n, hipStream_t stream);

}  // namespace lb
