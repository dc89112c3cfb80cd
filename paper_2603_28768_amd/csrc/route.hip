// Router softmax / top-k: the top-K routing step of the MoE layer of Sec. 2.1.
//
// A token is handled by one 16-lane DPP row of a 64-lane wavefront, so a wave routes four
// tokens at once and every cross-lane step is a row-local DPP move (quad permutes and
// row mirrors), not an LDS permute.  A lane holds the scores of experts 4*lane..4*lane+3,
// +64, +128, ... (16-byte loads; a token's row is read as contiguous 256-byte pieces).
// Up to 14 picks are made at once where that pays (route_block.h); otherwise, or where too many scores
// tie for that, each of the k picks is an arg-max over (score, expert id): first inside the lane in
// ascending expert order, then a four-step butterfly over the row.  Scores are compared
// raw, never their exponentials, and equal scores resolve to the lower expert id.
//
// A workgroup of eight waves covers 32 consecutive tokens.  While the picks are still in
// registers it also records, per expert, a 32-bit mask of the block's tokens that chose it:
// the number of set bits below a token's own bit is that assignment's rank among the
// block's assignments to the expert (experts of one token are distinct), and the
// population count is the block's contribution to the expert's load.
#include "route_block.h"

namespace craft {
namespace {

template <int NQ, bool PARTS>
__global__ __launch_bounds__(kRouteThreads) void route_kernel(RouteArgs a) {
    __shared__ uint32_t mask[kRouteMaxE];
    __shared__ uint64_t cand[kTokPerBlock][32];
    const int tid = threadIdx.x;
    const bool ranks = a.hist != nullptr;
    if (ranks) {
        for (int e = tid; e < a.E; e += kRouteThreads) mask[e] = 0u;
        if (a.ctrl && blockIdx.x == 0 && tid < CTRL_WORDS) a.ctrl[tid] = 0;
        __syncthreads();
    }
    const int sub = tid & 15, tl = tid >> 4;       // lane of the token's row; token inside the block
    const int64_t t = (int64_t)blockIdx.x * kTokPerBlock + tl;
    int my_id[kMaxPickSlots];
    route_block<NQ, PARTS>(a, t, tl, true, ranks ? mask : nullptr, cand, my_id);
    if (!ranks) return;
    __syncthreads();
#pragma unroll
    for (int s = 0; s < kMaxPickSlots; ++s) {
        const int j = s * 16 + sub;
        if (t < a.T && j < a.k)
            a.lrank[t * a.k + j] = (uint8_t)__popc(mask[my_id[s]] & ((1u << tl) - 1u));
    }
    int32_t *hrow = a.hist + (int64_t)blockIdx.x * a.E;
    for (int e = tid; e < a.E; e += kRouteThreads) hrow[e] = __popc(mask[e]);
}

__global__ void clear_ctrl_kernel(int32_t *ctrl) {
    if (threadIdx.x < CTRL_WORDS) ctrl[threadIdx.x] = 0;
}

}  // namespace

hipError_t launch_route(const RouteArgs &a, hipStream_t s) {
    if (a.T == 0) {
        // nothing to route; the control words still have to be cleared for the next stage
        // (a kernel rather than a memset node, so the call stays safe to capture in a graph)
        if (a.ctrl) hipLaunchKernelGGL(clear_ctrl_kernel, dim3(1), dim3(64), 0, s, a.ctrl);
        return hipGetLastError();
    }
    const int64_t nb = (a.T + kTokPerBlock - 1) / kTokPerBlock;
    dim3 grid((unsigned)nb), block(kRouteThreads);
    const int nq = (a.E + 63) / 64;
    if (nq > 6 && a.nparts > 1) return hipErrorInvalidValue;    // (a gate of so many experts is never split)
    auto go = [&](auto n) {
        if (n.value <= 6 && a.nparts > 1) hipLaunchKernelGGL((route_kernel<(n.value <= 6 ? n.value : 6), true>), grid, block, 0, s, a);
        else hipLaunchKernelGGL((route_kernel<n.value, false>), grid, block, 0, s, a);
    };
    if (nq <= 1) go(std::integral_constant<int, 1>{});
    else if (nq <= 2) go(std::integral_constant<int, 2>{});
    else if (nq <= 4) go(std::integral_constant<int, 4>{});
    else if (nq <= 6) go(std::integral_constant<int, 6>{});
    else if (nq <= 8) go(std::integral_constant<int, 8>{});
    else go(std::integral_constant<int, 16>{});
    return hipGetLastError();
}

}  // namespace craft
