// Expert weights (bf16) into the stream the packed FFN kernels read (see ffn_packed.hip).  Not
// part of a forward: this is model loading, and what a rank does with the experts it fetches
// at a rebalancing.
#include "kernels.h"

namespace craft {
namespace {

typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));

// The packed stream in 16-byte chunks: chunk ((step * groups + group) * 2 + half) * 64 + lane.
//   gate/up : group g = output columns 16g..16g+15; half 0 = gate rows 16g..16g+15, half 1 = the
//             up rows of the same columns
//   down    : group g = output columns 32g..32g+31; half h = down rows 32g+16h..+15
// Lane l of 32-wide step s holds row (l & 15) of its half, contraction elements 32s + 8(l>>4) .. +7:
// the row operand of one v_mfma_f32_16x16x32_bf16.  Rows and contraction elements past the matrix are zero.
//
// A workgroup re-orders 16 weight rows over kPartSteps steps; all three matrices in one launch.
// A wave takes pairs of neighbouring steps, whose requests read whole 128-byte lines of a row
// between them, has all of its eight requests under way before the first store, and stores 1 KiB
// of consecutive bytes per step.  Bound by memory: 4 bytes moved per weight, 5.26 TB/s at H = 7168,
// I = 2048 (33.5 us an expert; two launches of one thread per chunk, with a division each: 41 us).
constexpr int kPackThreads = 256;
constexpr int kPairs = 4;                              // step pairs per wave
constexpr int kPartSteps = 2 * kPairs * (kPackThreads / 64);
struct PackArgs {
    const unsigned short *w[3];                        // gate, up [I][H]; down [H][I]
    unsigned char *gateup, *down;
    int32_t H, I;
    int32_t gateup_groups, down_groups;                // padded to whole tiles
    int32_t gateup_parts, down_parts;                  // workgroups along the contraction
};
__global__ __launch_bounds__(kPackThreads) void pack_kernel(PackArgs a) {
    int b = blockIdx.x;
    const int gateup_blocks = 2 * a.gateup_groups * a.gateup_parts;
    const bool gateup = b < gateup_blocks;
    if (!gateup) b -= gateup_blocks;
    const int parts = gateup ? a.gateup_parts : a.down_parts;
    const int g = b / parts >> 1, h = b / parts & 1, part = b % parts;
    const int K = gateup ? a.H : a.I, N = gateup ? a.I : a.H;
    const int ksteps = (K + 255) / 256 * 8;
    const int64_t step_bytes = (int64_t)(gateup ? a.gateup_groups : a.down_groups) * 2048;
    const int row0 = gateup ? 16 * g : 32 * g + 16 * h;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r = row0 + (lane & 15), k_lane = 8 * (lane >> 4);
    const unsigned short *row = (gateup ? a.w[h] : a.w[2]) + (int64_t)min(r, N - 1) * K;
    unsigned char *out = (gateup ? a.gateup : a.down) + (int64_t)g * 2048 + h * 1024 + lane * 16;
    const int s0 = part * kPartSteps + 2 * wave;
    const u32x4_t zero = {0u, 0u, 0u, 0u};
    u32x4_t v[kPairs][2];
#pragma unroll
    for (int p = 0; p < kPairs; ++p)
#pragma unroll
        for (int j = 0; j < 2; ++j)
            v[p][j] = *reinterpret_cast<const u32x4_t *>(row + min(32 * (s0 + 8 * p + j) + k_lane, K - 8));
#pragma unroll
    for (int p = 0; p < kPairs; ++p)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int s = s0 + 8 * p + j;
            if (s < ksteps)
                __builtin_nontemporal_store(r < N && 32 * s + k_lane < K ? v[p][j] : zero,
                                            reinterpret_cast<u32x4_t *>(out + s * step_bytes));
        }
}

}  // namespace

void packed_sizes(int32_t H, int32_t I, size_t *gateup_bytes, size_t *down_bytes) {
    const size_t gu_groups = ((size_t)(I + 15) / 16 + 7) / 8 * 8, gu_steps = (size_t)(H + 255) / 256 * 16;
    const size_t dn_groups = ((size_t)(H + 31) / 32 + 7) / 8 * 8, dn_steps = (size_t)(I + 255) / 256 * 16;
    *gateup_bytes = gu_groups * gu_steps * 1024;
    *down_bytes = dn_groups * dn_steps * 1024;
}

hipError_t launch_pack(int32_t H, int32_t I, const void *wg, const void *wu, const void *wd,
                       void *pgu, void *pdn, hipStream_t s) {
    PackArgs a{{static_cast<const unsigned short *>(wg), static_cast<const unsigned short *>(wu),
                static_cast<const unsigned short *>(wd)},
               static_cast<unsigned char *>(pgu), static_cast<unsigned char *>(pdn), H, I,
               ((I + 15) / 16 + 7) / 8 * 8, ((H + 31) / 32 + 7) / 8 * 8, 0, 0};
    a.gateup_parts = ((H + 255) / 256 * 8 + kPartSteps - 1) / kPartSteps;
    a.down_parts = ((I + 255) / 256 * 8 + kPartSteps - 1) / kPartSteps;
    const int64_t blocks = 2 * ((int64_t)a.gateup_groups * a.gateup_parts + (int64_t)a.down_groups * a.down_parts);
    if (blocks >= (1ll << 32) / kPackThreads) return hipErrorInvalidValue;        // a launch has fewer than 2^32 threads
    hipLaunchKernelGGL(pack_kernel, dim3((unsigned)blocks), dim3(kPackThreads), 0, s, a);
    return hipGetLastError();
}

}  // namespace craft
