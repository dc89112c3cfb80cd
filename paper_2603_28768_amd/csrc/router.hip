// Gating-network scores, the input of top-K routing (Sec. 2.1).  The paper leaves the form of
// the network open; this is the usual linear gate,
//   logits[t][e] = sum_h x[t][h] * Wr[e][h],
// both operands contiguous along the contraction, fp32 accumulation, fp32 scores.  The top-k
// step consumes these scores exactly as it consumes scores handed in from outside.
//
// A skinny GEMM: few output columns (E = 128 .. 384), so the tokens' activations are what
// has to cross HBM (once) and the gate's weights are re-read from L2 by every workgroup.
// bf16: 32, 64 or 128 tokens against 64 to 256 experts per workgroup (nt_tile.h), the experts as the
// matrix instruction's row operand, so that a lane holds four neighbouring experts of a token:
// 16-byte stores.  Every workgroup pulls its experts' rows out of L2, so T H 2 (E / experts + E / tokens per
// workgroup) bytes move from L2 into the CUs; large tiles move less but there are few of them, so with a
// workspace the contraction is summed in up to 8 parts per tile, by one workgroup after one another or by
// several: those write their partial scores and a second kernel (or the routing kernel) adds them in
// ascending order of the split (a fixed order: the result does not depend on scheduling).
// fp32: one thread per score, a plain chain of fused multiply-adds (small configurations).
#include <algorithm>

#include "nt_tile.h"

namespace craft {
namespace {

// Tokens up to which the gate is read by thin tiles: few tall ones leave CUs without work (8 tokens:
// 23 us for scores of E = 256, H = 7168, thin 4.4).  Past it the small ones of the tiles below are the faster
// ones at every shape tried (129 tokens, H = 7168, us thin / tiles: E = 64 9.8 / 9.2, E = 256 14.7 / 7.3, E = 384
// 15.8 / 7.7); where below it they begin to be has not been measured.
constexpr int kThinBatch = 128;
constexpr int GK = 64;                  // contraction slab
typedef unsigned int gu32x4_t __attribute__((ext_vector_type(4)));
typedef const gu32x4_t __attribute__((address_space(1))) *gchunk_t;

// PARTED: a workgroup takes several parts of the contraction.
template <int FA, int FB, bool PARTED>
__global__ __launch_bounds__(kNtThreads) void router_logits_bf16_kernel(RouterArgs a) {
    __shared__ __attribute__((aligned(16))) unsigned char gate_smem[nt_lds_bytes<FA, FB>()];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    // Workgroups go round the XCDs: (tile of tokens, split) by (tile, split), so that a few tiles reach all of
    // them, and the blocks of experts of one, which read the same activations, one behind the other in one L2
    // (launch_bf16 says when).  (With the splits of a tile in one L2, 2 tiles of 150 tokens kept to two XCDs:
    // H = 2048, E = 160 9.8 us, so 9.0.)
    uint32_t tile = blockIdx.x, split = blockIdx.z, eblock = blockIdx.y;
    if (a.eblocks != 0) {
        const uint32_t eight = blockIdx.x >> 3, group = __umulhi(eight, a.eblocks_inv);
        eblock = eight - group * (uint32_t)a.eblocks;
        tile = group * 8 + (blockIdx.x & 7);
        if (a.nsplit > 1) {
            split = __umulhi(tile, a.tiles_inv);
            tile -= split * (uint32_t)a.tiles;
        }
    }
    const int64_t t0 = (int64_t)tile * (FB * 32);
    const int e0 = (int)eblock * (FA * 32);
    if (t0 >= a.T || split >= (uint32_t)a.nsplit) return;          // (the last eight are not all there)
    // this workgroup's share of the contraction (may be empty)
    const int nk = (a.H + GK - 1) / GK;
    const int kbeg = min(nk, (int)split * a.share), kend = min(nk, kbeg + a.share);
    float *dst = a.nsplit > 1 ? a.part + (int64_t)split * a.T * a.E : a.logits;
    // rows past the end are clamped into the matrix (their results are not stored)
    auto eoff = [&](int i) { return (uint32_t)min(i, a.E - 1 - e0) * (uint32_t)a.H * 2u; };
    auto toff = [&](int, int i) { return (uint32_t)min((int64_t)i, a.T - 1 - t0) * (uint32_t)a.H * 2u; };
    f32x4_t acc[FA][FB];
#pragma unroll
    for (int f = 0; f < FA; ++f)
#pragma unroll
        for (int g = 0; g < FB; ++g) acc[f][g] = (f32x4_t)(0.0f);
    const ubase_t wbase = uniform_base(static_cast<ubase_t>(a.w) + (int64_t)e0 * a.H * 2), xbase = uniform_base(static_cast<ubase_t>(a.x) + t0 * a.H * 2);
    if constexpr (PARTED) {
        // each part starts from zero, like one of a workgroup of its own
        f32x4_t sum[FA][FB];
#pragma unroll
        for (int f = 0; f < FA; ++f)
#pragma unroll
            for (int g = 0; g < FB; ++g) sum[f][g] = (f32x4_t)(0.0f);
        int cut = kbeg + a.per - 1;
        nt_tile<FA, FB>(gate_smem, wbase, eoff, xbase, toff, a.H, kbeg, kend, acc, [&](int ks) __attribute__((always_inline)) {
            if (ks != cut || ks == kend - 1) return;
            cut += a.per;
            nt_settle(acc);
#pragma unroll
            for (int f = 0; f < FA; ++f)
#pragma unroll
                for (int g = 0; g < FB; ++g) {
                    sum[f][g] += acc[f][g];
                    acc[f][g] = (f32x4_t)(0.0f);
                    asm volatile("s_nop 1" : "+a"(acc[f][g]));  // a matrix instruction reads it two cycles later at the earliest
                }
        });
#pragma unroll
        for (int f = 0; f < FA; ++f)
#pragma unroll
            for (int g = 0; g < FB; ++g) acc[f][g] = sum[f][g] + acc[f][g];
    } else {
        nt_tile<FA, FB>(gate_smem, wbase, eoff, xbase, toff, a.H, kbeg, kend, acc);
    }
    const bool whole = (a.E & 3) == 0 && (reinterpret_cast<uintptr_t>(dst) & 15) == 0;
#pragma unroll
    for (int g = 0; g < FB; ++g) {
        const int64_t t = t0 + ((wave & 1) * FB + g) * 16 + (lane & 15);
#pragma unroll
        for (int f = 0; f < FA; ++f) {
            const int e = e0 + ((wave >> 1) * FA + f) * 16 + (lane >> 4) * 4;
            if (t >= a.T || e >= a.E) continue;
            float *to = dst + t * a.E + e;
            if (whole) {
                *reinterpret_cast<f32x4_t *>(to) = acc[f][g];
            } else {
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if (e + c < a.E) to[c] = acc[f][g][c];
            }
        }
    }
}

// A small batch: nothing but the gate's weights to read, E H 2 bytes that a few tall tiles would
// pull through a few CUs (8 tokens, E = 256, H = 7168: 23 us).  A workgroup takes 16 experts against
// up to 64 tokens and one split of the contraction, its four waves every fourth 64-wide slab of
// that, both operands straight from global memory in the operand layout of
// v_mfma_f32_16x16x32_bf16; the waves' sums meet in LDS and are added in wave order.
constexpr int kThinWaves = 4;
constexpr int kThinTokens = 64;
template <int NXF>
__device__ __forceinline__ void thin_tile(const RouterArgs &a, int64_t t0, int e0, int kbeg, int kend, float *dst, f32x4_t *sums) {
    constexpr int PW = 4;                                  // slabs in flight per wave
    const int lane = threadIdx.x & 63, q = lane >> 4, r16 = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int hchunks = a.H >> 3;
    gchunk_t wrow = (gchunk_t)a.w + (int64_t)min(e0 + r16, a.E - 1) * hchunks, xrow[NXF];
#pragma unroll
    for (int g = 0; g < NXF; ++g) xrow[g] = (gchunk_t)a.x + min(t0 + 16 * g + r16, a.T - 1) * hchunks;
    f32x4_t acc[NXF];
#pragma unroll
    for (int g = 0; g < NXF; ++g) acc[g] = (f32x4_t)(0.0f);
    const gu32x4_t zero = {0u, 0u, 0u, 0u};
    for (int s0 = kbeg + wave; s0 < kend; s0 += PW * kThinWaves) {
        gu32x4_t w[PW][2], x[PW][2][NXF];
#pragma unroll
        for (int u = 0; u < PW; ++u)
#pragma unroll
            for (int st = 0; st < 2; ++st) {
                // past the split or the rows: read from inside them, replaced by zeros below
                const int c = min((s0 + u * kThinWaves) * 8 + st * 4 + q, hchunks - 1);
                w[u][st] = wrow[c];
#pragma unroll
                for (int g = 0; g < NXF; ++g) x[u][st][g] = xrow[g][c];
            }
#pragma unroll
        for (int u = 0; u < PW; ++u) {
            const int s = s0 + u * kThinWaves;
#pragma unroll
            for (int st = 0; st < 2; ++st) {
                const bool in = s < kend && s * 8 + st * 4 + q < hchunks;
                const bf16x8_t wf = __builtin_bit_cast(bf16x8_t, in ? w[u][st] : zero);
#pragma unroll
                for (int g = 0; g < NXF; ++g)
                    acc[g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf, __builtin_bit_cast(bf16x8_t, in ? x[u][st][g] : zero),
                                                                     acc[g], 0, 0, 0);
            }
        }
    }
#pragma unroll
    for (int g = 0; g < NXF; ++g) sums[(wave * NXF + g) * 64 + lane] = acc[g];
    __syncthreads();
    // element v of lane l: expert e0 + 4 (l >> 4) + v, token l & 15 of the fragment
    for (int g = wave; g < NXF; g += kThinWaves) {
        f32x4_t v = sums[g * 64 + lane];
#pragma unroll
        for (int z = 1; z < kThinWaves; ++z) v += sums[(z * NXF + g) * 64 + lane];
        const int64_t t = t0 + 16 * g + r16;
#pragma unroll
        for (int c = 0; c < 4; ++c)
            if (t < a.T && e0 + 4 * q + c < a.E) dst[t * a.E + e0 + 4 * q + c] = v[c];
    }
}
__global__ __launch_bounds__(64 * kThinWaves) void router_thin_kernel(RouterArgs a) {
    __shared__ f32x4_t sums[kThinWaves * (kThinTokens / 16) * 64];
    const int64_t t0 = (int64_t)blockIdx.y * kThinTokens;
    const int e0 = blockIdx.x * 16;
    const int nk = (a.H + GK - 1) / GK;
    const int kbeg = min(nk, (int)blockIdx.z * a.share), kend = min(nk, kbeg + a.share);
    float *dst = a.nsplit > 1 ? a.part + (int64_t)blockIdx.z * a.T * a.E : a.logits;
    const int64_t tokens = a.T - t0;
    if (tokens <= 16) thin_tile<1>(a, t0, e0, kbeg, kend, dst, sums);
    else if (tokens <= 32) thin_tile<2>(a, t0, e0, kbeg, kend, dst, sums);
    else thin_tile<4>(a, t0, e0, kbeg, kend, dst, sums);
}

// logits = sum of the partial scores, in ascending order of the split
template <typename V, int NSPLIT>
__global__ __launch_bounds__(256) void router_reduce_kernel(const V *part, int64_t n, V *logits) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    V v[NSPLIT];                                           // all parts are requested before the first is added
#pragma unroll
    for (int z = 0; z < NSPLIT; ++z) v[z] = part[(int64_t)z * n + i];
    V s = v[0];
#pragma unroll
    for (int z = 1; z < NSPLIT; ++z) s += v[z];
    logits[i] = s;
}

__global__ __launch_bounds__(256) void router_logits_f32_kernel(RouterArgs a) {
    const int64_t o = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (o >= a.T * a.E) return;
    const float *x = static_cast<const float *>(a.x) + (o / a.E) * a.H;
    const float *w = static_cast<const float *>(a.w) + (o % a.E) * a.H;
    float s = 0.0f;
    for (int h = 0; h < a.H; ++h) s = fmaf(x[h], w[h], s);
    a.logits[o] = s;
}

// Tiles whose workgroups may take several parts.  The others were never or hardly ever the ones expected to be
// fastest (5 million shapes of H = 8 to 16384), and the largest keeps 380 registers for the sums.
constexpr bool parted_tile(int fa, int tokens) { return fa == 2 || (fa <= 6 && tokens >= 2); }

template <typename V>
void launch_reduce(const RouterArgs &a, int nsplit, int64_t n, hipStream_t s) {
    const dim3 grid((unsigned)((n + 255) / 256)), block(256);
    const V *part = reinterpret_cast<const V *>(a.part);
    V *out = reinterpret_cast<V *>(a.logits);
    if (nsplit == 2) hipLaunchKernelGGL((router_reduce_kernel<V, 2>), grid, block, 0, s, part, n, out);
    else if (nsplit == 4) hipLaunchKernelGGL((router_reduce_kernel<V, 4>), grid, block, 0, s, part, n, out);
    else hipLaunchKernelGGL((router_reduce_kernel<V, 8>), grid, block, 0, s, part, n, out);
}
template <int FA, int FB>
hipError_t launch_bf16(const RouterArgs &a, hipStream_t s) {
    RouterArgs b = a;
    const int64_t tiles = (a.T + FB * 32 - 1) / (FB * 32), units = tiles * a.nsplit;
    const int eblocks = (a.E + FA * 32 - 1) / (FA * 32);
    dim3 grid((unsigned)tiles, (unsigned)eblocks, (unsigned)a.nsplit);
    // The blocks of experts of a tile meet in one L2 (2280 tokens of H = 7168, E = 130: 17.7 us a call, one block
    // after another 23.7) unless some XCD would get a round of workgroups more for it (10266 of H = 4096, E = 300, 81
    // tiles x 3 blocks: 62.9, so 43.2).  A contraction in one part comes out in several rounds of workgroups: there
    // one block follows another, whose rows then stay in L2, as long as the memory-side cache holds the activations
    // for the next block (E = 384, us meeting / one after another: 19060 tokens of H = 1024 38.9 / 32.8, 18555 of 5120
    // 149 / 136, 32764 of 6144 241 / 272).
    constexpr int fit = (160 << 10) / nt_lds_bytes<FA, FB>();      // workgroups a CU has LDS for
    const int at_once = fit * (a.num_cu > 8 ? a.num_cu / 8 : 1);   // and an XCD
    const bool meet = eblocks > 1 && (a.nparts > 1 ? ((units + 7) / 8 * eblocks + at_once - 1) / at_once <= (units * eblocks + 8 * at_once - 1) / (8 * at_once)
                                                   : a.T * a.H * 2 > ((int64_t)220 << 20));
    if (meet) {
        // the quotients by these are exact: fewer than 2^21 eights by up to 16 blocks, and a split launch has two
        // tiles or more and fewer than 4 num_cu + 8 units
        static_assert(kThinBatch >= 32 * 4, "tiles_inv of one tile");
        auto inverse = [](int64_t n) { return (uint32_t)((((uint64_t)1 << 32) + (uint64_t)n - 1) / (uint64_t)n); };
        b.eblocks = eblocks;
        b.tiles = (int32_t)tiles;
        b.eblocks_inv = inverse(eblocks);
        b.tiles_inv = inverse(tiles);
        grid = dim3((unsigned)((units + 7) / 8 * 8 * eblocks), 1, 1);
    }
    if constexpr (parted_tile(FA, FB))
        if (a.nparts > a.nsplit) {
            hipLaunchKernelGGL((router_logits_bf16_kernel<FA, FB, true>), grid, dim3(kNtThreads), 0, s, b);
            return hipGetLastError();
        }
    hipLaunchKernelGGL((router_logits_bf16_kernel<FA, FB, false>), grid, dim3(kNtThreads), 0, s, b);
    return hipGetLastError();
}
template <int FA>
hipError_t launch_bf16(const RouterArgs &a, int nxf, hipStream_t s) {
    return nxf == 1 ? launch_bf16<FA, 1>(a, s) : nxf == 2 ? launch_bf16<FA, 2>(a, s) : launch_bf16<FA, 4>(a, s);
}

}  // namespace

namespace {

// 16-row fragments of experts per wave, and blocks of experts, of tiles of up to `most` experts: blocks as
// even as they come.
int expert_blocks(int32_t E, int most) { return (E + most - 1) / most; }
int expert_fragments(int32_t E, int most) {
    const int rows = (E + expert_blocks(E, most) - 1) / expert_blocks(E, most);
    return rows <= 64 ? 2 : rows <= 128 ? 4 : rows <= 192 ? 6 : 8;
}
// Expected us of a launch and of the one that adds its parts.  A CU takes as many workgroups at a time as it has
// LDS for, each bound by what it loads (more so with three stages of LDS than with more) and slowed down by the
// others; parts in memory are written, read and added.  Fitted to 1030 shapes (H = 512 to 8192, E = 48 to 384,
// 129 to 16384 tokens; every tile and split of each, timed without host time between the calls): off by 16 %
// (rms), on 350 others as well.
double expected_us(const RouterShape &s, int64_t T, int32_t H, int32_t E, int32_t num_cu) {
    const int fa = expert_fragments(E, s.experts), nk = (H + GK - 1) / GK;
    const int stage = (fa + s.tokens) * 32 * 128, stages = nt_stages_of(stage), fit = (160 << 10) / (stages * stage);
    const int64_t wgs = (T + 32 * s.tokens - 1) / (32 * s.tokens) * expert_blocks(E, s.experts) * s.nsplit, per_cu = (wgs + num_cu - 1) / num_cu;
    const double slabs = (double)((nk + s.nparts - 1) / s.nparts) * (s.nparts / s.nsplit);
    const double slab = 0.061 * (fa + s.tokens) * (stages == 3 ? 1.115 : 1.0);
    auto at_once = [&](int64_t n) { return n > 0 ? 3.1 + slabs * slab * (0.27 + 0.73 * (double)n) : 0.0; };
    const double load = (double)(per_cu / fit) * at_once(fit) + at_once(per_cu % fit), mb = (double)T * E * 4e-6;
    return (load + (s.nsplit > 1 ? s.nsplit * mb * 0.51 + 2.1 : mb * 0.1)) * (s.nparts > s.nsplit ? 1.026 : 1.0);
}

}  // namespace

// With a workspace the contraction is summed in as many parts as bring tall tiles of all experts up to the CU
// count (at most 8, at least 4 slabs each; more than 384 experts are never split).  Asked by every call and
// every forward for the size of the workspace, which the tile choice below (0.3 us of host time) does not change.
int router_logits_parts(int64_t T, int32_t H, int32_t E, int32_t num_cu) {
    if (E > 384) return 1;
    const int64_t tiles = (T + 127) / 128;
    const int nk = (H + GK - 1) / GK;
    int parts = 1;
    while (parts < 8 && tiles * parts * 2 <= num_cu && nk / (parts * 2) >= 4) parts *= 2;
    return parts;
}

// The tile and the split of the contraction for a shape.  Without a workspace: short tiles, as many as
// there are CUs if possible.  With one: how many of the parts one workgroup takes after another, and how
// large the tiles are, follows expected_us: tall tiles of 256 experts, a workgroup per part, unless another way
// is expected to take less than 0.95 of their time.  Every other part left to another workgroup is a copy of the
// scores to write, read and add.  us a call, tall tiles with a workgroup per part / this: H = 7168, E = 256, 600 tokens
// 19.7 / 12.0, 2048 22.4 / 17.3; E = 384, 4096 49.2 / 40.0, 16384 129 / 112; H = 2880, E = 256, 4096 23.1 / 14.9, 8192
// 30.9 / 24.6.  Over 300 shapes (H = 1024 to 7168, E = 64 to 384, 150 to 16384 tokens) it takes 0.74 of the time of tall
// tiles in the mean, from 0.40 to 1.06 (8192 tokens of H = 4096, E = 128: 24.1 / 25.4), over 500 drawn ones 0.77, up to
// 1.13 (8703 of H = 4880, E = 256: 56.7 / 64.2).
RouterShape router_logits_shape(int64_t T, int32_t H, int32_t E, int32_t num_cu, bool workspace) {
    RouterShape s{1, 256, 1, 1};
    if (!workspace || E > 384) {
        s.tokens = E <= 384 && (T + 63) / 64 >= (int64_t)num_cu ? 2 : 1;
        return s;
    }
    s.tokens = 4;
    s.nparts = s.nsplit = router_logits_parts(T, H, E, num_cu);
    if (T <= kThinBatch || H >= kNtRowLimit || s.nparts == 1) return s;
    RouterShape best = s;
    double best_us = expected_us(s, T, H, E, num_cu) * 0.95;
    for (int tokens = 1; tokens <= 4; tokens *= 2)
        for (int experts = 64; experts <= 256; experts += 64) {
            if (experts > 64 && expert_blocks(E, experts) == expert_blocks(E, experts - 64)) continue;
            const int64_t wgs = (T + 32 * tokens - 1) / (32 * tokens) * expert_blocks(E, experts);
            for (int nsplit = 1; nsplit <= s.nparts; nsplit *= 2) {
                if (wgs * nsplit < num_cu / 4 || wgs * nsplit > 4 * num_cu) continue;
                if (nsplit < s.nparts && !parted_tile(expert_fragments(E, experts), tokens)) continue;
                const RouterShape c{tokens, experts, s.nparts, nsplit};
                const double us = expected_us(c, T, H, E, num_cu);
                if (us < best_us) { best_us = us; best = c; }
            }
        }
    return best;
}

hipError_t launch_router_logits(const RouterArgs &a, hipStream_t s, int *nsplit_out) {
    if (nsplit_out) *nsplit_out = 1;
    if (a.T == 0) return hipSuccess;
    if (a.dtype == CRAFT_F32) {
        const int64_t n = a.T * a.E;
        hipLaunchKernelGGL(router_logits_f32_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, a);
        return hipGetLastError();
    }
    const RouterShape shape = router_logits_shape(a.T, a.H, a.E, a.num_cu, a.part != nullptr);
    const int nxf = shape.tokens, nsplit = shape.nsplit;
    if (nsplit_out && a.keep_parts) *nsplit_out = nsplit;
    RouterArgs b = a;
    b.nsplit = nsplit;
    b.nparts = shape.nparts;
    const int nk = (a.H + GK - 1) / GK;
    b.per = (nk + b.nparts - 1) / b.nparts;
    b.share = b.per * (b.nparts / b.nsplit);
    hipError_t err;
    if (a.T <= kThinBatch || a.H >= kNtRowLimit) {         // (thin tiles take rows of any length)
        const dim3 grid((unsigned)((a.E + 15) / 16), (unsigned)((a.T + kThinTokens - 1) / kThinTokens), (unsigned)nsplit);
        hipLaunchKernelGGL(router_thin_kernel, grid, dim3(64 * kThinWaves), 0, s, b);
        err = hipGetLastError();
    } else {
        const int fa = expert_fragments(a.E, shape.experts);
        err = fa == 2 ? launch_bf16<2>(b, nxf, s) : fa == 4 ? launch_bf16<4>(b, nxf, s) : fa == 6 ? launch_bf16<6>(b, nxf, s)
                                                                                                  : launch_bf16<8>(b, nxf, s);
    }
    if (err != hipSuccess || nsplit == 1 || a.keep_parts) return err;
    const int64_t n = a.T * a.E;
    if (n % 4 == 0 && (reinterpret_cast<uintptr_t>(a.logits) & 15) == 0) launch_reduce<f32x4_t>(a, nsplit, n / 4, s);
    else launch_reduce<float>(a, nsplit, n, s);
    return hipGetLastError();
}

}  // namespace craft
