// Gating-network scores, the input of top-K routing (Sec. 2.1).  The paper leaves the form of
// the network open; this is the usual linear gate,
//   logits[t][e] = sum_h x[t][h] * Wr[e][h],
// both operands contiguous along the contraction, fp32 accumulation, fp32 scores.  The top-k
// step consumes these scores exactly as it consumes scores handed in from outside.
//
// A skinny GEMM: few output columns (E = 128 .. 384), so the tokens' activations are what
// has to cross HBM (once) and the gate's weights are re-read from L2 by every workgroup.
// bf16: 32, 64 or 128 tokens against up to 256 experts per workgroup (nt_tile.h), the experts as the
// matrix instruction's row operand, so that a lane holds four neighbouring experts of a token:
// 16-byte stores.  Every workgroup pulls the whole gate out of L2, so T H 2 (1 + E / tokens per
// workgroup) bytes move from L2 into the CUs; taller workgroups move less but there are only
// T / 128 of them, so with a workspace the contraction is split over up to 8 workgroups per tile:
// each writes its partial scores and a second kernel (or the routing kernel) adds them in ascending
// order of the split (a fixed order: the result does not depend on scheduling).
// fp32: one thread per score, a plain chain of fused multiply-adds (small configurations).
#include "nt_tile.h"

namespace craft {
namespace {

// Tokens up to which the gate is read by thin tiles: few tall ones leave CUs without work (8 tokens:
// 23 us for scores of E = 256, H = 7168, thin 4.4).  From there on it depends on E, thin / tall with the
// sum of the parts at 192 tokens: E = 256 16.5 / 19.4, E = 128 14.4 / 13.5, E = 384 21.4 / 16.6; at 1024
// tokens 45 / 22.
constexpr int kThinBatch = 128;
constexpr int GK = 64;                  // contraction slab
typedef unsigned int gu32x4_t __attribute__((ext_vector_type(4)));
typedef const gu32x4_t __attribute__((address_space(1))) *gchunk_t;

template <int FA, int FB>
__global__ __launch_bounds__(kNtThreads) void router_logits_bf16_kernel(RouterArgs a) {
    __shared__ __attribute__((aligned(16))) unsigned char gate_smem[nt_lds_bytes<FA, FB>()];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int64_t t0 = (int64_t)blockIdx.x * (FB * 32);
    const int e0 = blockIdx.y * (FA * 32);
    // this workgroup's share of the contraction (may be empty)
    const int nk = (a.H + GK - 1) / GK, per = (nk + a.nsplit - 1) / a.nsplit;
    const int kbeg = min(nk, (int)blockIdx.z * per), kend = min(nk, kbeg + per);
    float *dst = a.nsplit > 1 ? a.part + (int64_t)blockIdx.z * a.T * a.E : a.logits;
    // rows past the end are clamped into the matrix (their results are not stored)
    auto eoff = [&](int i) { return (uint32_t)min(i, a.E - 1 - e0) * (uint32_t)a.H * 2u; };
    auto toff = [&](int i) { return (uint32_t)min((int64_t)i, a.T - 1 - t0) * (uint32_t)a.H * 2u; };
    f32x4_t acc[FA][FB];
#pragma unroll
    for (int f = 0; f < FA; ++f)
#pragma unroll
        for (int g = 0; g < FB; ++g) acc[f][g] = (f32x4_t)(0.0f);
    nt_tile<FA, FB>(gate_smem, uniform_base(static_cast<ubase_t>(a.w) + (int64_t)e0 * a.H * 2), eoff,
                    uniform_base(static_cast<ubase_t>(a.x) + t0 * a.H * 2), toff, a.H, kbeg, kend, acc);
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
    const int nk = (a.H + GK - 1) / GK, per = (nk + a.nsplit - 1) / a.nsplit;
    const int kbeg = min(nk, (int)blockIdx.z * per), kend = min(nk, kbeg + per);
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
    const dim3 grid((unsigned)((a.T + FB * 32 - 1) / (FB * 32)), (unsigned)((a.E + FA * 32 - 1) / (FA * 32)), (unsigned)a.nsplit);
    hipLaunchKernelGGL((router_logits_bf16_kernel<FA, FB>), grid, dim3(kNtThreads), 0, s, a);
    return hipGetLastError();
}
template <int FA>
hipError_t launch_bf16(const RouterArgs &a, int nxf, hipStream_t s) {
    return nxf == 1 ? launch_bf16<FA, 1>(a, s) : nxf == 2 ? launch_bf16<FA, 2>(a, s) : launch_bf16<FA, 4>(a, s);
}

}  // namespace

// Tile height (32-token fragments per workgroup) and split of the contraction for a shape.
// Without a workspace: short tiles, as many as there are CUs if possible.  With one: the
// tallest tile, and as many splits as bring the workgroups up to the CU count (at most 8, at least 4
// slabs each).  Workgroups are counted in blocks of up to 384 experts, not the 256 of a tile, and more
// than 384 experts are never split: 257 to 384 get twice the workgroups this aims at (T = 16384, E = 384:
// 512, two rounds), more get short tiles.  No shape is slower for it than with the tiles of 512
// experts that the count was made for.
void router_logits_shape(int64_t T, int32_t H, int32_t E, int32_t num_cu, bool workspace, int *nxf, int *nsplit) {
    const int nb = E > 512 ? 4 : (E + 127) / 128;
    *nsplit = 1;
    if (!workspace || nb > 3) {
        *nxf = nb <= 3 && (T + 63) / 64 >= (int64_t)num_cu ? 2 : 1;
        return;
    }
    *nxf = 4;
    const int64_t tiles = (T + 127) / 128 * ((E + nb * 128 - 1) / (nb * 128));
    const int nk = (H + GK - 1) / GK;
    int sp = 1;
    while (sp < 8 && tiles * sp * 2 <= num_cu && nk / (sp * 2) >= 4) sp *= 2;
    *nsplit = sp;
}

hipError_t launch_router_logits(const RouterArgs &a, hipStream_t s) {
    if (a.T == 0) return hipSuccess;
    if (a.dtype == CRAFT_F32) {
        const int64_t n = a.T * a.E;
        hipLaunchKernelGGL(router_logits_f32_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, a);
        return hipGetLastError();
    }
    int nxf, nsplit;
    router_logits_shape(a.T, a.H, a.E, a.num_cu, a.part != nullptr, &nxf, &nsplit);
    RouterArgs b = a;
    b.nsplit = nsplit;
    hipError_t err;
    if (a.T <= kThinBatch || a.H >= kNtRowLimit) {         // (thin tiles take rows of any length)
        const dim3 grid((unsigned)((a.E + 15) / 16), (unsigned)((a.T + kThinTokens - 1) / kThinTokens), (unsigned)nsplit);
        hipLaunchKernelGGL(router_thin_kernel, grid, dim3(64 * kThinWaves), 0, s, b);
        err = hipGetLastError();
    } else {
        // blocks of up to 256 experts, as even as they come
        const int blocks = (a.E + 255) / 256, rows = (a.E + blocks - 1) / blocks;
        err = rows <= 64 ? launch_bf16<2>(b, nxf, s) : rows <= 128 ? launch_bf16<4>(b, nxf, s)
              : rows <= 192 ? launch_bf16<6>(b, nxf, s) : launch_bf16<8>(b, nxf, s);
    }
    if (err != hipSuccess || nsplit == 1 || a.keep_parts) return err;
    const int64_t n = a.T * a.E;
    if (n % 4 == 0 && (reinterpret_cast<uintptr_t>(a.logits) & 15) == 0) launch_reduce<f32x4_t>(a, nsplit, n / 4, s);
    else launch_reduce<float>(a, nsplit, n, s);
    return hipGetLastError();
}

}  // namespace craft
