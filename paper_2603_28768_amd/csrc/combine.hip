// Gather-weighted combine: the last step of the MoE layer of Sec. 2.1, each token's sum of
// its experts' outputs scaled by the routing weights.  A 64-lane wavefront takes a piece of a token's row, 2 or 3 KiB; a lane owns
// 16-byte column chunks of it.  Only assignments whose dispatched position falls inside this rank's row range
// contribute, added in ascending j with fp32 accumulation; there are no atomics, so the
// result does not depend on scheduling.  Tokens with no assignment on the rank get zeros.
//
// A large batch is bound by HBM (mostly zero rows to write), a small one by its chain of round trips on
// the few CUs that have a wave.  A forward (bf16, E = 64, k = 4, I = 64, one of eight ranks) with whole rows
// per wave (8 KiB a round) / in pieces, us: H = 7168, 40 tokens 28.5 / 25.9, 256 40.8 / 37.7, 1024 100.6 / 99.2,
// 8192 141.6 / 139.9; H = 1024, 4096 tokens 47.6 / 45.7, 32768 96.7 / 80.4; H = 4096, 8192 tokens the same.
#include <hip/hip_bf16.h>

#include <algorithm>

#include "kernels.h"

namespace craft {
namespace {

// A 16-byte piece of a row as it is loaded, and how it unpacks to fp32 / packs from it.
template <typename T> struct Chunk;
template <> struct Chunk<float> {
    static constexpr int N = 4;
    __device__ static void unpack(const uint4 &q, float (&v)[4]) {
        v[0] = __uint_as_float(q.x); v[1] = __uint_as_float(q.y);
        v[2] = __uint_as_float(q.z); v[3] = __uint_as_float(q.w);
    }
    __device__ static uint4 pack(const float (&v)[4]) {
        return make_uint4(__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2]),
                          __float_as_uint(v[3]));
    }
};
template <> struct Chunk<__hip_bfloat16> {
    static constexpr int N = 8;
    __device__ static void unpack(const uint4 &q, float (&v)[8]) {
        const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            v[2 * i] = __uint_as_float(w[i] << 16);
            v[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
        }
    }
    __device__ static uint32_t rne(float f) {       // fp32 -> bf16 bits, nearest even
        const uint32_t u = __float_as_uint(f);
        return (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
    }
    __device__ static uint4 pack(const float (&v)[8]) {
        uint4 q;
        q.x = rne(v[0]) | (rne(v[1]) << 16);
        q.y = rne(v[2]) | (rne(v[3]) << 16);
        q.z = rne(v[4]) | (rne(v[5]) << 16);
        q.w = rne(v[6]) | (rne(v[7]) << 16);
        return q;
    }
};

// A wave takes 64 U chunks of one token's row, one request round; the `parts` waves of a row sit in
// neighbouring workgroups.  `first`: the launch's first token.
template <typename T, int U>
__global__ __launch_bounds__(256) void combine_kernel(CombineArgs a, uint32_t parts, int64_t first) {
    constexpr int N = Chunk<T>::N;
    const int lane = threadIdx.x & 63;
    const uint32_t tokens = blockIdx.x / parts, part = blockIdx.x - tokens * parts;
    const int64_t t = first + (int64_t)tokens * 4 + (threadIdx.x >> 6);
    if (t >= a.T) return;
    const int32_t lo = a.slot_off[a.s_lo], hi = a.slot_off[a.s_hi];
    const bool dead = a.ctrl[CTRL_OVERFLOW] != 0;
    int32_t d = -1;
    float wj = 0.0f;
    if (lane < a.k) {
        d = a.dest[t * a.k + lane];
        wj = a.w[t * a.k + lane];
    }
    const bool mine = !dead && lane < a.k && d >= lo && d < hi;
    const unsigned long long live = __ballot(mine);
    const T *y = static_cast<const T *>(a.y);
    T *out = static_cast<T *>(a.out) + t * a.H;
    // A lane past the end of the row only skips its loads and its store (shuffles need every lane).
    // The rows of up to G assignments are requested together before any of them is added (in
    // ascending j, as always): what a wave takes is a chain of memory latencies, one per round
    // of requests, and a token of the busiest rank has several of its experts there.
    constexpr int G = 4;
    int c0[U];
    bool inside[U];
    float acc[U][N];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int chunk = (int)part * U * 64 + u * 64 + lane;
        inside[u] = chunk < a.H / N;
        c0[u] = chunk * N;
#pragma unroll
        for (int i = 0; i < N; ++i) acc[u][i] = 0.0f;
    }
    unsigned long long m = live;
    while (m) {
        const T *row[G];
        float wv[G];
        int n = 0;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            row[g] = y;
            wv[g] = 0.0f;
            if (m) {
                const int j = __ffsll((long long)m) - 1;
                m &= m - 1;
                row[g] = y + (int64_t)(__shfl(d, j, 64) - lo) * a.H;
                wv[g] = __shfl(wj, j, 64);
                n = g + 1;
            }
        }
        uint4 raw[G][U];
#pragma unroll
        for (int g = 0; g < G; ++g)
            if (g < n) {
#pragma unroll
                for (int u = 0; u < U; ++u)
                    raw[g][u] = inside[u] ? *reinterpret_cast<const uint4 *>(row[g] + c0[u])
                                          : make_uint4(0, 0, 0, 0);
            }
#pragma unroll
        for (int g = 0; g < G; ++g)
            if (g < n) {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    float v[N];
                    Chunk<T>::unpack(raw[g][u], v);
#pragma unroll
                    for (int i = 0; i < N; ++i) acc[u][i] += wv[g] * v[i];
                }
            }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (inside[u]) {
            // written once and not read again by this launch: a streaming store
            typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
            const uint4 q = Chunk<T>::pack(acc[u]);
            const u32x4 v = {q.x, q.y, q.z, q.w};
            __builtin_nontemporal_store(v, reinterpret_cast<u32x4 *>(out + c0[u]));
        }
}

template <typename T, int U>
void launch_pieces(const CombineArgs &a, hipStream_t s) {
    constexpr int64_t kRow = 64 * Chunk<T>::N * U;
    const int64_t parts = (a.H + kRow - 1) / kRow, groups = (a.T + 3) / 4;
    // a launch has fewer than 2^32 threads (of one with more only the remainder runs, without an error)
    const int64_t most = std::max<int64_t>(1, (1ll << 31) / 256 / parts);
    for (int64_t g = 0; g < groups; g += most)
        hipLaunchKernelGGL((combine_kernel<T, U>), dim3((unsigned)(std::min(most, groups - g) * parts)), dim3(256), 0, s, a,
                           (uint32_t)parts, g * 4);
}

// Pieces of 2 KiB, or of 3 KiB where the last one of 2 would be a wave for little: a row of 2 to 2.5 KiB,
// and in a large batch, bound by what its waves write, a row of more than three pieces whose last one is
// not full, unless pieces of 3 KiB leave yet more lanes idle (by more than a request of one wave).  The
// forward above, pieces of 2 / 3 KiB, us: H = 1032, 64 tokens 19.4 / 19.2, 1024 42.5 / 40.1, 32768 99.0 / 91.0;
// H = 3080, 4096 tokens 87.4 / 84.8, 32768 182.5 / 169.9 (whole rows 174.3); H = 3592, 16384 140.7 / 136.1 (136.8);
// H = 7176, 16384 247.9 / 243.3 (244.3).  Not H = 2056, 32768 tokens 130.9 / 134.5, H = 4616, 16384 166.4 / 170.5,
// nor few tokens: H = 3080, 8 tokens 18.1 / 18.3, 2048 77.3 / 78.3.
template <typename T>
void launch_rows(const CombineArgs &a, hipStream_t s) {
    const int64_t chunks = a.H / Chunk<T>::N, two = (chunks + 127) / 128 * 128, three = (chunks + 191) / 192 * 192;
    if ((chunks > 128 && chunks <= 160) || (a.T >= 4096 && chunks > 384 && chunks < two && three <= two + 64)) launch_pieces<T, 3>(a, s);
    else launch_pieces<T, 2>(a, s);
}

}  // namespace

hipError_t launch_combine(const CombineArgs &a, hipStream_t s) {
    if (a.T == 0) return hipSuccess;
    if (a.dtype == CRAFT_F32) launch_rows<float>(a, s);
    else launch_rows<__hip_bfloat16>(a, s);
    return hipGetLastError();
}

}  // namespace craft
