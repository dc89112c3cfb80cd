// Expert weights in 8 bits: OCP FP8 E4M3 codes with one fp32 scale per weight row, and their
// re-ordering into the stream the packed FFN kernels read (see ffn_packed.hip).  Not part of
// a forward: this is model loading.
//
// E4M3: 1 sign bit, 4 exponent bits (bias 7), 3 mantissa bits; exponent field 0 is subnormal
// (mantissa / 8 * 2^-6); no infinities; S.1111.111 is NaN; the largest finite value is 448.
#include <algorithm>

#include "kernels.h"

namespace craft {
namespace {

constexpr int kQuantThreads = 256;

// Nearest E4M3 magnitude to a >= 0, ties to the even mantissa, saturating at 448.  The value
// grid inside one binade is 2^(e-3), so the mantissa is a rounded quotient; below 2^-6 the
// grid is 2^-9 throughout.  rintf rounds halves to even, which is the rule for the code too
// (the last mantissa bit is the last bit of the code, and a carry into the next binade lands
// on its first, even, value).
__device__ __forceinline__ uint32_t e4m3_magnitude(float a) {
    if (!(a < 448.0f)) return 0x7e;
    if (a < 0.015625f) return (uint32_t)rintf(a * 512.0f);          // 0..8; 8 is the smallest normal
    const int e = (int)((__float_as_uint(a) >> 23) & 0xff) - 127;   // floor(log2 a), a is normal here
    const int n = (int)rintf(ldexpf(a, 3 - e));                     // 8..16
    const uint32_t code = n == 16 ? (uint32_t)(e + 8) << 3 : ((uint32_t)(e + 7) << 3) | (uint32_t)(n - 8);
    return code > 0x7e ? 0x7e : code;
}

// A row's scale and what dividing by it takes.  The code of an element is decided by the
// correctly rounded fp32 quotient w / s.  With y the correctly rounded reciprocal of s and
// q = w y, the sum q + (w - s q) y is that quotient (Markstein 1990) unless an intermediate
// leaves the normal range: with s between 2^-60 and 2^60 none does for a quotient of 2^-10 or
// more, and everything below is code 0 either way.  Three operations instead of the ten or so
// of a division, which is what keeps the kernels below bound by memory.  Other rows (an
// infinity in them, or next to nothing) take the division.
struct RowScale {
    float s, inv;
    bool fast;
};
__device__ __forceinline__ RowScale row_scale(float amax) {
    RowScale r;
    r.s = amax > 0.0f ? amax / 448.0f : 1.0f;
    r.inv = 1.0f / r.s;
    r.fast = r.s >= 0x1p-60f && r.s <= 0x1p60f;
    return r;
}
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ float low_value(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float high_value(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }
__device__ __forceinline__ float max_abs(float m, const u32x4_t &w) {
#pragma unroll
    for (int i = 0; i < 4; ++i) m = fmaxf(fmaxf(m, fabsf(low_value(w[i]))), fabsf(high_value(w[i])));
    return m;
}
// The codes of 4 bf16 values (two words, low half first).
__device__ __forceinline__ uint32_t four_codes(uint32_t w0, uint32_t w1, const RowScale &r) {
    const float a[4] = {fabsf(low_value(w0)), fabsf(high_value(w0)), fabsf(low_value(w1)), fabsf(high_value(w1))};
    float q[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float q0 = a[i] * r.inv;
        q[i] = fminf(fmaf(fmaf(-r.s, q0, a[i]), r.inv, q0), 448.0f);      // a NaN saturates too
    }
    int c = __builtin_amdgcn_cvt_pk_fp8_f32(q[0], q[1], 0, false);        // nearest, ties to even
    c = __builtin_amdgcn_cvt_pk_fp8_f32(q[2], q[3], c, true);
    // the sign bits: the high bytes of the four halves
    return (uint32_t)c | (__builtin_amdgcn_perm(w1, w0, 0x07050301u) & 0x80808080u);
}
__device__ __forceinline__ uint32_t four_codes_divided(uint32_t w0, uint32_t w1, float s) {
    const float v[4] = {low_value(w0), high_value(w0), low_value(w1), high_value(w1)};
    uint32_t c = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float q = v[i] / s;
        c |= (e4m3_magnitude(fabsf(q)) | (__float_as_uint(q) >> 31 << 7)) << (8 * i);
    }
    return c;
}
__device__ __forceinline__ u32x2_t eight_codes(const u32x4_t &w, const RowScale &r) {
    u32x2_t c;
    if (r.fast) {
        c[0] = four_codes(w[0], w[1], r);
        c[1] = four_codes(w[2], w[3], r);
    } else {
        c[0] = four_codes_divided(w[0], w[1], r.s);
        c[1] = four_codes_divided(w[2], w[3], r.s);
    }
    return c;
}

// One workgroup per weight row: the row maximum, the scale, then the codes.  Bound by memory:
// 16-byte loads, all requested before the first is used, and the row stays in registers
// between the two passes over it (up to kKeep chunks per thread; what is longer is read again,
// out of the L2).
constexpr int kKeep = 4;
__global__ __launch_bounds__(kQuantThreads) void quantize_e4m3_kernel(const u32x4_t *w, int32_t chunks,
                                                                      u32x2_t *codes, float *scale) {
    __shared__ float part[kQuantThreads / 64];
    const int64_t r = blockIdx.x;
    const u32x4_t *row = w + r * chunks;
    u32x2_t *out = codes + r * chunks;
    u32x4_t keep[kKeep];
    const u32x4_t none = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int i = 0; i < kKeep; ++i) {
        const int c = i * kQuantThreads + threadIdx.x;
        keep[i] = c < chunks ? row[c] : none;
    }
    float amax = 0.0f;
#pragma unroll
    for (int i = 0; i < kKeep; ++i) amax = max_abs(amax, keep[i]);
    for (int c = kKeep * kQuantThreads + threadIdx.x; c < chunks; c += kQuantThreads) amax = max_abs(amax, row[c]);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) amax = fmaxf(amax, __shfl_xor(amax, off, 64));
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = amax;
    __syncthreads();
    amax = fmaxf(fmaxf(part[0], part[1]), fmaxf(part[2], part[3]));
    const RowScale rs = row_scale(amax);
    if (threadIdx.x == 0) scale[r] = rs.s;
#pragma unroll
    for (int i = 0; i < kKeep; ++i) {
        const int c = i * kQuantThreads + threadIdx.x;
        if (c < chunks) out[c] = eight_codes(keep[i], rs);
    }
    for (int c = kKeep * kQuantThreads + threadIdx.x; c < chunks; c += kQuantThreads) out[c] = eight_codes(row[c], rs);
}

// Quantisation and re-ordering in one pass over an expert's bf16 matrices: no codes in memory in
// between, one launch for the three matrices.  A workgroup owns 16 weight rows, which are one
// fragment of every 32-wide step: it finds the rows' maxima, keeps the rows in registers (a
// wave takes pairs of neighbouring steps, so that the four lanes of a row read whole 128-byte
// lines between the two; up to kPairs pairs per wave, K = 8192 at 1024 threads), and writes
// each step's fragment as 512 consecutive bytes.  Longer rows are read a second time.
// Bound by memory: 3 bytes per weight.  Sixteen waves with 14 requests of 1 KiB each keep
// enough in flight for one workgroup per CU.  At H = 7168, I = 2048: 28 us an expert, 4.7 TB/s
// (three quantisations, two re-orderings and two copies of scales: 128 us).  The streaming
// stores, whose lines nobody reads soon, are worth 34 -> 28 us; streaming loads lose 2 us of
// it (the two steps of a pair share lines), and workgroups of 8 waves or the down matrix first
// changed nothing.
constexpr int kPackThreads = 1024;
constexpr int kPackWaves = kPackThreads / 64;
struct QuantPackArgs {
    const unsigned short *w[3];    // gate, up [I][H]; down [H][I]
    unsigned char *gateup, *down;  // packed streams, the scales behind them
    int64_t gateup_stream, down_stream;   // bytes of the streams
    int32_t H, I;
    int32_t gateup_groups, down_groups;   // padded to whole tiles
    int32_t first;                        // row block of the launch's first workgroup
};
template <int PAIRS>
__device__ __forceinline__ void quantize_pack_rows(const unsigned short *rows, int live, int K, int ksteps,
                                                   unsigned char *out, int64_t step_bytes, float *scale,
                                                   float (&part)[kPackWaves][16]) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r = lane & 15, k_lane = 8 * (lane >> 4);
    const unsigned short *row = rows + (int64_t)min(r, live - 1) * K;
    const bool mine = r < live;
    // no branch around a request: what lies past the matrix is read from inside the row (which
    // changes no maximum) and stored as zeros
    auto fetch = [&](int step) __attribute__((always_inline)) {
        return *reinterpret_cast<const u32x4_t *>(row + min(32 * step + k_lane, K - 8));
    };
    constexpr int KEEP = PAIRS > 0 ? PAIRS : 1;
    u32x4_t keep[KEEP][2];
    float amax = 0.0f;
    if (PAIRS > 0) {
#pragma unroll
        for (int p = 0; p < PAIRS; ++p)
#pragma unroll
            for (int j = 0; j < 2; ++j) keep[p][j] = fetch(2 * (wave + kPackWaves * p) + j);
#pragma unroll
        for (int p = 0; p < PAIRS; ++p)
#pragma unroll
            for (int j = 0; j < 2; ++j) amax = max_abs(amax, keep[p][j]);
    } else {
        for (int s = 2 * wave; s < ksteps; s += 2 * kPackWaves) amax = max_abs(max_abs(amax, fetch(s)), fetch(s + 1));
    }
    amax = fmaxf(amax, __shfl_xor(amax, 16, 64));
    amax = fmaxf(amax, __shfl_xor(amax, 32, 64));
    if (lane < 16) part[wave][lane] = amax;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kPackWaves; ++w) amax = fmaxf(amax, part[w][r]);
    RowScale rs = row_scale(amax);
    if (threadIdx.x < live) scale[threadIdx.x] = rs.s;        // live <= 16: lanes of the first wave
    auto put = [&](int step, const u32x4_t &w) __attribute__((always_inline)) {
        const u32x2_t zero = {0u, 0u};
        __builtin_nontemporal_store(mine && 32 * step + k_lane < K ? eight_codes(w, rs) : zero,
                                    reinterpret_cast<u32x2_t *>(out + step * step_bytes + lane * 8));
    };
    if (PAIRS > 0 && __all(rs.fast)) {
        rs.fast = true;                            // known from here on: no division beside each store
#pragma unroll
        for (int p = 0; p < PAIRS; ++p)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int s = 2 * (wave + kPackWaves * p) + j;
                if (s < ksteps) put(s, keep[p][j]);
            }
    } else {
        for (int s = 2 * wave; s < ksteps; s += 2 * kPackWaves) {
            put(s, fetch(s));
            put(s + 1, fetch(s + 1));
        }
    }
}
__global__ __launch_bounds__(kPackThreads) void quantize_pack_e4m3_kernel(QuantPackArgs a) {
    __shared__ float part[kPackWaves][16];
    int b = a.first + blockIdx.x;
    const bool gateup = b < 2 * a.gateup_groups;
    if (!gateup) b -= 2 * a.gateup_groups;
    const int g = b >> 1, h = b & 1;
    const int K = gateup ? a.H : a.I, N = gateup ? a.I : a.H;
    const int ksteps = (K + 255) / 256 * 8;
    const int64_t step_bytes = (int64_t)(gateup ? a.gateup_groups : a.down_groups) * 1024;
    const int row0 = gateup ? 16 * g : 32 * g + 16 * h;
    unsigned char *out = (gateup ? a.gateup : a.down) + (int64_t)g * 1024 + h * 512;
    if (row0 >= N) {                               // padding groups: zero codes
        const u32x2_t zero = {0u, 0u};
        for (int s = threadIdx.x >> 6; s < ksteps; s += kPackWaves)
            *reinterpret_cast<u32x2_t *>(out + s * step_bytes + (threadIdx.x & 63) * 8) = zero;
        return;
    }
    const unsigned short *rows = (gateup ? a.w[h] : a.w[2]) + (int64_t)row0 * K;
    float *scale = reinterpret_cast<float *>(gateup ? a.gateup + a.gateup_stream : a.down + a.down_stream) +
                   (gateup ? h * N : 0) + row0;
    const int live = min(16, N - row0);
    const int pairs = (ksteps / 2 + kPackWaves - 1) / kPackWaves;
    if (pairs <= 2) quantize_pack_rows<2>(rows, live, K, ksteps, out, step_bytes, scale, part);
    else if (pairs <= 4) quantize_pack_rows<4>(rows, live, K, ksteps, out, step_bytes, scale, part);
    else if (pairs <= 8) quantize_pack_rows<8>(rows, live, K, ksteps, out, step_bytes, scale, part);
    else quantize_pack_rows<0>(rows, live, K, ksteps, out, step_bytes, scale, part);
}

// One 8-byte chunk of the packed stream per thread: the layout of the bf16 stream (step-major,
// 8 column groups per tile, two 16-row fragments per group, 64 lanes per fragment), with 8 codes
// where it has 8 bf16 values.
//   gate/up : group g = output columns 16g..16g+15; half 0 = gate rows 16g..16g+15, half 1 = the
//             up rows of the same columns
//   down    : group g = output columns 32g..32g+31; half h = down rows 32g+16h..+15
// Lane l of 32-wide step s holds row (l & 15) of its half, contraction elements 32s + 8(l>>4) .. +7.
__global__ void pack_e4m3_kernel(const uint8_t *ca, const uint8_t *cb, int rows, int K, int gc,
                                 int64_t nchunks, int ksteps, uint2 *out) {
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= nchunks) return;
    const int l = (int)(c & 63);
    const int h = (int)(c >> 6) & 1;
    const int64_t sg = c >> 7;
    const int64_t ngroups = nchunks / 128 / ksteps;
    const int s = (int)(sg / ngroups);
    const int64_t g = sg % ngroups;
    const int r = l & 15;
    const int k0 = 32 * s + 8 * (l >> 4);
    int64_t row;
    const uint8_t *src;
    if (gc == 16) { row = g * 16 + r; src = h ? cb : ca; }
    else { row = g * 32 + 16 * h + r; src = ca; }
    uint2 v = make_uint2(0, 0);
    if (row < rows && k0 < K) v = *reinterpret_cast<const uint2 *>(src + row * K + k0);
    out[c] = v;
}

__global__ void copy_scales_kernel(const float *a, const float *b, int n, float *out) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = a[i];
    else if (b && i < 2 * n) out[i] = b[i - n];
}

}  // namespace

void packed_sizes_e4m3(int32_t H, int32_t I, size_t *gateup_bytes, size_t *down_bytes) {
    const size_t gu_groups = ((size_t)(I + 15) / 16 + 7) / 8 * 8, gu_steps = (size_t)(H + 255) / 256 * 16;
    const size_t dn_groups = ((size_t)(H + 31) / 32 + 7) / 8 * 8, dn_steps = (size_t)(I + 255) / 256 * 16;
    *gateup_bytes = gu_groups * gu_steps * 512 + (size_t)2 * I * sizeof(float);
    *down_bytes = dn_groups * dn_steps * 512 + (size_t)H * sizeof(float);
}

hipError_t launch_quantize_e4m3(const void *w, int64_t rows, int32_t K, uint8_t *codes, float *scale,
                                hipStream_t s) {
    // a launch has fewer than 2^32 threads
    constexpr int64_t kMost = (1ll << 31) / kQuantThreads;
    for (int64_t r = 0; r < rows; r += kMost) {
        hipLaunchKernelGGL(quantize_e4m3_kernel, dim3((unsigned)std::min(kMost, rows - r)), dim3(kQuantThreads), 0, s,
                           static_cast<const u32x4_t *>(w) + r * (K / 8), K / 8, reinterpret_cast<u32x2_t *>(codes) + r * (K / 8), scale + r);
    }
    return hipGetLastError();
}

hipError_t launch_quantize_pack_e4m3(int32_t H, int32_t I, const void *wg, const void *wu, const void *wd,
                                     void *pgu, void *pdn, hipStream_t s) {
    size_t gub, dnb;
    packed_sizes_e4m3(H, I, &gub, &dnb);
    QuantPackArgs a{{static_cast<const unsigned short *>(wg), static_cast<const unsigned short *>(wu),
                     static_cast<const unsigned short *>(wd)},
                    static_cast<unsigned char *>(pgu), static_cast<unsigned char *>(pdn),
                    (int64_t)(gub - (size_t)2 * I * sizeof(float)), (int64_t)(dnb - (size_t)H * sizeof(float)),
                    H, I, ((I + 15) / 16 + 7) / 8 * 8, ((H + 31) / 32 + 7) / 8 * 8, 0};
    constexpr int32_t kMost = (1ll << 31) / kPackThreads;
    const int32_t blocks = 2 * (a.gateup_groups + a.down_groups);
    for (; a.first < blocks; a.first += kMost)
        hipLaunchKernelGGL(quantize_pack_e4m3_kernel, dim3((unsigned)std::min(kMost, blocks - a.first)), dim3(kPackThreads), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_pack_e4m3(int32_t H, int32_t I, const uint8_t *cg, const uint8_t *cu, const uint8_t *cd,
                            const float *sg, const float *su, const float *sd, void *pgu, void *pdn,
                            hipStream_t s) {
    size_t gub, dnb;
    packed_sizes_e4m3(H, I, &gub, &dnb);
    const size_t gu_stream = gub - (size_t)2 * I * sizeof(float), dn_stream = dnb - (size_t)H * sizeof(float);
    const int64_t c1 = (int64_t)(gu_stream / 8), c2 = (int64_t)(dn_stream / 8);
    hipLaunchKernelGGL(pack_e4m3_kernel, dim3((unsigned)((c1 + 255) / 256)), dim3(256), 0, s, cg, cu, I, H,
                       16, c1, (H + 255) / 256 * 8, static_cast<uint2 *>(pgu));
    hipLaunchKernelGGL(pack_e4m3_kernel, dim3((unsigned)((c2 + 255) / 256)), dim3(256), 0, s, cd, cd, H, I,
                       32, c2, (I + 255) / 256 * 8, static_cast<uint2 *>(pdn));
    float *gus = reinterpret_cast<float *>(static_cast<unsigned char *>(pgu) + gu_stream);
    float *dns = reinterpret_cast<float *>(static_cast<unsigned char *>(pdn) + dn_stream);
    hipLaunchKernelGGL(copy_scales_kernel, dim3((unsigned)((2 * I + 255) / 256)), dim3(256), 0, s, sg, su, I, gus);
    hipLaunchKernelGGL(copy_scales_kernel, dim3((unsigned)((H + 255) / 256)), dim3(256), 0, s, sd,
                       static_cast<const float *>(nullptr), H, dns);
    return hipGetLastError();
}

}  // namespace craft
