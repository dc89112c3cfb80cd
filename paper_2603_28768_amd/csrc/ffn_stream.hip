// Grouped SwiGLU expert FFN of a small batch: every slot has few rows, so the two GEMMs of the
// expert FFN (Sec. 2.1) are nothing but streaming the live slots' weights through the chip once.
//
// The tiles of ffn_packed.hip give a slot 2 nt workgroups (64 per GEMM with two live slots of
// H = 7168, I = 2048), which leaves most CUs without a weight to fetch.  Here the unit of work
// is one column group (32 weight rows) of one slot against up to 64 of its rows, and the four
// waves of a workgroup share its contraction: wave w takes the 64-wide slabs w, w + 4, ..  Two
// live slots make 256 units of the gate/up GEMM and 448 of the down GEMM.  Bound by memory: a
// wave keeps whole slabs in flight in registers (PW of them, 4 KiB of weights each), weights
// and activation rows alike straight from global memory in the operand layout of
// v_mfma_f32_16x16x32_bf16: nothing is shared between the waves before the end, so the loop has
// neither LDS nor barriers, and two workgroups per CU cover one another's start and end.  The
// waves' partial sums meet in LDS and are added in wave order (a fixed order).  Two slots of a row or
// two: gate/up 48.6 -> 19.6 us, down 18.4 -> 11.7; three of a dozen rows in E4M3: 40.6 -> 18.3 (4.8 TB/s of
// codes) and 16.0 -> 11.4.
//
// Weights are the packed streams (bf16 or E4M3) or the row-major matrices themselves: 16 rows
// of 64 bytes per request, the two steps of a slab completing their 128-byte lines.
#include "ffn_common.h"

namespace craft {
namespace {

constexpr int kWaves = 4;
constexpr int kThreads = 64 * kWaves;
constexpr int kMaxNXF = kStreamRows / 16;
enum { kPackedBf16 = 0, kPackedE4M3 = 1, kRowMajor = 2 };

// Slabs in flight per wave: what fits 256 registers beside the accumulators (a slab is 16
// registers of weights, 8 as E4M3 codes, and 8 of activations per 16 rows).  Plain loads: with
// streaming ones a forward with two slots of 57 and 52 rows took 90 us instead of 80.
constexpr int ring_slabs(int src, int nxf) {
    return nxf == 1 ? 8 : nxf == 2 ? 6 : src == kPackedE4M3 ? 4 : 3;
}

struct Unit {
    int slot, group;           // slot of the rank, column group
    int row, m0, rows;         // the slot's first row among the rank's; the unit's rows inside the slot
    ubase_t w[2];              // the slot's weights (row-major gate/up: gate and up)
};

template <bool GATEUP, int SRC, int NXF>
__device__ __forceinline__ void stream_unit(const FfnArgs &a, const Unit &t, int K, int N, int wave, f32x4_t *part) {
    const int group = t.group;
    constexpr bool W8 = SRC == kPackedE4M3;
    constexpr int PW = ring_slabs(SRC, NXF);
    constexpr int GC = GATEUP ? 16 : 32;
    typedef typename WFrag<W8>::type F;
    const int lane = threadIdx.x & 63, q = lane >> 4, r16 = lane & 15;
    const uint32_t row_bytes = (uint32_t)K * 2u;

    // activation fragments: 1 KiB per 16 rows and step, in operand order
    const uint32_t xfrag = (uint32_t)((K + 63) / 64) * 2048u;
    const int32_t frag0 = stream_fragment(t.row, t.slot, t.m0);
    const ubase_t xb = uniform_base(static_cast<ubase_t>(GATEUP ? a.xpk : a.act) + (int64_t)frag0 * xfrag);
    uint32_t xl[NXF];
#pragma unroll
    for (int g = 0; g < NXF; ++g) xl[g] = (uint32_t)lane * 16u + (uint32_t)g * xfrag;

    // weights: a base per half plus the lane's 32-bit offset
    const int groups_padded = ((N + GC - 1) / GC + kPackGroups - 1) / kPackGroups * kPackGroups;
    const uint32_t wstep = (uint32_t)groups_padded * 128u * (uint32_t)sizeof(F);
    const ubase_t *wb = t.w;
    uint32_t wl[2];
#pragma unroll
    for (int h = 0; h < 2; ++h)
        wl[h] = SRC == kRowMajor ? (uint32_t)min(group * GC + (GATEUP ? 0 : 16 * h) + r16, N - 1) * row_bytes
                                 : (uint32_t)(group * 128 + lane) * (uint32_t)sizeof(F);

    F w[PW][2][2];
    bf16x8_t x[PW][2][NXF];
    f32x4_t acc[2][NXF];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int g = 0; g < NXF; ++g) acc[h][g] = (f32x4_t)(0.0f);

    // This wave's slabs are wave, wave + kWaves, ..: n of them.  The slab requested next and the
    // one multiplied next are running scalars that the compiler is not to take apart: it would
    // keep the addresses of a whole trip of the loop in registers.
    const int nslabs = (K + 63) / 64;
    const int n = (nslabs - wave + kWaves - 1) / kWaves;
    int next = wave, now = wave;
    auto request = [&](int u) __attribute__((always_inline)) {
        asm volatile("" : "+s"(next));
        // row-major weights: past the end of a row the lane reads from inside it
        const uint32_t k0 = (uint32_t)next * 128u + (uint32_t)q * 16u, kend = row_bytes - 16u;
        const uint32_t koff[2] = {k0 < kend ? k0 : kend, k0 + 64u < kend ? k0 + 64u : kend};
        const uint32_t off = (uint32_t)next * 2u * wstep;       // the packed matrix stays below 4 GiB
#pragma unroll
        for (int st = 0; st < 2; ++st)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                if (SRC == kRowMajor) {
                    uint32_t o = wl[h] + koff[st];
                    w[u][st][h] = wload<false, F>(wb[h], o);
                } else {
                    w[u][st][h] = wload<false, F>(wb[0] + (off + (uint32_t)st * wstep + (uint32_t)h * 64u * (uint32_t)sizeof(F)), wl[0]);
                }
            }
#pragma unroll
        for (int st = 0; st < 2; ++st)
#pragma unroll
            for (int g = 0; g < NXF; ++g)
                x[u][st][g] = wload<false, bf16x8_t>(xb + ((uint32_t)next * 2048u + (uint32_t)st * 1024u), xl[g]);
        next += kWaves;
    };
    auto multiply = [&](int u) __attribute__((always_inline)) {
        asm volatile("" : "+s"(now));
#pragma unroll
        for (int st = 0; st < 2; ++st) {
            // past the contraction packed weights are zero, row-major ones are replaced by zeros,
            // and so are the activations: nothing was written there
            const bool past = (uint32_t)(now * 128 + st * 64 + q * 16) >= row_bytes;
            if (past)
#pragma unroll
                for (int g = 0; g < NXF; ++g) x[u][st][g] = bf16x8_t{};
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                bf16x8_t wf = widen(w[u][st][h]);
                if (past && SRC == kRowMajor) wf = bf16x8_t{};
#pragma unroll
                for (int g = 0; g < NXF; ++g)
                    acc[h][g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf, x[u][st][g], acc[h][g], 0, 0, 0);
            }
        }
        now += kWaves;
    };
    if (n >= PW) {
        // no branch around a request while the ring is full: the waits count requests, and
        // have to find the same number on every path
#pragma unroll
        for (int u = 0; u < PW; ++u) { request(u); __builtin_amdgcn_sched_barrier(0); }
        int left = n - PW;
        for (; left >= PW; left -= PW)
#pragma unroll
            for (int u = 0; u < PW; ++u) {
                multiply(u);
                request(u);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
        for (int u = 0; u < PW; ++u) {
            multiply(u);
            if (u < left) request(u);
        }
#pragma unroll
        for (int u = 0; u < PW - 1; ++u)
            if (u < left) multiply(u);
    } else {
#pragma unroll
        for (int u = 0; u < PW - 1; ++u)
            if (u < n) request(u);
#pragma unroll
        for (int u = 0; u < PW - 1; ++u)
            if (u < n) multiply(u);
    }

    // Sum over the waves.  Element v of lane l is weight row 4 (l >> 4) + v of its half and row
    // l & 15 of its fragment: a thread adds up four neighbouring columns of one row.
    constexpr int PIECES = 2 * NXF;
    __syncthreads();                               // the last unit's sums have been read
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int g = 0; g < NXF; ++g) part[(wave * PIECES + h * NXF + g) * 64 + lane] = acc[h][g];
    __syncthreads();
    auto total = [&](int piece) __attribute__((always_inline)) {
        f32x4_t s = part[piece * 64 + lane];
#pragma unroll
        for (int v = 1; v < kWaves; ++v) s += part[(v * PIECES + piece) * 64 + lane];
        return s;
    };
    const float *scale = nullptr;                  // E4M3: row scales behind the codes
    if (W8) scale = reinterpret_cast<const float *>(wb[0] + (size_t)((K + 255) / 256 * 8) * wstep);
    for (int piece = wave; piece < (GATEUP ? NXF : PIECES); piece += kWaves) {
        const int g = piece % NXF, h = piece / NXF;
        const int m = 16 * g + r16, col = group * GC + 16 * h + 4 * q;
        f32x4_t v = total(piece);
        if (GATEUP) {
            f32x4_t up = total(NXF + piece);
            if (W8 && col < N) {
                v *= *reinterpret_cast<const f32x4_t *>(scale + col);
                up *= *reinterpret_cast<const f32x4_t *>(scale + N + col);
            }
#pragma unroll
            for (int c = 0; c < 4; ++c) v[c] = (SRC == kRowMajor ? silu(v[c]) : silu_fast(v[c])) * up[c];   // as the tiles of each
        } else if (W8 && col < N) {
            v *= *reinterpret_cast<const f32x4_t *>(scale + col);
        }
        if (m < t.rows && col < N) {
            // gate/up: into the fragments that the down GEMM reads
            unsigned char *dst = GATEUP ? static_cast<unsigned char *>(a.act) + (int64_t)(frag0 + g) * ((uint32_t)((N + 63) / 64) * 2048u) +
                                              stream_piece((uint32_t)col >> 3, r16) + (col & 4) * 2
                                        : static_cast<unsigned char *>(a.y) + ((int64_t)(t.row + t.m0 + m) * N + col) * 2;
            *reinterpret_cast<uint2 *>(dst) = make_uint2(bf16_pair(v[0], v[1]), bf16_pair(v[2], v[3]));
        }
    }
}

// What a workgroup looks up for its units, copied to LDS in one round trip.
struct StreamTables {
    static constexpr int kMaxSlots = 256;
    int32_t mt_start[kMaxSlots + 1], order[kMaxSlots], slot_off[kMaxSlots + 1];
    const void *w[2][kMaxSlots];
};

template <bool GATEUP, int SRC>
__global__ __launch_bounds__(kThreads, 2) void ffn_stream_kernel(FfnArgs a) {
    __shared__ f32x4_t part[kWaves * 2 * kMaxNXF * 64];
    __shared__ StreamTables tt;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int32_t *mt_start = a.mt_start + (GATEUP ? 0 : a.nslots + 1);
    const void *const *w0 = SRC == kRowMajor ? (GATEUP ? a.w_gate : a.w_down) : GATEUP ? a.wp_gateup : a.wp_down;
    const void *const *w1 = SRC == kRowMajor && GATEUP ? a.w_up : w0;
    const bool small = a.nslots <= StreamTables::kMaxSlots;
    if (small) {
        for (int i = threadIdx.x; i <= a.nslots; i += kThreads) {
            // (no branch around a load)
            const int last = min(i, a.nslots - 1);
            const int32_t start = mt_start[i], off = a.slot_off[a.s_lo + i], slot = a.order[last];
            const void *p0 = w0[last], *p1 = w1[last];
            tt.mt_start[i] = start;
            tt.slot_off[i] = off;
            tt.order[last] = slot;
            tt.w[0][last] = p0;
            tt.w[1][last] = p1;
        }
        __syncthreads();
    }
    auto mt_at = [&](int i) { return small ? tt.mt_start[i] : mt_start[i]; };
    auto off_at = [&](int i) { return small ? tt.slot_off[i] : a.slot_off[a.s_lo + i]; };
    const int K = GATEUP ? a.H : a.I, N = GATEUP ? a.I : a.H;
    constexpr int GC = GATEUP ? 16 : 32;
    const int ngroups = (N + GC - 1) / GC;
    const int total = mt_at(a.nslots) * ngroups;           // small_dispatch bounds the rows: far below 2^31
    const int32_t lo_pos = off_at(0);
    // Row-tiles innermost: the passes over one column group's weights follow one another.
    // Workgroups go round the XCDs, and so do consecutive units: few of them still use every
    // XCD's path to memory.
    for (int w = blockIdx.x; w < total; w += gridDim.x) {
        int lo = 0, hi = a.nslots;                 // position of the slot: mt_start[lo] ngroups <= w
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (mt_at(mid) * ngroups <= w) lo = mid; else hi = mid;
        }
        const int tiles = mt_at(lo + 1) - mt_at(lo), rem = w - mt_at(lo) * ngroups;
        Unit u;
        u.slot = __builtin_amdgcn_readfirstlane(small ? tt.order[lo] : a.order[lo]);
        u.group = __builtin_amdgcn_readfirstlane(rem / tiles);
        u.row = __builtin_amdgcn_readfirstlane(off_at(u.slot) - lo_pos);
        u.m0 = __builtin_amdgcn_readfirstlane(rem % tiles * kStreamRows);
        u.rows = min(kStreamRows, __builtin_amdgcn_readfirstlane(off_at(u.slot + 1) - lo_pos) - u.row - u.m0);
        u.w[0] = uniform_base(small ? tt.w[0][u.slot] : w0[u.slot]);
        u.w[1] = uniform_base(small ? tt.w[1][u.slot] : w1[u.slot]);
        if (u.rows <= 16) stream_unit<GATEUP, SRC, 1>(a, u, K, N, wave, part);
        else if (u.rows <= 32) stream_unit<GATEUP, SRC, 2>(a, u, K, N, wave, part);
        else stream_unit<GATEUP, SRC, kMaxNXF>(a, u, K, N, wave, part);
    }
}

template <bool GATEUP>
hipError_t launch_stream(const FfnArgs &a, bool packed, hipStream_t s) {
    if (a.nslots <= 0 || a.max_rows <= 0) return hipSuccess;
    const int N = GATEUP ? a.I : a.H, gc = GATEUP ? 16 : 32;
    const int64_t ngroups = (N + gc - 1) / gc;
    const int64_t bound = (a.max_rows / kStreamRows + a.nslots) * ngroups;      // most units any batch can have
    int64_t grid = std::min<int64_t>(bound, (int64_t)a.num_cu * 2);
    const dim3 g((unsigned)grid), b(kThreads);
    if (!packed) hipLaunchKernelGGL((ffn_stream_kernel<GATEUP, kRowMajor>), g, b, 0, s, a);
    else if (a.w8) hipLaunchKernelGGL((ffn_stream_kernel<GATEUP, kPackedE4M3>), g, b, 0, s, a);
    else hipLaunchKernelGGL((ffn_stream_kernel<GATEUP, kPackedBf16>), g, b, 0, s, a);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_gateup_stream(const FfnArgs &a, bool packed, hipStream_t s) { return launch_stream<true>(a, packed, s); }
hipError_t launch_down_stream(const FfnArgs &a, bool packed, hipStream_t s) { return launch_stream<false>(a, packed, s); }

}  // namespace craft
