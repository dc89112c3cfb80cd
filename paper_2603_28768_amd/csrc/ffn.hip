// Grouped SwiGLU expert FFN of one rank (Sec. 2.1: each expert is an up-projection, a
// non-linearity and a down-projection; here down(silu(gate x) * up x)).
//
// Two grouped GEMMs over the rank's slots, both "NT" (activation rows and weight rows are
// contiguous along the contraction):
//   gate/up : act[r][i] = silu(sum_h x[r][h] Wg[i][h]) * (sum_h x[r][h] Wu[i][h])
//   down    : y[r][h]   = sum_i act[r][i] Wd[h][i]
//
// Work is cut into tiles of (slot, column tile, row tile).  Slots differ wildly in rows
// under skewed routing, so the tile list is data dependent: a prefix table of row tiles per
// slot is left in device memory, a persistent grid takes its first tiles by position and the
// rest from a counter, busiest slots first; a slot with no rows contributes no tile, a slot with
// few rows one (ragged) row tile per column tile.  Row tiles of the same (slot, column tile)
// are adjacent in the list and the workgroup-to-tile mapping keeps neighbours on one XCD, so
// a weight tile is fetched from HBM once and re-read from that XCD's L2.
//
// bf16 path: 256 weight rows against 32, 64 or 128 activation rows (nt_tile.h).  For gate/up
// the weight rows of a tile are 128 gate and the 128 matching up rows, 16 of one followed by 16 of
// the other, so that gate and up of one output meet in the same lane and element of two
// accumulators: SwiGLU is applied in registers.  The gate/up GEMM reads its rows straight from x
// through the dispatch permutation (no staged copy).  A slab of a tall tile, 48 KiB, takes 0.87 us in a
// launch of one slot and one round (2304 rows, I = 1536: gate/up 105.3 us at H = 7168, 23.2 at 1024), twice its
// matrix instructions; which of the latency of loads that miss the L2 and the issue of reads and requests holds
// it there has not been taken apart (a CU reads three times as fast out of its L2 in a plain loop).  Taller tiles move less but come out in fewer rounds.  1777 tokens on 17 slots,
// H = 4096, I = 1536: gate/up 190 -> 117 us, down 84 -> 63 (before: 128 x 128 tiles through registers, one
// slab ahead).  A cold slot's tile is bound by what one CU gets out of HBM, about 42 GB/s whatever it has in
// flight: 256 weight rows of 4096 elements take it 50 us.  Where a launch would end with them the cold
// slots therefore get 64 weight rows a tile (below); a forward of those 1777 tokens 195 -> 178 us, 1100 tokens 183 -> 158,
// of 4767 on slots of H = 5120, I = 2048 430 -> 406; without a cold slot the same within 2 %.  With 128 rows a tile 183.
//
// fp32 path: units of 16 columns and 32 rows from the same tile list (small configurations).
#include <type_traits>

#include "nt_tile.h"

namespace craft {
namespace {

// ------------------------------------------------------------------ bf16 / MFMA
// Row of the A operand of a tile -> weight row, relative to the tile's first output column.  For
// gate/up, 16 gate rows are followed by the 16 up rows of the same columns.
template <bool GATEUP> static __device__ __forceinline__ int weight_row(int r) {
    return GATEUP ? (r >> 5) * 16 + (r & 15) : r;
}

// 32 FA weight rows: FA = 8, or 2 for a tile of a quarter of the width
template <bool GATEUP, int FA, int FB, bool FAR>
__device__ __forceinline__ int32_t bf16_tile(const FfnArgs &a, const Tile &t, unsigned char *smem, int K, int N, int32_t lo_pos,
                                             int32_t *counter) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    // The activation rows of a full tile are all looked up before one of them is needed.  Left to where it is
    // needed, the compiler asks for each when the last one has come, as its registers run: four round
    // trips in front of every tile (4473 rows of H = 1024, I = 1536, gate/up 46.0 us, so 42.9).  The narrow tiles
    // are as fast either way (the forward of 1777 tokens 189.8 and 191.7) and keep their registers.
    constexpr bool AHEAD = GATEUP && FA == 8;
    auto row_at = [&](int r) { return min(r, t.rows - 1); };
    int32_t pair[FB];
    if (AHEAD)
#pragma unroll
        for (int i = 0; i < FB; ++i) pair[i] = a.src[t.pos0 + t.m0 + row_at(32 * i + ((int)threadIdx.x >> 3))];
    // chunks of 32 rows of A: the first two waves fetch gate rows, the others up rows
    const void *w = GATEUP ? (wave < 2 ? a.w_gate[t.slot] : a.w_up[t.slot]) : a.w_down[t.slot];
    const ubase_t wbase = uniform_base(static_cast<ubase_t>(w) + (int64_t)t.n0 * K * 2);
    auto woff = [&](int r) { return (uint64_t)min(weight_row<GATEUP>(r), N - 1 - t.n0) * (uint64_t)K * 2u; };
    const ubase_t xbase = uniform_base(GATEUP ? static_cast<ubase_t>(a.x)
                                              : static_cast<ubase_t>(a.act) + (int64_t)(t.pos0 + t.m0 - lo_pos) * K * 2);
    typedef typename std::conditional<FAR, uint64_t, uint32_t>::type off_t;
    auto xoff_far = [&](int i, int r) {
        return (uint64_t)(GATEUP ? (AHEAD ? pair[i] : a.src[t.pos0 + t.m0 + row_at(r)]) / a.k : row_at(r)) * (uint64_t)K * 2u;
    };
    auto xoff = [&](int i, int r) { return (off_t)xoff_far(i, r); };
    f32x4_t acc[FA][FB];
#pragma unroll
    for (int f = 0; f < FA; ++f)
#pragma unroll
        for (int g = 0; g < FB; ++g) acc[f][g] = (f32x4_t)(0.0f);
    // (the other wave's matrix counts too: all waves have to take the same path)
    const uintptr_t bits = reinterpret_cast<uintptr_t>(GATEUP ? a.w_gate[t.slot] : a.w_down[t.slot]) |
                           reinterpret_cast<uintptr_t>(GATEUP ? a.w_up[t.slot] : a.w_down[t.slot]);
    const int nk = (K + 63) / 64;
    if (K >= kNtRowLimit) nt_tile_unaligned<FA, FB, true>(smem, wbase, woff, xbase, xoff_far, K, 0, nk, acc);
    else if ((__builtin_amdgcn_readfirstlane((int)bits) & 15) == 0) nt_tile<FA, FB>(smem, wbase, woff, xbase, xoff, K, 0, nk, acc);
    else nt_tile_unaligned<FA, FB, false>(smem, wbase, woff, xbase, xoff, K, 0, nk, acc);
    // the next tile is claimed here, its number arrives while the results are stored
    // (an increment: an add of a uniform value becomes a wave-wide reduction)
    int32_t claimed = 0;
    if (threadIdx.x == 0) claimed = (int32_t)atomicInc(reinterpret_cast<unsigned int *>(counter), 0xffffffffu);
    unsigned short *outp = static_cast<unsigned short *>(GATEUP ? a.act : a.y);
#pragma unroll
    for (int g = 0; g < FB; ++g) {
        const int m = ((wave & 1) * FB + g) * 16 + (lane & 15);
        unsigned short *orow = outp + (int64_t)(t.pos0 + t.m0 + m - lo_pos) * N;
#pragma unroll
        for (int f = 0; f < FA; f += GATEUP ? 2 : 1) {
            const int col = t.n0 + weight_row<GATEUP>(((wave >> 1) * FA + f) * 16) + (lane >> 4) * 4;
            if (m >= t.rows || col >= N) continue;
            float v[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) v[c] = GATEUP ? silu(acc[f][g][c]) * acc[f + (GATEUP ? 1 : 0)][g][c] : acc[f][g][c];
            *reinterpret_cast<uint2 *>(orow + col) = make_uint2(bf16_pair(v[0], v[1]), bf16_pair(v[2], v[3]));
        }
    }
    return claimed;
}

// The tile list: the busy slots' tiles, then those of the cold slots, one row-tile each, at a quarter of
// the width, so that the launch does not end with a tile that streams 256 weight rows through one CU.  All
// stay at full width where every tile is in a single round, and where quarters are no gain: where the cold
// tiles find room beside the last round of the busy ones (276 + 120 tiles of K = 4096 on 256 CUs: a quarter as
// wide +8.8 us of a forward of 224), and where they are many and short, so that a small tile's fixed part
// counts (640 + 592 of K = 512: +8.8 us of 230): narrow_cold_tiles.  264 launches of 300 drawn batches: quarters everywhere cost
// more than 1 % of the forward in 40 of them, by this rule in 4 (the worst 228 + 36 of K = 1408, 4 %), which
// keeps 96 % of what they save.
template <bool GATEUP, bool FAR>
__global__ __launch_bounds__(kNtThreads, 1) void ffn_bf16_kernel(FfnArgs a) {
    __shared__ __attribute__((aligned(16))) unsigned char ffn_smem[kNtLds];
    __shared__ TileTables tt;
    __shared__ int64_t next_item;
    const int32_t *mt_start = a.mt_start + (GATEUP ? 0 : a.nslots + 1);
    const bool small = a.nslots <= TileTables::kMaxSlots;
    if (small) load_tile_tables(a, mt_start, tt);
    const int32_t lo_pos = first_row(a, tt, small);
    const int K = GATEUP ? a.H : a.I;              // contraction length
    const int N = GATEUP ? a.I : a.H;              // output columns
    constexpr int BN = GATEUP ? 128 : 256;         // output columns per tile
    const int nt = (N + BN - 1) / BN;
    int64_t wide = (int64_t)tiles_before(mt_start, tt, small, a.nslots) * nt, total = wide;
    if (wide > (int64_t)gridDim.x) {
        const int32_t hot = ctrl_word(a, tt, small, CTRL_HOT_SLOTS);
        const int64_t busy = (int64_t)tiles_before(mt_start, tt, small, hot) * nt, cold = wide - busy;
        if (narrow_cold_tiles(busy, cold, gridDim.x, K)) {
            wide = busy;
            total = busy + 4 * cold;
        }
    }
    int32_t *const counter = a.ctrl + (GATEUP ? CTRL_WORK_GATEUP : CTRL_WORK_DOWN);
    auto next = [&](int32_t claimed) {
        if (threadIdx.x == 0) next_item = (int64_t)gridDim.x + claimed;
        __syncthreads();
        return next_item;                          // (written again only after the next tile's barriers)
    };
    int64_t w = first_tile(total);                 // first tile by position, the rest on demand
    const int32_t fmax = GATEUP ? a.frags_gu : a.frags_dn;
    while (w < wide) {
        Tile t = small ? decode_tile(a, tt, w, nt, BN, fmax) : decode_tile(a, mt_start, w, nt, BN, fmax);
        t.slot = __builtin_amdgcn_readfirstlane(t.slot);
        t.n0 = __builtin_amdgcn_readfirstlane(t.n0);
        t.rows = __builtin_amdgcn_readfirstlane(t.rows);
        int32_t claimed;
        if (t.rows <= 32) claimed = bf16_tile<GATEUP, 8, 1, FAR>(a, t, ffn_smem, K, N, lo_pos, counter);
        else if (t.rows <= 64) claimed = bf16_tile<GATEUP, 8, 2, FAR>(a, t, ffn_smem, K, N, lo_pos, counter);
        else claimed = bf16_tile<GATEUP, 8, 4, FAR>(a, t, ffn_smem, K, N, lo_pos, counter);
        w = next(claimed);
    }
    while (__builtin_expect(w < total, 0)) {       // (out of the way of the others' code, which is fetched first)
        const int64_t u = w - wide;
        const int32_t pos = ctrl_word(a, tt, small, CTRL_HOT_SLOTS) + (int32_t)(u / (4 * nt));
        Tile t;
        t.slot = __builtin_amdgcn_readfirstlane(small ? tt.order[pos] : a.order[pos]);
        t.pos0 = small ? tt.slot_off[t.slot] : a.slot_off[a.s_lo + t.slot];
        t.rows = __builtin_amdgcn_readfirstlane((small ? tt.slot_off[t.slot + 1] : a.slot_off[a.s_lo + t.slot + 1]) - t.pos0);
        t.m0 = 0;
        t.n0 = __builtin_amdgcn_readfirstlane((int32_t)(u % (4 * nt)) * (BN / 4));
        int32_t claimed = 0;
        if (t.n0 < N) {
            if (t.rows <= 32) claimed = bf16_tile<GATEUP, 2, 1, FAR>(a, t, ffn_smem, K, N, lo_pos, counter);
            else claimed = bf16_tile<GATEUP, 2, 2, FAR>(a, t, ffn_smem, K, N, lo_pos, counter);
        } else {                                   // the last quarters may lie past the matrix
            if (threadIdx.x == 0) claimed = (int32_t)atomicInc(reinterpret_cast<unsigned int *>(counter), 0xffffffffu);
            __syncthreads();                       // next_item has been read by all
        }
        w = next(claimed);
    }
}

// ------------------------------------------------------------------------ fp32
// A unit is 16 output columns (16 weight rows, for gate/up 16 of each) against up to 32 activation
// rows; the four waves take every fourth 16-wide piece of the contraction and add their sums up
// in LDS, in wave order.  Both operands go straight from memory into the operand registers of
// v_mfma_f32_16x16x4_f32, 16 bytes per lane: lane l holds row l & 15, elements 4 (l >> 4) .. + 3 of a
// piece, and the four matrix instructions of a piece take one of them each.  These layers are small
// and a launch is a chain of round trips: looking up the unit, its rows, one or two rounds of
// operands.  256 tokens, H = 128, I = 256: gate/up 13.9 -> 7.3 us, down 17.0 -> 6.0 (before: 32 x 32
// tiles of plain multiply-adds, staged through LDS by one wave's worth of requests at a time).
constexpr int FN = 16;            // output columns per unit
constexpr int FK = 16;            // contraction elements per piece
constexpr int kF32Waves = 4;
typedef float f32x4_a4_t __attribute__((ext_vector_type(4), aligned(4)));

// rows: 16-row fragments of activations, 1 or 2
template <bool GATEUP, int NXF>
__device__ __forceinline__ void f32_unit(const FfnArgs &a, const Tile &t, int K, int N, int32_t lo_pos, f32x4_t *part) {
    constexpr int NW = GATEUP ? 2 : 1, PW = 4;     // weight fragments; pieces in flight per wave
    const int lane = threadIdx.x & 63, q = lane >> 4, r16 = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const float *w[NW], *x[NXF];
    const float *wbase[2] = {static_cast<const float *>(GATEUP ? a.w_gate[t.slot] : a.w_down[t.slot]),
                             GATEUP ? static_cast<const float *>(a.w_up[t.slot]) : nullptr};
    // 16 bytes at a time from weights that are aligned to that (rows are whole multiples of it)
    const bool whole = ((reinterpret_cast<uintptr_t>(wbase[0]) | reinterpret_cast<uintptr_t>(wbase[1])) & 15) == 0;
#pragma unroll
    for (int h = 0; h < NW; ++h) w[h] = wbase[h] + (int64_t)min(t.n0 + r16, N - 1) * K;
#pragma unroll
    for (int g = 0; g < NXF; ++g) {
        const int32_t pos = t.pos0 + t.m0 + min(16 * g + r16, t.rows - 1);
        x[g] = GATEUP ? static_cast<const float *>(a.x) + (int64_t)(a.src[pos] / a.k) * K
                      : static_cast<const float *>(a.act) + (int64_t)(pos - lo_pos) * K;
    }
    f32x4_t acc[NW][NXF];
#pragma unroll
    for (int h = 0; h < NW; ++h)
#pragma unroll
        for (int g = 0; g < NXF; ++g) acc[h][g] = (f32x4_t)(0.0f);
    const int pieces = (K + FK - 1) / FK;
    for (int c0 = wave; c0 < pieces; c0 += PW * kF32Waves) {
        f32x4_t wv[PW][NW], xv[PW][NXF];
        // past the end: read from inside the row, replaced by zeros below
        if (whole) {
#pragma unroll
            for (int u = 0; u < PW; ++u)
#pragma unroll
                for (int h = 0; h < NW; ++h)
                    wv[u][h] = *reinterpret_cast<const f32x4_t *>(w[h] + min((c0 + u * kF32Waves) * FK + 4 * q, K - 4));
        } else {
#pragma unroll
            for (int u = 0; u < PW; ++u)
#pragma unroll
                for (int h = 0; h < NW; ++h)
                    wv[u][h] = *reinterpret_cast<const f32x4_a4_t *>(w[h] + min((c0 + u * kF32Waves) * FK + 4 * q, K - 4));
        }
#pragma unroll
        for (int u = 0; u < PW; ++u)
#pragma unroll
            for (int g = 0; g < NXF; ++g)
                xv[u][g] = *reinterpret_cast<const f32x4_t *>(x[g] + min((c0 + u * kF32Waves) * FK + 4 * q, K - 4));
#pragma unroll
        for (int u = 0; u < PW; ++u) {
            const bool in = (c0 + u * kF32Waves) * FK + 4 * q < K;
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int h = 0; h < NW; ++h)
#pragma unroll
                    for (int g = 0; g < NXF; ++g)
                        acc[h][g] = __builtin_amdgcn_mfma_f32_16x16x4f32(in ? wv[u][h][e] : 0.0f, in ? xv[u][g][e] : 0.0f,
                                                                         acc[h][g], 0, 0, 0);
        }
    }
    __syncthreads();                               // the last unit's sums have been read
#pragma unroll
    for (int h = 0; h < NW; ++h)
#pragma unroll
        for (int g = 0; g < NXF; ++g) part[((wave * NW + h) * NXF + g) * 64 + lane] = acc[h][g];
    __syncthreads();
    // element v of lane l is weight row 4 (l >> 4) + v and row l & 15 of its fragment
    if (wave < NXF) {
        f32x4_t s[NW];
#pragma unroll
        for (int h = 0; h < NW; ++h) {
            s[h] = part[(h * NXF + wave) * 64 + lane];
#pragma unroll
            for (int v = 1; v < kF32Waves; ++v) s[h] += part[((v * NW + h) * NXF + wave) * 64 + lane];
        }
        if (GATEUP)
#pragma unroll
            for (int c = 0; c < 4; ++c) s[0][c] = (s[0][c] / (1.0f + expf(-s[0][c]))) * s[NW - 1][c];
        const int m = 16 * wave + r16, col = t.n0 + 4 * q;
        if (m < t.rows && col < N)                 // N is a multiple of 4
            *reinterpret_cast<f32x4_t *>(static_cast<float *>(GATEUP ? a.act : a.y) +
                                         (int64_t)(t.pos0 + t.m0 + m - lo_pos) * N + col) = s[0];
    }
}

template <bool GATEUP>
__global__ __launch_bounds__(64 * kF32Waves) void ffn_f32_kernel(FfnArgs a) {
    __shared__ f32x4_t part[kF32Waves * 2 * 2 * 64];
    __shared__ TileTables tt;
    const int K = GATEUP ? a.H : a.I;
    const int N = GATEUP ? a.I : a.H;
    const int nt = (N + FN - 1) / FN;
    const int32_t *mt_start = a.mt_start + (GATEUP ? 0 : a.nslots + 1);
    const int32_t fmax = GATEUP ? a.frags_gu : a.frags_dn;
    const bool small = a.nslots <= TileTables::kMaxSlots;
    if (small) load_tile_tables(a, mt_start, tt);
    const int64_t total = (int64_t)tiles_before(mt_start, tt, small, a.nslots) * nt;
    const int32_t lo_pos = first_row(a, tt, small);
    for (int64_t w = blockIdx.x; w < total; w += gridDim.x) {
        const Tile t = small ? decode_tile(a, tt, w, nt, FN, fmax) : decode_tile(a, mt_start, w, nt, FN, fmax);
        if (t.rows <= 16) f32_unit<GATEUP, 1>(a, t, K, N, lo_pos, part);
        else f32_unit<GATEUP, 2>(a, t, K, N, lo_pos, part);
    }
}

template <bool GATEUP>
hipError_t launch_ffn(const FfnArgs &a, hipStream_t s) {
    if (a.nslots <= 0 || a.max_rows <= 0) return hipSuccess;
    const int N = GATEUP ? a.I : a.H;
    if (a.dtype == CRAFT_BF16) {
        const int bn = GATEUP ? 128 : 256;
        const int64_t nt = (N + bn - 1) / bn;
        // most tiles of full width that any batch can have: cold slots get narrow ones only in a launch of more than
        // a round of wide tiles, whose grid is every CU
        const int64_t bound = (a.max_rows / (kFragsBf16 * 32) + a.nslots) * nt;
        int64_t grid = std::min<int64_t>(bound, (int64_t)a.num_cu);
        grid = std::max<int64_t>(8, (grid + 7) / 8 * 8);
        // token rows are fetched at 32-bit offsets where x allows it
        if constexpr (GATEUP)
            if (a.far_x) {
                hipLaunchKernelGGL((ffn_bf16_kernel<GATEUP, true>), dim3((unsigned)grid), dim3(kNtThreads), 0, s, a);
                return hipGetLastError();
            }
        hipLaunchKernelGGL((ffn_bf16_kernel<GATEUP, false>), dim3((unsigned)grid), dim3(kNtThreads), 0, s, a);
    } else {
        const int64_t nt = (N + FN - 1) / FN;
        const int64_t bound = (a.max_rows / (kFragsF32 * 32) + a.nslots) * nt;
        const int64_t grid = std::min<int64_t>(bound, (int64_t)a.num_cu * 4);
        hipLaunchKernelGGL(ffn_f32_kernel<GATEUP>, dim3((unsigned)grid), dim3(64 * kF32Waves), 0, s, a);
    }
    return hipGetLastError();
}

}  // namespace

hipError_t launch_gateup(const FfnArgs &a, hipStream_t s) { return launch_ffn<true>(a, s); }
hipError_t launch_down(const FfnArgs &a, hipStream_t s) { return launch_ffn<false>(a, s); }

}  // namespace craft
