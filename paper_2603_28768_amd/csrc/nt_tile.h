// The contraction of one tile of a matrix product C = A B^T whose operands are both stored row by
// row along the contraction (bf16): up to 256 rows of A against up to 128 rows of B per workgroup
// of four waves, 2 x 2 of them, on v_mfma_f32_16x16x32_bf16.
//
// Both operands travel from global memory straight into LDS (dma_chunk) in 64-wide slabs of 128
// bytes per row, unpadded, the eight 16-byte pieces of row r in the order piece ^ (r & 7) so that the
// fragment reads (16 rows at one contraction offset) hit every bank once.  Three stages, four where
// they fit, five or six of the small tiles': while one slab is multiplied the next is on its way or landed and the ones after it are
// requested, up to 96 KiB in flight per CU.  The fragments of the next 32-wide step are read while the present
// one is multiplied, across the slab's barrier too: the barrier stands in front of a slab's second
// step, by when every wave has read all of the slab (its reads are complete at the barrier) and the
// slab after it has landed.
#pragma once

#include <type_traits>

#include "ffn_common.h"

namespace craft {

constexpr int kNtThreads = 256;
// FA, FB: 16-row fragments of A and B per wave
template <int FA, int FB> constexpr int nt_stage_bytes() { return (FA + FB) * 32 * 128; }
constexpr int kNtLds = 3 * 12 * 32 * 128;          // three stages of 256 + 128 rows
constexpr int nt_stages_of(int bytes) { return bytes <= 12 << 10 ? 6 : bytes <= 16 << 10 ? 5 : bytes * 4 <= kNtLds ? 4 : 3; }
template <int FA, int FB> constexpr int nt_stages() { return nt_stages_of(nt_stage_bytes<FA, FB>()); }
template <int FA, int FB> constexpr int nt_lds_bytes() { return nt_stages<FA, FB>() * nt_stage_bytes<FA, FB>(); }

// Before an accumulator is read: more idle cycles than a matrix instruction takes to be read, then
// every accumulator passes through a statement ordered behind them.
template <int FA, int FB> static __device__ __forceinline__ void nt_settle(f32x4_t (&acc)[FA][FB]) {
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
#pragma unroll
    for (int f = 0; f < FA; ++f)
#pragma unroll
        for (int g = 0; g < FB; ++g) asm volatile("" : "+a"(acc[f][g]));
}

// Rows of this many elements: 256 of them stay inside a 32-bit byte offset.
constexpr int kNtRowLimit = 1 << 23;
// abase, bbase: wave-uniform; aoff, boff: the byte offset of a row (0 .. 32 FA - 1, 32 FB - 1) from them, B's also
// told which chunk of 32 rows it is in (row 32 chunk + threadIdx.x / 8, always).  K: elements
// per row, a multiple of 8, less than kNtRowLimit.  acc[f][g] += A fragment wa FA + f x B fragment wb FB + g, where wave w of
// the workgroup is (wa, wb) = (w >> 1, w & 1); element v of lane l is row 4 (l >> 4) + v of A's fragment
// and row l & 15 of B's.  kbeg, kend: the slabs to take.  Ends with a barrier and nothing in flight.
// `after_slab` runs behind every slab.
struct NothingAfter { __device__ __forceinline__ void operator()(int) const {} };
template <int FA, int FB, typename AOFF, typename BOFF, typename AFTER = NothingAfter>
static __device__ __forceinline__ void nt_tile(unsigned char *smem, ubase_t abase, const AOFF &aoff_of, ubase_t bbase,
                                               const BOFF &boff_of, int K, int kbeg, int kend, f32x4_t (&acc)[FA][FB],
                                               const AFTER &after_slab = AFTER{}) {
    constexpr int STAGEB = nt_stage_bytes<FA, FB>(), S = nt_stages<FA, FB>();
    const int lane = threadIdx.x & 63, q = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)smem;
    const uint32_t lds_wave = lds0 + (uint32_t)__builtin_amdgcn_readfirstlane(wave * 8 * 128);
    const uint32_t piece = (uint32_t)(((lane & 7) ^ ((lane >> 3) & 7)) * 16);
    const uint32_t fo = (uint32_t)((lane & 15) * 128 + ((q ^ (lane & 7)) & 7) * 16);
    const uint32_t fa0 = fo + (uint32_t)((wave >> 1) * FA * 16 * 128), fb0 = fo + (uint32_t)((FA * 32 + (wave & 1) * FB * 16) * 128);
    if (kbeg >= kend) return;
    uint32_t aoff[FA];
    decltype(boff_of(0, 0)) boff[FB];              // 32 or 64 bits
    const int lr = (int)threadIdx.x >> 3;          // this lane's row of a 32-row chunk
#pragma unroll
    for (int i = 0; i < FA; ++i) aoff[i] = (uint32_t)aoff_of(32 * i + lr);
#pragma unroll
    for (int i = 0; i < FB; ++i) boff[i] = boff_of(i, 32 * i + lr);
    typedef const bf16x8_t __attribute__((address_space(3))) *lds_frag_t;
    constexpr int NR = FA + FB;                    // requests per slab and fragments per step
    // where this lane reads slab ks; pieces past the rows are read from inside them (zeroed below)
    auto at = [&](int ks) __attribute__((always_inline)) {
        const uint32_t k = (uint32_t)ks * 128u + piece, last = (uint32_t)K * 2u - 16u;
        return k < last ? k : last;
    };
    auto dest = [&](int i, int s) __attribute__((always_inline)) {
        return lds_wave + (uint32_t)(s * STAGEB) + (uint32_t)(32 * i * 128);      // B's chunks follow A's
    };
    auto request = [&](int i, uint32_t koff) __attribute__((always_inline)) {
        if (i < FA) dma_request(abase, aoff[i < FA ? i : 0] + koff);
        else if constexpr (sizeof(boff[0]) == 4) dma_request(bbase, boff[i < FA ? 0 : i - FA] + koff);
        else dma_request_at(bbase + (boff[i < FA ? 0 : i - FA] + koff));
    };
    bf16x8_t a[2][FA], b[2][FB];
    // fragment j of a step into register set `set`: B's first, the next multiplications start with those
    auto fetch = [&](int set, int j, uint32_t stage, int step) __attribute__((always_inline)) {
        const uint32_t x = (uint32_t)step * 64u;
        if (j < FB) b[set][j < FB ? j : 0] = *(lds_frag_t)(uintptr_t)((stage + (fb0 ^ x)) + 16 * j * 128);
        else a[set][j < FB ? 0 : j - FB] = *(lds_frag_t)(uintptr_t)((stage + (fa0 ^ x)) + 16 * (j - FB) * 128);
    };
    // One 32-wide step: the fragments of set SET multiplied, the next step's fetched into the other
    // set and half of a slab requested meanwhile, all of it dealt out behind single matrix
    // instructions.  In one piece, reads and requests stop the matrix pipes of all four waves for
    // as long as they take together (scores of 8192 tokens, E = 256, H = 7168: 48 us, dealt out 43).
    auto half = [&](auto SET, auto DMA, uint32_t next, int next_step, uint32_t koff, int s2) __attribute__((always_inline)) {
        constexpr int set = SET.value;
        constexpr int D0 = set ? (NR + 1) / 2 : 0, ND = !DMA.value ? 0 : set ? NR / 2 : (NR + 1) / 2;
        constexpr int M = FA * FB, OPS = NR + 2 * ND;
#pragma unroll
        for (int m = 0; m < M; ++m) {
            mfma16<false>(a[set][m / FB], b[set][m % FB], acc[m / FB][m % FB]);
#pragma unroll
            for (int o = m * OPS / M; o < (m + 1) * OPS / M; ++o) {
                if (o < NR) fetch(set ^ 1, o, next, next_step);
                else if ((o - NR) % 2 == 0) dma_to(dest(D0 + (o - NR) / 2, s2));
                else {
                    // behind the same matrix instruction as its destination: a load may not follow M0 at once
                    if (o > m * OPS / M) asm volatile("s_nop 0");
                    request(D0 + (o - NR) / 2, koff);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // the last slab of ragged rows: zeros past their end, in both operands
    // (s_nop: a matrix instruction may read what a vector instruction wrote two cycles later)
    auto cut = [&](int set, int k) __attribute__((always_inline)) {
        const bool past = k + q * 8 >= K;
#pragma unroll
        for (int g = 0; g < FB; ++g) {
            b[set][g] = past ? bf16x8_t{} : b[set][g];
            asm volatile("s_nop 1" : "+v"(b[set][g]));
        }
#pragma unroll
        for (int f = 0; f < FA; ++f) {
            a[set][f] = past ? bf16x8_t{} : a[set][f];
            asm volatile("s_nop 1" : "+v"(a[set][f]));
        }
    };
    const std::integral_constant<int, 0> set0;
    const std::integral_constant<int, 1> set1;
    const std::true_type with;
    const std::false_type without;
    const int last = K & 63 ? K >> 6 : -1;         // the slab that is cut, if any
    for (int j = 0; j < S - 1 && kbeg + j < kend; ++j) {
        const uint32_t koff = at(kbeg + j);
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            dma_to(dest(i, j));
            asm volatile("s_nop 0");
            request(i, koff);
        }
    }
    if (kbeg + S - 2 < kend) dma_wait<(S - 2) * NR>();
    else dma_wait<0>();
    __syncthreads();
#pragma unroll
    for (int j = 0; j < NR; ++j) fetch(0, j, lds0, 0);
    int s = 0, ks = kbeg;
    // Slab ks + S - 1 goes where slab ks - 1 was: all of its reads were complete at the last
    // barrier.  At this one, slab ks + 1 has landed: its requests are older than those of the
    // slabs behind it, of which the last has been requested by half.
    for (; ks + S - 1 < kend; ++ks) {
        const int s1 = s + 1 < S ? s + 1 : 0, s2 = s > 0 ? s - 1 : S - 1;
        const uint32_t here = lds0 + (uint32_t)(s * STAGEB), there = lds0 + (uint32_t)(s1 * STAGEB), koff = at(ks + S - 1);
        half(set0, with, here, 1, koff, s2);
        dma_wait<(S - 3) * NR + (NR + 1) / 2>();
        __syncthreads();
        half(set1, with, there, 0, koff, s2);
        after_slab(ks);
        s = s1;
    }
    for (; ks < kend; ++ks) {
        const int s1 = s + 1 < S ? s + 1 : 0;
        const uint32_t here = lds0 + (uint32_t)(s * STAGEB), there = lds0 + (uint32_t)(s1 * STAGEB);
        if (ks == last) cut(0, ks * 64);
        half(set0, without, here, 1, 0u, 0);
        dma_wait<0>();
        __syncthreads();
        if (ks == last) cut(1, ks * 64 + 32);
        half(set1, without, there, 0, 0u, 0);      // after the last slab: read and not used
        after_slab(ks);
        s = s1;
    }
    __syncthreads();                               // the stages may be filled again
    nt_settle(acc);
}

// The same product for rows of A that are not 16-byte aligned, which loads into LDS ask for, and, with
// FAR, for rows of any length (64-bit offsets).  Through registers and two stages: a slab is multiplied
// while the next one goes into the other stage and the one after that travels, one barrier per slab.
// 1777 tokens on 17 slots, H = 4096, I = 1536, weights two bytes past alignment: 334 us a forward (one
// slab at a time: 930; aligned: 206).  Not what holds it back: reading the two aligned blocks of a
// piece instead of one that straddles them (352), two slabs on their way (349).
template <int FA, int FB, bool FAR, typename AOFF, typename BOFF>
static __device__ __forceinline__ void nt_tile_unaligned(unsigned char *smem, ubase_t abase, const AOFF &aoff_of, ubase_t bbase,
                                                         const BOFF &boff_of, int K, int kbeg, int kend, f32x4_t (&acc)[FA][FB]) {
    const int lane = threadIdx.x & 63, q = lane >> 4, wave = (int)threadIdx.x >> 6, lr = (int)threadIdx.x >> 3;
    typedef unsigned short u16x8_t __attribute__((ext_vector_type(8)));
    typedef unsigned short u16x8_a2_t __attribute__((ext_vector_type(8), aligned(2)));
    // global, not flat: a wait for LDS would wait for flat loads too
    typedef const u16x8_a2_t __attribute__((address_space(1))) *chunk_t;
    typedef typename std::conditional<FAR, uint64_t, uint32_t>::type off_t;
    constexpr int STAGEB = nt_stage_bytes<FA, FB>();
    const int c = lane & 7, place = lr * 128 + (c ^ (lr & 7)) * 16;
    off_t aoff[FA];
    decltype(boff_of(0, 0)) boff[FB];
#pragma unroll
    for (int i = 0; i < FA; ++i) aoff[i] = (off_t)aoff_of(32 * i + lr);
#pragma unroll
    for (int i = 0; i < FB; ++i) boff[i] = boff_of(i, 32 * i + lr);
    u16x8_t av[FA], bv[FB];
    // (past the rows or the last slab: read from inside the rows, replaced by zeros on the way into
    // LDS or not used; no branch around a request, the waits count them)
    auto load = [&](int ks) __attribute__((always_inline)) {
        const off_t k = min((off_t)ks * 128u + (off_t)c * 16u, (off_t)K * 2u - 16u);
#pragma unroll
        for (int i = 0; i < FA; ++i) av[i] = *(chunk_t)(abase + (aoff[i] + k));
#pragma unroll
        for (int i = 0; i < FB; ++i) bv[i] = *(chunk_t)(bbase + (boff[i] + k));
        __builtin_amdgcn_sched_barrier(0);
    };
    auto store = [&](int u, int ks) __attribute__((always_inline)) {
        unsigned char *stage = smem + u * STAGEB;
        const bool in = (off_t)ks * 128u + (off_t)c * 16u < (off_t)K * 2u;
#pragma unroll
        for (int i = 0; i < FA; ++i) *reinterpret_cast<u16x8_t *>(stage + 32 * i * 128 + place) = in ? av[i] : u16x8_t{};
#pragma unroll
        for (int i = 0; i < FB; ++i) *reinterpret_cast<u16x8_t *>(stage + 32 * (FA + i) * 128 + place) = in ? bv[i] : u16x8_t{};
    };
    // slab ks is in stage u: multiplied, while the one after it goes into the other stage and the one
    // after that is requested
    auto slab = [&](int u, int ks) __attribute__((always_inline)) {
        const unsigned char *stage = smem + u * STAGEB;
        bf16x8_t a[2][FA], b[2][FB];
#pragma unroll
        for (int step = 0; step < 2; ++step) {
            const int at = (lane & 15) * 128 + (((step * 4 + q) ^ (lane & 7)) & 7) * 16;
#pragma unroll
            for (int g = 0; g < FB; ++g) b[step][g] = *reinterpret_cast<const bf16x8_t *>(stage + (FA * 32 + ((wave & 1) * FB + g) * 16) * 128 + at);
#pragma unroll
            for (int f = 0; f < FA; ++f) a[step][f] = *reinterpret_cast<const bf16x8_t *>(stage + ((wave >> 1) * FA + f) * 16 * 128 + at);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int f = 0; f < FA; ++f)
#pragma unroll
            for (int g = 0; g < FB; ++g) acc[f][g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[0][f], b[0][g], acc[f][g], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        store(u ^ 1, ks + 1);
        load(ks + 2);
#pragma unroll
        for (int f = 0; f < FA; ++f)
#pragma unroll
            for (int g = 0; g < FB; ++g) acc[f][g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[1][f], b[1][g], acc[f][g], 0, 0, 0);
        __syncthreads();
    };
    if (kbeg >= kend) return;
    load(kbeg);
    store(0, kbeg);
    load(kbeg + 1);
    __syncthreads();
    for (int ks = kbeg; ks < kend; ks += 2) {
        slab(0, ks);
        if (ks + 1 < kend) slab(1, ks + 1);
    }
}

}  // namespace craft
