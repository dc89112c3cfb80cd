// Pieces shared by the grouped-GEMM kernels: the tile list walk and small device helpers.
#pragma once

#include <algorithm>

#include "kernels.h"

namespace craft {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

struct Tile {
    int32_t slot;      // local slot index
    int32_t m0;        // first row inside the slot
    int32_t rows;      // valid rows in this tile
    int32_t n0;        // first output column
    int32_t pos0;      // global dispatch position of the slot's first row
    int32_t mtile;     // index of the row-tile in the list of all row-tiles of the busy slots
    int32_t single;    // 1 when this is the slot's only row-tile (nobody else reads its weights)
};

// Flattened work item w -> tile.  nt = column tiles per slot, bn = columns per tile.
// mt_start[p] = row-tiles before position p of the busiest-first slot order.  A slot's rows
// are cut into F 32-row fragments and m row-tiles (row_tiles), either f fragments each with
// a remainder at the end, or shared as evenly as whole fragments allow (row-tile i takes
// fragments floor(i F / m) .. floor((i+1) F / m)); the launch says which.
//
// Inside a slot the m x nt tiles are listed column by column, or (`blocked`) block by block:
// bands of kBandRows row-tiles, a band cut into blocks of kBlockCols column tiles, a block
// column by column.  A run of consecutive list entries, which is what runs at one time (tiles
// are handed out in list order), is then a compact rectangle of tiles that needs few row-tiles
// of activations and few column tiles of weights between them, where a run of the column
// order needs every row-tile of the slot for each of its columns.  At T = 32768 (five rounds of
// tiles) the step is 4 % faster with 8 x 8 blocks than column by column (4 x 8, 8 x 4: 3 %;
// 2 x 16, 16 x 16, 1 x 8: 2 %); the packed kernels use the block order for launches of more
// than two rounds.
constexpr int kBandRows = 8;
constexpr int kBlockCols = 8;
struct TileTables {
    static constexpr int kMaxSlots = 256;
    int32_t mt_start[kMaxSlots + 1];
    int32_t order[kMaxSlots];
    int32_t slot_off[kMaxSlots + 1];      // offsets of the rank's slots, busiest-first order undone
    int32_t ctrl[CTRL_WORDS];             // the control words (the counters among them as the launch finds them)
};
static __device__ __forceinline__ void load_tile_tables(const FfnArgs &a, const int32_t *mt_start,
                                                        TileTables &tt) {
    // no branch around a load: everything travels in one round trip
    const int32_t word = a.ctrl[min((int)threadIdx.x, CTRL_WORDS - 1)];
    for (int i = threadIdx.x; i <= a.nslots; i += blockDim.x) {
        const int last = min(i, a.nslots - 1);
        const int32_t start = mt_start[i], off = a.slot_off[a.s_lo + i], slot = a.order[last];
        tt.mt_start[i] = start;
        tt.slot_off[i] = off;
        tt.order[last] = slot;
    }
    if (threadIdx.x < CTRL_WORDS) tt.ctrl[threadIdx.x] = word;
    __syncthreads();
}
// A control word, an entry of the first table and the rank's first row, from the copy where there is one.
static __device__ __forceinline__ int32_t ctrl_word(const FfnArgs &a, const TileTables &tt, bool small, int i) {
    return __builtin_amdgcn_readfirstlane(small ? tt.ctrl[i] : a.ctrl[i]);
}
static __device__ __forceinline__ int32_t tiles_before(const int32_t *mt_start, const TileTables &tt, bool small, int32_t p) {
    return __builtin_amdgcn_readfirstlane(small ? tt.mt_start[p] : mt_start[p]);
}
static __device__ __forceinline__ int32_t first_row(const FfnArgs &a, const TileTables &tt, bool small) {
    return __builtin_amdgcn_readfirstlane(small ? tt.slot_off[0] : a.slot_off[a.s_lo]);
}
// MT, ORD, OFF: the three tables, in global memory or in a workgroup's LDS copy
// fmax > 0: row-tiles of fmax fragments and a remainder; fmax < 0: shared evenly
template <typename MT, typename ORD, typename OFF>
static __device__ __forceinline__ Tile decode_tile_in(int32_t nslots, const MT &mt_start, const ORD &order,
                                                      const OFF &slot_off, int64_t w, int32_t nt, int32_t bn,
                                                      int32_t fmax, bool blocked) {
    const int32_t qn = (int32_t)(w / nt);
    int32_t lo = 0, hi = nslots;                   // find p: mt_start[p] <= qn < mt_start[p+1]
    while (hi - lo > 1) {
        const int32_t mid = (lo + hi) >> 1;
        if (mt_start[mid] <= qn) lo = mid; else hi = mid;
    }
    const int32_t mt_first = mt_start[lo];
    const int32_t mts = mt_start[lo + 1] - mt_first;
    const int32_t s = order[lo];
    const int32_t rem = (int32_t)(w - (int64_t)mt_first * nt);
    const int32_t band = blocked ? kBandRows : mts;             // column by column: one band, one column per block
    const int32_t bcols = blocked ? kBlockCols : 1;
    const int32_t r0 = rem / (band * nt) * band;                // first row-tile of the band
    const int32_t rj = min(band, mts - r0);                     // row-tiles in this band
    const int32_t in_band = rem - r0 * nt;
    const int32_t cb = in_band / (rj * bcols);                  // block of columns inside the band
    const int32_t in_block = in_band - cb * rj * bcols;
    const int32_t i = r0 + in_block % rj;
    const int32_t col = cb * bcols + in_block / rj;
    Tile t;
    t.slot = s;
    t.pos0 = slot_off[s];
    const int32_t slot_rows = slot_off[s + 1] - t.pos0;
    const int32_t frags = (slot_rows + 31) >> 5;
    const int32_t f0 = fmax > 0 ? i * fmax : (int32_t)((int64_t)i * frags / mts);
    const int32_t f1 = fmax > 0 ? min(f0 + fmax, frags) : (int32_t)((int64_t)(i + 1) * frags / mts);
    t.m0 = f0 * 32;
    t.rows = min(f1 * 32, slot_rows) - t.m0;
    t.n0 = col * bn;
    t.mtile = mt_first + i;
    t.single = mts == 1 ? 1 : 0;
    return t;
}
static __device__ __forceinline__ Tile decode_tile(const FfnArgs &a, const int32_t *mt_start, int64_t w,
                                                   int32_t nt, int32_t bn, int32_t fmax, bool blocked = false) {
    return decode_tile_in(a.nslots, mt_start, a.order, a.slot_off + a.s_lo, w, nt, bn, fmax, blocked);
}
static __device__ __forceinline__ Tile decode_tile(const FfnArgs &a, const TileTables &tt, int64_t w,
                                                   int32_t nt, int32_t bn, int32_t fmax, bool blocked = false) {
    return decode_tile_in(a.nslots, tt.mt_start, tt.order, tt.slot_off, w, nt, bn, fmax, blocked);
}

// Workgroups are dealt to the 8 XCDs round-robin; give each XCD a contiguous run of the first
// gridDim.x tiles, so that tiles sharing weights meet in one L2.  A list shorter than the grid is
// shared evenly: runs of gridDim.x / 8 would leave whole XCDs, and their paths to memory, without
// a tile (two live slots of H = 7168, I = 2048 with 32 column tiles each ran on two of the eight).
// Returns `total` or more where there is nothing to do.  The grid is a multiple of 8.
static __device__ __forceinline__ int64_t first_tile(int64_t total) {
    const int64_t g = gridDim.x, b = blockIdx.x;
    const int64_t run = total < g ? (total + 7) / 8 : g / 8;
    return b / 8 < run ? (b % 8) * run + b / 8 : total;
}

static __device__ __forceinline__ float silu(float g) { return g / (1.0f + __expf(-g)); }
// The same with the hardware reciprocal (1 ulp) instead of a correctly rounded division: the
// result is rounded to bf16 right after.
static __device__ __forceinline__ float silu_fast(float g) {
    return g * __builtin_amdgcn_rcpf(1.0f + __expf(-g));
}
// Two fp32 values to a pair of bf16 (round to nearest even) in one 32-bit word, low half first:
// a single v_cvt_pk_bf16_f32 on gfx950.
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
static __device__ __forceinline__ uint32_t bf16_pair(float lo, float hi) {
    const f32x2_t v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}

// A packed stream holds a multiple of kPackGroups column groups (whole full-width tiles).
constexpr int kPackGroups = 8;
typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));
// A weight fragment as it sits in registers: 8 bf16 values, or 8 E4M3 codes that are widened (exactly): by the
// streaming kernel in front of the MFMA that uses them, by the packed tiles once per step, behind other MFMAs.
template <bool W8> struct WFrag { typedef bf16x8_t type; };
template <> struct WFrag<true> { typedef u32x2_t type; };

static __device__ __forceinline__ bf16x8_t widen(bf16x8_t w) { return w; }
// Two neighbouring codes (the lower or upper half of a word) to a pair of bf16: one instruction,
// exact for every code (the scale is 1).  Through fp32 it takes two.
template <bool UPPER> static __device__ __forceinline__ uint32_t widen_pair(uint32_t codes) {
    return __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(codes, 1.0f, UPPER));
}
typedef unsigned int wide_t __attribute__((ext_vector_type(4)));       // eight bf16 values, a pair per word
static __device__ __forceinline__ bf16x8_t widen(u32x2_t w) {
    const wide_t r = {widen_pair<false>(w[0]), widen_pair<true>(w[0]), widen_pair<false>(w[1]), widen_pair<true>(w[1])};
    return __builtin_bit_cast(bf16x8_t, r);
}

// Every global load of the contraction loop is addressed as a wave-uniform 64-bit base (scalar
// registers, advanced with scalar adds) plus a 32-bit byte offset per lane: no 64-bit vector
// arithmetic per request, and half the address registers to hand to the memory pipeline.
typedef const unsigned char *ubase_t;
static __device__ __forceinline__ ubase_t uniform_base(const void *p) {
    const uint64_t v = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return reinterpret_cast<ubase_t>(((uint64_t)hi << 32) | lo);
}
// A weight fragment that no other tile of the launch reads (a cold slot's: it has one
// row-tile): a streaming load, which leaves the L2 to the weights and rows that are shared.
template <bool ONCE, typename F>
static __device__ __forceinline__ F wload(ubase_t base, uint32_t &off) {
    // the lane's offset never changes inside a tile; widened to 64 bits once outside the loop it
    // would no longer be recognised as the 32-bit offset of a scalar-base request
    // (redefined in place, so that no copy is made)
    asm volatile("" : "+v"(off));
    const F __attribute__((address_space(1))) *p = (const F __attribute__((address_space(1))) *)(base + off);
    if (ONCE) return __builtin_nontemporal_load(p);
    return *p;
}

// 16 bytes per lane from base + off straight into LDS at lds + 16 * lane (lds: the byte address
// of the wave's 1 KiB destination, wave-uniform; it goes through M0, which the compiler keeps
// nothing in across statements).  The compiler does not know that this is a load: it neither
// counts it among the outstanding requests (its own waits for other loads then only wait longer
// than needed, requests complete in order) nor waits for it before LDS reads (dma_wait does).
static __device__ __forceinline__ void dma_chunk(ubase_t base, uint32_t off, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :: "s"(lds), "v"(off), "s"(base) : "memory");
}
// dma_chunk in two statements, with at least one instruction between them
static __device__ __forceinline__ void dma_to(uint32_t lds) { asm volatile("s_mov_b32 m0, %0" :: "s"(lds) : "memory"); }
static __device__ __forceinline__ void dma_request(ubase_t base, uint32_t off) {
    asm volatile("global_load_lds_dwordx4 %0, %1" :: "v"(off), "s"(base) : "memory");
}
// the same from an address of the lane's own
static __device__ __forceinline__ void dma_request_at(ubase_t p) {
    asm volatile("global_load_lds_dwordx4 %0, off" :: "v"(p) : "memory");
}
// wait until at most N of this wave's requests are outstanding
template <int N> static __device__ __forceinline__ void dma_wait() {
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory");
}

// acc += w x^T for a 16-row weight fragment and a 16-row activation fragment over 32
// contraction elements.  Written out as an instruction whose accumulator operand is both read
// and written (an accumulation register tuple, "+a"): a tall tile's 64 accumulators fill the
// accumulation half of the register file exactly, and every copy the register allocator makes
// when result and addend are two values costs moves through the other half.  The compiler does
// not know that this is a matrix instruction: the waits it would insert between a matrix
// instruction and a read of its result are the caller's — inside the
// contraction loop an accumulator is touched again only a whole half-step later.
// FRESH: an operand has just been written by ordinary vector instructions (8-bit weights
// widened to bf16); a matrix instruction may read such a register two issue cycles later at
// the earliest, which the compiler would see to for an instruction it knows.
template <bool FRESH>
static __device__ __forceinline__ void mfma16(bf16x8_t w, bf16x8_t x, f32x4_t &c) {
    if (FRESH) asm("s_nop 1\n\tv_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(w), "v"(x));
    else asm("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(w), "v"(x));
}

}  // namespace craft
