// Internal launcher interface between the host API (forward.cpp) and the HIP kernels.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

#include "plan_internal.h"

namespace craft {

// Tokens handled by one workgroup of the routing and dispatch kernels.  Ranks of
// assignments inside a block are taken from a 32-bit token mask per expert.
constexpr int kTokPerBlock = 32;
// Blocks of tokens whose per-expert counts one workgroup of the scan kernel prefixes.
constexpr int kScanChunk = 256;

// Control words at the start of the workspace.
enum { CTRL_TICKET = 0, CTRL_ROWS = 1, CTRL_OVERFLOW = 2, CTRL_MTILES = 3,
       CTRL_HOT_SLOTS = 6,                         // slots of the rank with more than kColdRows rows
       CTRL_LIVE_SLOTS = 7,                        // slots of the rank with any rows
       CTRL_RIDERS_GATEUP = 8, CTRL_RIDERS_DOWN = 9,   // rider units carried by the busy slots' tiles, per GEMM
       CTRL_COLD2_SLOTS = 10,                      // cold slots with two fragments (33 .. kColdRows rows)
       CTRL_WORK_GATEUP = 4, CTRL_WORK_DOWN = 5,   // dynamic tile counters of the two GEMMs
       CTRL_WORDS = 16 };

// A slot with at most this many rows is "cold": its tiles do next to no matrix work and are
// bound by streaming the weights.  The packed FFN cuts their column tiles in half (twice as
// many, half as long), because what the tail of a launch costs is the length of a cold tile
// and the aggregate weight bandwidth grows with the number of CUs streaming at once.
constexpr int kColdRows = 64;

// Riders.  During a tile of a busy slot the CU's matrix pipeline is busy and HBM is not;
// during a cold slot's tile it is the other way round.  So a tile of a busy slot carries a
// "rider unit" along: one 32-row fragment of a cold slot against half a column tile of that
// slot's weights (one column group per wave), streamed through a second weight ring and
// costing four more MFMAs of 16 x 16 x 32 per 32-wide step.  Half a tile, not a whole one,
// because a CU's vector memory path (64 bytes per clock) is already two-thirds used by the
// tile's own operands.
// The units of the cold slots, in busiest-first order (two-fragment slots first), go to the
// tiles of the list one each, from the first tile on: unit u rides on tile u.  A two-fragment
// slot is carried whole or not at all.  Tiles of more than kRiderHostFrags fragments have no
// registers left for a rider: a launch with taller tiles carries none.
constexpr int kRiderHostFrags = 7;

// Most 32-row fragments a row-tile of the grouped GEMMs may have (the tile table is built for
// a height chosen per launch, up to these).
constexpr int kFragsBf16 = 4;      // LDS-staged bf16 kernels (row-major weights): 128 rows
constexpr int kFragsPacked = 8;    // weight-streaming bf16 kernels (packed weights): 256 rows
constexpr int kFragsF32 = 1;

// Small batches (ffn_stream.hip): most rows of a slot against one pass over its weights, and
// where its activations lie.  They are kept as operand fragments: 16 rows x 32 contraction
// elements are 64 lanes x 16 bytes, lane l holding row l & 15, elements 8 (l >> 4) .. + 7; the
// fragments of one row group follow one another, whole 64-wide slabs of them.  Read as rows, the
// 16 pieces of a request lie a row apart and cost more than the weights do (H = 7168, two slots of
// 57 and 52 rows: forward 78 us as rows, 61 as fragments).  A slot starts a fragment of its own;
// rows / 16 + slots before it is always room enough for the earlier ones.
constexpr int kStreamRows = 64;
__host__ __device__ inline int32_t stream_fragment(int32_t first_row, int32_t slot, int32_t row) {
    return (first_row >> 4) + slot + (row >> 4);
}
// byte offset of 16-byte piece c (elements 8c ..) of row r16 of a fragment row
__host__ __device__ inline uint32_t stream_piece(uint32_t c, uint32_t r16) {
    return (c >> 2) * 1024u + ((c & 3u) * 16u + r16) * 16u;
}
inline size_t stream_bytes(int64_t max_rows, int32_t nslots, int32_t K) {
    return (size_t)(max_rows / 16 + nslots + 1) * (size_t)((K + 63) / 64) * 2048;
}
constexpr int kBM_packed = kFragsPacked * 32;

// How a launch cuts the F 32-row fragments of a slot into row-tiles: frags > 0, tiles of that many
// and a remainder; frags < 0, ceil(10 F / -frags) tiles that share them as evenly as whole
// fragments allow (tenths, so that there are more than four ways to cut a few slots).
__host__ __device__ inline int32_t row_tiles(int32_t F, int32_t frags) {
    return frags > 0 ? (F + frags - 1) / frags : (10 * F - frags - 1) / -frags;
}
// most fragments of a row-tile
__host__ __device__ inline int32_t tile_height(int32_t frags) { return frags > 0 ? frags : (9 - frags) / 10; }

// Row-major bf16 FFN: whether the cold slots' tiles of a launch (`cold` at full width behind `busy` ones, contraction
// K) are a quarter as wide; ffn.hip says why, the choice of streaming asks the same for the loads it expects.
constexpr int kNarrowLength = 1024;                // contraction from which on a whole round of cold tiles may be
static inline __host__ __device__ bool narrow_cold_tiles(int64_t busy, int64_t cold, int64_t cus, int64_t K) {
    const int64_t over = busy % cus, room = over ? cus - over : 0;     // CUs without a tile of the last round of busy ones
    return busy + cold > cus && cold > room && cold * kNarrowLength <= cus * K;
}

struct RouterArgs {
    int32_t dtype;
    const void *x;            // [T][H]
    const void *w;            // [E][H] gate weights
    int64_t T;
    int32_t H, E;
    float *logits;            // [T][E]
    int32_t num_cu;
    float *part;              // [nsplit][T][E] partial scores when the contraction is split; may be null
    int32_t nsplit;           // set by the launcher: workgroups per tile
    bool keep_parts;          // with a split contraction: leave the sums to the reader of `part`
    // set by the launcher, so that no workgroup divides in front of its first request
    int32_t nparts = 1;       // parts of the contraction that are summed by themselves, a multiple of nsplit
    int32_t per = 0;          // slabs of a part
    int32_t share = 0;        // slabs of a workgroup
    int32_t eblocks = 0;      // blocks of experts, where those of a tile are to meet in one XCD; 0: numbered by the grid
    int32_t tiles = 0;        // tiles of tokens
    uint32_t eblocks_inv = 0, tiles_inv = 0;       // 2^32 / eblocks, 2^32 / tiles, rounded up
};
// nsplit: if not null, the copies of the scores left in `part` with keep_parts (1: none, they are in `logits`)
hipError_t launch_router_logits(const RouterArgs &a, hipStream_t s, int *nsplit = nullptr);
// Parts the contraction is summed in with a workspace, which is sized for them.
int router_logits_parts(int64_t T, int32_t H, int32_t E, int32_t num_cu);
struct RouterShape {
    int tokens;               // 32-token fragments of a tile
    int experts;              // most experts of a tile
    int nparts, nsplit;       // as in RouterArgs
};
RouterShape router_logits_shape(int64_t T, int32_t H, int32_t E, int32_t num_cu, bool workspace);

struct RouteArgs {
    const float *logits;
    int64_t T;
    int32_t E, k, renorm;
    int32_t *ids;       // [T][k]
    float *w;           // [T][k]
    uint8_t *lrank;     // [T][k] rank of the assignment among same-expert ones of its block; may be null
    int32_t *hist;      // [NB][E] per-block expert counts; may be null
    int32_t *ctrl;      // control words to clear; may be null
    int32_t nparts;     // > 1: a score is the sum of this many partial scores, [nparts][T][E] at `logits` (E <= 384)
};
hipError_t launch_route(const RouteArgs &a, hipStream_t s);

struct ScanArgs {
    int32_t *hist;            // [NB][E] in: counts per block; out: exclusive prefix over the blocks of a chunk
    int32_t *chunk_tot;       // [chunks][E] totals of the chunks (scratch; more than one chunk only)
    int32_t *chunk_base;      // [chunks][E] out: sum of the earlier chunks' totals
    int32_t NB, E;
    const int32_t *tables;    // device tables of this (layer, rank)
    int32_t S, s_lo, s_hi;
    int64_t max_rows;
    int32_t *counts;          // [E]
    int32_t *slot_cnt;        // [S]
    int32_t *slot_off;        // [S+1]
    int32_t *ctrl;
    int32_t *user_counts, *user_slot_cnt, *user_slot_off;   // optional copies
};
hipError_t launch_scan(const ScanArgs &a, hipStream_t s);

struct DispatchArgs {
    const int32_t *ids;
    const uint8_t *lrank;
    const int32_t *base;      // [NB][E] prefixes inside a chunk of blocks
    const int32_t *chunk_base; // [chunks][E] on top of them; null when there is one chunk
    int64_t T;
    int32_t k, E;
    const int32_t *tables;
    const int32_t *slot_off;
    int32_t *dest, *src;
    int32_t *user_dest, *user_src;
    // for the extra workgroup that builds the tile tables of the grouped GEMMs
    const int32_t *slot_cnt;  // [S] rows per slot
    int32_t s_lo, s_hi;       // the rank's slots
    int32_t frags_gu, frags_dn;   // how a slot's rows are cut (row_tiles), gate/up and down GEMM
    int32_t nt_gu, nt_dn;     // column tiles per slot of the two packed GEMMs; 0: no riders
    int32_t *mt_start;        // [2][s_hi - s_lo + 1] row-tile prefix over the rank's slots, busiest slot
                              // first: for the gate/up GEMM, then for the down GEMM
    int32_t *order;           // [s_hi - s_lo] local slot at each position of that order
    int32_t *ctrl;
};
hipError_t launch_dispatch(const DispatchArgs &a, hipStream_t s);

// Without the scan: see dispatch_direct_kernel, and direct_dispatch for where.  Batches of at most
// kSmallBlocks 32-token blocks need no other launch, larger ones launch_prefix over chunks of
// kDirectChunk blocks.
constexpr int kSmallBlocks = 32;
constexpr int kDirectChunk = kScanChunk / 2;   // the totals take the room of the scan's chunk_tot and chunk_base
struct DirectDispatchArgs {
    DispatchArgs d;           // base: the blocks' counts, or their prefixes inside a chunk; chunk_base, slot_off and slot_cnt unused
    craft_tables_header lay;  // of d.tables, known on the host: one round trip less
    int32_t S;
    int64_t max_rows;
    int32_t *counts, *slot_cnt, *slot_off_out;
    int32_t *user_counts, *user_slot_cnt, *user_slot_off;   // optional copies
    const void *x;            // [T][H] bf16
    int32_t H;
    unsigned char *xpk;       // where the small-batch FFN reads the token rows; null: not copied
    // set by the launcher
    const int32_t *tot;       // [ntot][E] counts of the chunks of blocks
    int32_t ntot, chunk_blocks, slices, span;
    bool local;               // the blocks' prefixes inside their chunk come on top
};
bool direct_dispatch(int64_t T, int32_t E, int32_t S);
bool small_dispatch(int64_t T, int32_t S);
hipError_t launch_prefix(int32_t *hist, int32_t *chunk_tot, int32_t NB, int32_t E, hipStream_t s);
// route: a batch for which routed_dispatch holds is routed by the same launch; else null
bool routed_dispatch(int64_t T, int32_t E, int32_t S);
hipError_t launch_dispatch_direct(DirectDispatchArgs a, const int32_t *chunk_tot, const RouteArgs *route, hipStream_t s);

struct FfnArgs {
    int32_t dtype;
    int32_t H, I, k;
    int32_t s_lo, nslots;
    const void *x;                 // [T][H]
    const int32_t *src;            // [A]
    const int32_t *slot_off;       // [S+1]
    const int32_t *mt_start;       // [2][nslots+1]: gate/up, down
    const int32_t *order;          // [nslots]
    int32_t *ctrl;
    const void *const *w_gate, *const *w_up, *const *w_down;   // row-major weights per slot
    const void *const *wp_gateup, *const *wp_down;             // fragment-packed weights per slot
    const void *xpk;               // small batches: token rows as fragments
    void *act;                     // [max_rows][I] SwiGLU activations; small batches: as fragments
    void *y;                       // [max_rows][H]
    int64_t max_rows;
    int32_t num_cu;
    int32_t w8;                    // packed weights are E4M3 codes with row scales behind the stream
    int32_t frags_gu, frags_dn;    // how the tile tables cut a slot's rows (row_tiles)
    bool far_x;                    // x has rows more than 4 GiB from its start (row-major weights only)
};
hipError_t launch_gateup(const FfnArgs &a, hipStream_t s);
hipError_t launch_down(const FfnArgs &a, hipStream_t s);
hipError_t launch_gateup_packed(const FfnArgs &a, hipStream_t s);
hipError_t launch_down_packed(const FfnArgs &a, hipStream_t s);
hipError_t launch_gateup_stream(const FfnArgs &a, bool packed, hipStream_t s);
hipError_t launch_down_stream(const FfnArgs &a, bool packed, hipStream_t s);
void packed_sizes(int32_t H, int32_t I, size_t *gateup_bytes, size_t *down_bytes);
hipError_t launch_pack(int32_t H, int32_t I, const void *wg, const void *wu, const void *wd,
                       void *pgu, void *pdn, hipStream_t s);
void packed_sizes_e4m3(int32_t H, int32_t I, size_t *gateup_bytes, size_t *down_bytes);
hipError_t launch_quantize_e4m3(const void *w, int64_t rows, int32_t K, uint8_t *codes, float *scale,
                                hipStream_t s);
hipError_t launch_quantize_pack_e4m3(int32_t H, int32_t I, const void *wg, const void *wu, const void *wd,
                                     void *pgu, void *pdn, hipStream_t s);
hipError_t launch_pack_e4m3(int32_t H, int32_t I, const uint8_t *cg, const uint8_t *cu, const uint8_t *cd,
                            const float *sg, const float *su, const float *sd, void *pgu, void *pdn,
                            hipStream_t s);

struct CombineArgs {
    int32_t dtype;
    int64_t T;
    int32_t k, H;
    const void *y;
    const int32_t *dest;
    const float *w;
    const int32_t *slot_off;
    int32_t s_lo, s_hi;
    const int32_t *ctrl;
    void *out;
};
hipError_t launch_combine(const CombineArgs &a, hipStream_t s);

struct LoadArgs {
    const int32_t *ids;       // [L][T][k]
    int32_t L, k, E;
    int64_t T, batch_tokens, B;
    int64_t *counts;          // [B][L][E]
};
hipError_t launch_expert_load(const LoadArgs &a, hipStream_t s);
hipError_t launch_probe_copy(const void *src, void *dst, int64_t bytes, int32_t num_cu, hipStream_t s);
hipError_t launch_probe_read(const void *src, int64_t bytes, int32_t passes, int32_t blocks, uint32_t *sink,
                             hipStream_t s);
hipError_t launch_probe_mfma(int32_t blocks, int32_t iters, float *sink, hipStream_t s);
hipError_t launch_probe_mfma_operands(int32_t shape, int32_t data, int32_t blocks, int32_t iters, float *sink,
                                      hipStream_t s);
hipError_t launch_load_accumulate(const int32_t *counts, int64_t n, int64_t *window, hipStream_t s);

}  // namespace craft
