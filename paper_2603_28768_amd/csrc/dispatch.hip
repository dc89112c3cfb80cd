// Expert-load counts and replica-aware stable dispatch (Sec. 1 / Alg. 1: a replicated
// expert's tokens are spread evenly over its copies).
//
// The i-th assignment (in flat token-major order) that names expert e goes to that
// expert's copy i mod c_e, and is the (i div c_e)-th row of that copy's slot.  i is
// assembled from two parts: the assignment's rank inside its 32-token block (recorded by
// the routing kernel) and the number of assignments to e in all earlier blocks.  The latter is an
// exclusive prefix over blocks, either from scan_kernel, which also leaves the slots' offsets, for
// dispatch_kernel; or put together by every workgroup of dispatch_direct_kernel for itself, from
// the counts of a few blocks or prefix_kernel's totals of chunks of them (see direct_dispatch for which).
// No result depends on the order in which atomics retire, so indices are reproducible bit for bit.
#include <algorithm>

#include "route_block.h"

namespace craft {
namespace {

constexpr int kScanThreads = 1024;
constexpr int kScanWaves = kScanThreads / 64;
static_assert(kScanChunk % kScanWaves == 0, "a chunk is dealt to the waves in equal parts");

// Exclusive scan over the workgroup of one value per thread (wave shuffles, then one LDS
// exchange between the WAVES waves).  Returns the exclusive prefix; *total gets the sum.
template <int WAVES>
__device__ __forceinline__ int32_t block_exclusive_scan(int32_t v, int32_t *wsum /*[WAVES]*/,
                                                        int32_t *total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int32_t inc = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int32_t o = __shfl_up(inc, off, 64);
        if (lane >= off) inc += o;
    }
    __syncthreads();                       // wsum may still be read from an earlier scan
    if (lane == 63) wsum[wave] = inc;
    __syncthreads();
    int32_t before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
        const int32_t s = wsum[w];
        if (w < wave) before += s;
        all += s;
    }
    *total = all;
    return before + inc - v;
}

// Blocks of tokens are taken in chunks of kScanChunk; a workgroup handles one chunk for 64
// experts (a single workgroup walks over all experts when there is only one chunk).  Wave w
// owns 16 consecutive blocks of the chunk and a lane owns one expert: each wave sums its
// blocks (kept in registers), the waves' sums are prefix-combined through LDS, and the
// per-block counts are rewritten as exclusive prefixes inside the chunk.  With several
// chunks the chunk totals go to memory and the workgroup that finishes last (ticket
// counter) turns them into per-chunk bases, which the dispatch kernel adds.  That workgroup
// (trivially the only one) also derives what needs all counts and what the dispatch indices
// wait for: rows per slot, slot offsets and the rank's row count.
__global__ __launch_bounds__(kScanThreads) void scan_kernel(ScanArgs a) {
    __shared__ int32_t part[kScanWaves][64];
    __shared__ int32_t wsum[kScanWaves];
    __shared__ int32_t cnt_lds[1024];
    __shared__ int32_t last_flag;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    constexpr int kKeep = kScanChunk / kScanWaves;         // blocks per wave
    const bool single = gridDim.x == 1;
    const int groups = (a.E + 63) / 64;
    const int chunk = single ? 0 : (int)blockIdx.x / groups;
    const int cb1 = min(a.NB, (chunk + 1) * kScanChunk);
    const int b0 = min(cb1, chunk * kScanChunk + wave * kKeep), b1 = min(cb1, b0 + kKeep);

    for (int grp = single ? 0 : (int)blockIdx.x % groups; grp < (single ? groups : (int)blockIdx.x % groups + 1); ++grp) {
        const int e = grp * 64 + lane;
        int32_t keep[kKeep];
        int32_t sum = 0;
        if (e < a.E) {
#pragma unroll
            for (int i = 0; i < kKeep; ++i) {
                keep[i] = b0 + i < b1 ? a.hist[(int64_t)(b0 + i) * a.E + e] : 0;
                sum += keep[i];
            }
        }
        part[wave][lane] = sum;
        __syncthreads();
        int32_t before = 0, total = 0;
#pragma unroll
        for (int w = 0; w < kScanWaves; ++w) {
            const int32_t v = part[w][lane];
            if (w < wave) before += v;
            total += v;
        }
        if (e < a.E) {
            int32_t run = before;
#pragma unroll
            for (int i = 0; i < kKeep; ++i)
                if (b0 + i < b1) { a.hist[(int64_t)(b0 + i) * a.E + e] = run; run += keep[i]; }
            if (wave == 0) {
                if (single) {
                    a.counts[e] = total;
                    if (a.user_counts) a.user_counts[e] = total;
                    cnt_lds[e] = total;
                } else {
                    a.chunk_tot[(int64_t)chunk * a.E + e] = total;
                }
            }
        }
        __syncthreads();                   // `part` is reused by the next group
    }

    if (!single) {
        // publish, then take a ticket
        __threadfence();
        __syncthreads();
        if (threadIdx.x == 0) {
            const int32_t ticket = atomicAdd(&a.ctrl[CTRL_TICKET], 1);
            last_flag = ticket == (int32_t)gridDim.x - 1;
        }
        __syncthreads();
        if (!last_flag) return;
        __threadfence();
        // chunk totals -> chunk bases and the experts' counts
        const int chunks = (int)gridDim.x / groups;
        for (int32_t e = threadIdx.x; e < a.E; e += kScanThreads) {
            int32_t run = 0;
            for (int c = 0; c < chunks; ++c) {
                a.chunk_base[(int64_t)c * a.E + e] = run;
                run += __hip_atomic_load(a.chunk_tot + (int64_t)c * a.E + e, __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_AGENT);
            }
            a.counts[e] = run;
            if (a.user_counts) a.user_counts[e] = run;
            cnt_lds[e] = run;
        }
    }
    __syncthreads();

    const craft_tables_header *hdr = reinterpret_cast<const craft_tables_header *>(a.tables);
    const int32_t *copies = a.tables + hdr->off_copies;
    const int32_t *slot_expert = a.tables + hdr->off_slot_expert;
    const int32_t *slot_copy = a.tables + hdr->off_slot_copy;

    // rows of slot p: tokens i < n of its expert with i mod c == q.  Slots are taken in
    // chunks of one per thread; `carry` is the running offset across chunks.
    // The two offsets that bound the rank's rows stay in LDS: reading them back from global
    // memory would be one more dependent round trip in this serial tail.
    __shared__ int32_t bound_pos[2];
    int32_t carry = 0, lo_pos = 0, hi_pos = 0;
    for (int32_t base = 0; base < a.S; base += kScanThreads) {
        const int32_t p = base + threadIdx.x;
        int32_t r = 0;
        if (p < a.S) {
            const int32_t ex = slot_expert[p];
            const int32_t n = cnt_lds[ex], c = copies[ex], q = slot_copy[p];
            r = n > q ? (n - q + c - 1) / c : 0;
        }
        int32_t chunk_total;
        const int32_t off = carry + block_exclusive_scan<kScanWaves>(r, wsum, &chunk_total);
        if (p < a.S) {
            a.slot_cnt[p] = r;
            a.slot_off[p] = off;
            if (a.user_slot_cnt) a.user_slot_cnt[p] = r;
            if (a.user_slot_off) a.user_slot_off[p] = off;
            if (p == a.s_lo) bound_pos[0] = off;
            if (p == a.s_hi) bound_pos[1] = off;
        }
        carry += chunk_total;
    }
    if (threadIdx.x == 0) {
        a.slot_off[a.S] = carry;
        if (a.user_slot_off) a.user_slot_off[a.S] = carry;
    }
    __syncthreads();
    lo_pos = a.s_lo < a.S ? bound_pos[0] : carry;
    hi_pos = a.s_hi < a.S ? bound_pos[1] : carry;
    // this rank's rows; refuse the batch when they exceed the staging buffers
    const int32_t rank_rows = hi_pos - lo_pos;
    const bool ovf = (int64_t)rank_rows > a.max_rows;
    if (threadIdx.x == 0) {
        a.ctrl[CTRL_ROWS] = rank_rows;
        a.ctrl[CTRL_OVERFLOW] = ovf ? 1 : 0;
        a.ctrl[CTRL_TICKET] = 0;
    }
}

// Rider units: one per tile of the busy slots while they last; a two-fragment slot (4 nt units) is
// carried whole or not at all.
__device__ __forceinline__ int32_t rider_units(int64_t nt, int32_t cut, int32_t hot_mtiles, int32_t ncold, int32_t ncold2) {
    const int64_t units2 = (int64_t)ncold2 * 4 * nt, units = units2 + (int64_t)(ncold - ncold2) * 2 * nt;
    int64_t carried = tile_height(cut) <= kRiderHostFrags ? min((int64_t)hot_mtiles * nt, units) : 0;
    if (nt > 0 && carried < units2) carried = carried / (4 * nt) * (4 * nt);
    return (int32_t)carried;
}

// The tables of build_tile_tables for up to 64 slots: one wave, a slot per lane, and not a barrier (the
// general form waits at two dozen).  They are what the dispatch launch of a small batch ends with.  A
// forward with the general form / this, us: 8 tokens on 3 slots 16.1 / 14.5, on 17 17.9 / 16.3, on 34 18.5 /
// 17.5, on 64 19.4 / 19.3; 4096 tokens on 17 slots 39.2 / 37.6; 256 tokens of the tiny fp32 layer 23.6 / 21.9.
template <typename ROWS>
__device__ void build_tile_tables_wave(const DispatchArgs &a, bool ovf, const ROWS &rows_of) {
    const int32_t nslots = a.s_hi - a.s_lo, lane = threadIdx.x;
    const int32_t mine = lane < nslots ? rows_of(lane) : -1;
    int32_t pos = lane < nslots ? 0 : lane;
    for (int32_t j = 0; j < nslots; ++j) {
        const int32_t other = __builtin_amdgcn_readlane(mine, j);
        pos += lane < nslots && (other > mine || (other == mine && j < lane)) ? 1 : 0;
    }
    if (lane < nslots) a.order[pos] = lane;
    const int32_t sorted = __builtin_amdgcn_ds_permute(pos * 4, mine);     // rows of the slot at this lane's position
    const int32_t hot = ovf ? 0 : __popcll(__ballot(sorted > kColdRows)), live = ovf ? 0 : __popcll(__ballot(sorted > 0));
    const int32_t ncold = live - hot, ncold2 = ovf ? 0 : __popcll(__ballot(sorted > 32)) - hot;
    const int32_t F = sorted > 0 && !ovf ? (sorted + 31) >> 5 : 0;
    const int32_t cut[2] = {a.frags_gu, a.frags_dn};
    int32_t mt[2], run[2];
#pragma unroll
    for (int kind = 0; kind < 2; ++kind) run[kind] = mt[kind] = row_tiles(F, cut[kind]);
#pragma unroll
    for (int d = 1; d < 64; d *= 2) {
        const int32_t up[2] = {__shfl_up(run[0], d, 64), __shfl_up(run[1], d, 64)};
#pragma unroll
        for (int kind = 0; kind < 2; ++kind) run[kind] += lane >= d ? up[kind] : 0;
    }
    int32_t riders[2], mtotal[2];
#pragma unroll
    for (int kind = 0; kind < 2; ++kind) {
        int32_t *mt_out = a.mt_start + kind * (nslots + 1);
        if (lane < nslots) mt_out[lane] = run[kind] - mt[kind];
        mtotal[kind] = __builtin_amdgcn_readlane(run[kind], 63);
        if (lane == 0) mt_out[nslots] = mtotal[kind];
        const int32_t hot_mtiles = hot > 0 ? __builtin_amdgcn_readlane(run[kind], hot - 1) : 0;
        riders[kind] = rider_units(kind == 0 ? a.nt_gu : a.nt_dn, cut[kind], hot_mtiles, ncold, ncold2);
    }
    if (lane == 0) {
        a.ctrl[CTRL_HOT_SLOTS] = hot;
        a.ctrl[CTRL_LIVE_SLOTS] = live;
        a.ctrl[CTRL_COLD2_SLOTS] = ncold2;
        a.ctrl[CTRL_RIDERS_GATEUP] = riders[0];
        a.ctrl[CTRL_RIDERS_DOWN] = riders[1];
        a.ctrl[CTRL_MTILES] = mtotal[0];
    }
}

// What the grouped GEMMs need beyond the slot offsets: the rank's slots ordered by rows, the
// row-tile prefixes of both GEMMs over that order and the rider units.  None of it is needed
// for the dispatch indices, so it is built by one extra workgroup of the dispatch launch
// while the others write dest / src, instead of at the end of the scan's serial tail.
template <int kTableThreads, typename ROWS>
__device__ void build_tile_tables(const DispatchArgs &a, bool ovf, const ROWS &rows_of) {
    __shared__ int32_t rank_slot_rows[1024];
    __shared__ int32_t sorted_rows[1024];
    __shared__ int32_t wsum[kTableThreads / 64];
    __shared__ int32_t prefix_len[3];
    __shared__ int32_t hot_mtiles;
    const int32_t nslots = a.s_hi - a.s_lo;
    if (nslots <= 64) {
        if (threadIdx.x < 64) build_tile_tables_wave(a, ovf, rows_of);
        return;
    }
    for (int32_t sl = threadIdx.x; sl < nslots; sl += kTableThreads) rank_slot_rows[sl] = rows_of(sl);
    if (threadIdx.x < 3) prefix_len[threadIdx.x] = 0;
    __syncthreads();
    // Order the rank's slots by rows, busiest first (ties: lower slot), so the tile list
    // starts with the matrix-bound tiles and ends with the cheap weight-streaming ones.
    for (int32_t sl = threadIdx.x; sl < nslots; sl += kTableThreads) {
        const int32_t mine = rank_slot_rows[sl];
        int32_t pos = 0;
        for (int32_t j = 0; j < nslots; ++j) {
            const int32_t other = rank_slot_rows[j];
            pos += (other > mine || (other == mine && j < sl)) ? 1 : 0;
        }
        a.order[pos] = sl;
        sorted_rows[pos] = mine;
    }
    __syncthreads();
    // the busy and the live slots are prefixes of the busiest-first order, and so are the slots
    // with more than one fragment
    for (int32_t pos = threadIdx.x; pos < nslots; pos += kTableThreads) {
        const int32_t r = sorted_rows[pos], nxt = pos + 1 < nslots ? sorted_rows[pos + 1] : 0;
        if (r > kColdRows && nxt <= kColdRows) prefix_len[0] = pos + 1;
        if (r > 0 && nxt <= 0) prefix_len[1] = pos + 1;
        if (r > 32 && nxt <= 32) prefix_len[2] = pos + 1;
    }
    __syncthreads();
    const int32_t hot = ovf ? 0 : prefix_len[0], live = ovf ? 0 : prefix_len[1];
    const int32_t ncold = live - hot;
    const int32_t ncold2 = max(0, min(prefix_len[2], live) - hot);   // cold slots with two fragments
    // row-tiles per slot: its 32-row fragments over the launch's tile height, rounded up
    int32_t mtotal[2], riders[2];
    for (int kind = 0; kind < 2; ++kind) {
        const int32_t cut = kind == 0 ? a.frags_gu : a.frags_dn;
        int32_t *mt_out = a.mt_start + kind * (nslots + 1);
        int32_t carry = 0;
        if (threadIdx.x == 0) hot_mtiles = 0;
        __syncthreads();
        for (int32_t base = 0; base < nslots; base += kTableThreads) {
            const int32_t pos = base + threadIdx.x;
            const int32_t F = pos < nslots && !ovf ? (sorted_rows[pos] + 31) >> 5 : 0;
            const int32_t mt = row_tiles(F, cut);
            int32_t chunk_total;
            const int32_t off = carry + block_exclusive_scan<kTableThreads / 64>(mt, wsum, &chunk_total);
            if (pos < nslots) mt_out[pos] = off;
            if (pos == hot) hot_mtiles = off;      // row-tiles of the busy slots
            carry += chunk_total;
        }
        __syncthreads();
        if (threadIdx.x == 0) mt_out[nslots] = carry;
        if (threadIdx.x == 0 && hot >= nslots) hot_mtiles = carry;
        mtotal[kind] = carry;
        __syncthreads();
        riders[kind] = rider_units(kind == 0 ? a.nt_gu : a.nt_dn, cut, hot_mtiles, ncold, ncold2);
        __syncthreads();                           // hot_mtiles is rewritten by the next kind
    }
    if (threadIdx.x == 0) {
        a.ctrl[CTRL_HOT_SLOTS] = hot;
        a.ctrl[CTRL_LIVE_SLOTS] = live;
        a.ctrl[CTRL_COLD2_SLOTS] = ncold2;
        a.ctrl[CTRL_RIDERS_GATEUP] = riders[0];
        a.ctrl[CTRL_RIDERS_DOWN] = riders[1];
        a.ctrl[CTRL_MTILES] = mtotal[0];
    }
}

__global__ __launch_bounds__(256) void dispatch_kernel(DispatchArgs a) {
    if (blockIdx.x == gridDim.x - 1) {             // the extra workgroup: tile tables of the GEMMs
        build_tile_tables<256>(a, a.ctrl[CTRL_OVERFLOW] != 0, [&](int32_t sl) { return a.slot_cnt[a.s_lo + sl]; });
        return;
    }
    const craft_tables_header *hdr = reinterpret_cast<const craft_tables_header *>(a.tables);
    const int32_t *copies = a.tables + hdr->off_copies;
    const int32_t *efirst = a.tables + hdr->off_efirst;
    const int32_t *eslots = a.tables + hdr->off_eslots;
    const int64_t A = a.T * a.k;
    const int32_t per_block = kTokPerBlock * a.k;
    const int32_t *base = a.base + (int64_t)blockIdx.x * a.E;
    // several chunks of blocks: the prefixes are chunk-local, the chunk's base comes on top
    const int32_t *cbase = a.chunk_base ? a.chunk_base + (int64_t)(blockIdx.x / kScanChunk) * a.E : nullptr;
    for (int32_t i = threadIdx.x; i < per_block; i += blockDim.x) {
        const int64_t as = (int64_t)blockIdx.x * per_block + i;
        if (as >= A) break;
        const int32_t e = a.ids[as];
        const int32_t idx = base[e] + (cbase ? cbase[e] : 0) + (int32_t)a.lrank[as];   // i-th assignment of expert e
        const int32_t c = copies[e];
        const int32_t q = idx % c;
        const int32_t p = eslots[efirst[e] + q];
        const int32_t d = a.slot_off[p] + idx / c;
        a.dest[as] = d;
        a.src[d] = (int32_t)as;
        if (a.user_dest) a.user_dest[as] = d;
        if (a.user_src) a.user_src[d] = (int32_t)as;
    }
}

// Per-expert prefixes over the blocks of a chunk and the chunk's totals, nothing that needs another
// workgroup's results: a workgroup takes kDirectChunk blocks for 64 experts, a wave an eighth of
// them, a lane one expert.
constexpr int kDirectWaves = 8;
__global__ __launch_bounds__(64 * kDirectWaves) void prefix_kernel(int32_t *hist, int32_t *tot, int32_t NB, int32_t E) {
    __shared__ int32_t part[kDirectWaves][64];
    constexpr int kKeep = kDirectChunk / kDirectWaves;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int groups = (E + 63) / 64, chunk = blockIdx.x / groups, e = blockIdx.x % groups * 64 + lane;
    const int b0 = chunk * kDirectChunk + wave * kKeep;
    int32_t keep[kKeep], sum = 0;
#pragma unroll
    for (int i = 0; i < kKeep; ++i) keep[i] = hist[(int64_t)min(b0 + i, NB - 1) * E + min(e, E - 1)];
#pragma unroll
    for (int i = 0; i < kKeep; ++i) sum += b0 + i < NB ? keep[i] : 0;
    part[wave][lane] = sum;
    __syncthreads();
    int32_t run = 0, total = 0;
#pragma unroll
    for (int w = 0; w < kDirectWaves; ++w) {
        const int32_t v = part[w][lane];
        if (w < wave) run += v;
        total += v;
    }
    if (e >= E) return;
#pragma unroll
    for (int i = 0; i < kKeep; ++i)
        if (b0 + i < NB) { hist[(int64_t)(b0 + i) * E + e] = run; run += keep[i]; }
    if (wave == 0) tot[(int64_t)chunk * E + e] = total;
}

// Dispatch without a serial step in front of it.  Every workgroup derives what it needs for itself
// -- the experts' counts from the totals of the chunks of blocks, the rows and offsets of the slots --
// and needs no other workgroup's results.  In a batch of up to kSmallBlocks blocks a chunk is a
// single block, whose counts the routing kernel has left: no other launch at all.  In a larger one
// prefix_kernel runs in front (a forward scanned / direct, us: E = 256, 8192 tokens 44.1 / 39.0, 32768 65.5 /
// 56.4, 65536 85.1 / 71.6; E = 384, 16384 58.1 / 48.3; E = 1024, 65536 223.6 / 183.7).
// A workgroup handles one block of 32 tokens, a few neighbouring ones in a large batch.  COPY, for the
// small-batch FFN: the token rows bound for this rank are copied into fragment order on the way, by
// sa.slices workgroups per block that take a share of the columns each (the first one writes
// dest / src).  The last workgroup builds the tile tables.
//
// NQ > 0, a batch of a single block: the workgroups route it as well, each for itself (the work of the
// routing kernel, which has a single workgroup for such a batch, too), and nothing about ids, ranks and
// counts goes through memory between two launches.  A forward with a routing launch / without, us: 8 tokens,
// E = 256, k = 8 22.0 / 20.0, with a gate's parts to add 34.9 / 32.0; 32 tokens, E = 384, k = 8 34.9 / 33.2, with
// parts 45.1 / 42.9; k = 64, where the arg-max rounds are most of it, 101.6 / 99.6 and with parts 157.1 / 155.8.
constexpr int kDirectThreads = 512;
constexpr int kDirectSlots = 2048;
static_assert(kDirectThreads == kRouteThreads, "a workgroup routes its block itself");
template <bool COPY, int NQ = 0, bool PARTS = false>
__global__ __launch_bounds__(kDirectThreads) void dispatch_direct_kernel(DirectDispatchArgs sa, RouteArgs ra) {
    const DispatchArgs &a = sa.d;
    constexpr bool ROUTE = NQ > 0;
    __shared__ uint32_t mask[ROUTE ? kRouteMaxE : 1];
    __shared__ uint64_t cand[ROUTE ? kTokPerBlock : 1][32];
    int my_id[kMaxPickSlots];
    const int tl = threadIdx.x >> 4, sub = threadIdx.x & 15;
    __shared__ int32_t cnt[1024], before[1024], ncopies[1024];
    __shared__ uint16_t first[1024], slots_of[kDirectSlots];
    __shared__ int32_t soff[kDirectSlots + 1];
    __shared__ int32_t wsum[kDirectThreads / 64];
    __shared__ int32_t list_len;
    __shared__ int32_t list[COPY ? 2 * kTokPerBlock * 64 : 1];     // token and packed row of the assignments to copy
    const int32_t *copies = a.tables + sa.lay.off_copies;
    const int32_t *efirst = a.tables + sa.lay.off_efirst;
    const int32_t *eslots = a.tables + sa.lay.off_eslots;
    const int32_t *slot_expert = a.tables + sa.lay.off_slot_expert;
    const int32_t *slot_copy = a.tables + sa.lay.off_slot_copy;
    const bool tables = blockIdx.x == gridDim.x - 1;
    // Workgroups go round the XCDs; neighbouring blocks stay on one: their entries of src lie side by
    // side, and a line that several XCDs write pieces of is written back by each of them.
    const int32_t spans = (int32_t)gridDim.x - 1;          // (with one slice: a multiple of 8)
    const int32_t turn = blockIdx.x / sa.slices, slice = blockIdx.x % sa.slices;
    const int32_t b = ROUTE ? 0 : (sa.slices > 1 ? turn : turn % 8 * (spans / 8) + turn / 8) * sa.span;
    const bool writer = tables;                            // of what there is one of per batch
    const int32_t own = b / sa.chunk_blocks;               // (a span lies inside one chunk)

    // Everything that is looked up through something else later on is requested here, at once:
    // the launch is a chain of round trips to memory, and this is the only long link.
    const int32_t per_block = kTokPerBlock * a.k, mine_n = per_block * sa.span;
    const int64_t A = a.T * a.k, as0 = (int64_t)b * per_block;
    constexpr int kFirst = 2;                              // assignments of a thread that are looked up ahead
    int32_t e0[kFirst], rank0[kFirst];                     // expert, place among its assignments of the chunk
#pragma unroll
    for (int u = 0; u < kFirst; ++u) {
        const int32_t i = threadIdx.x + u * kDirectThreads;
        const bool have = !ROUTE && !tables && i < mine_n && as0 + i < A;
        e0[u] = have ? a.ids[as0 + i] : 0;
        rank0[u] = have ? (int32_t)a.lrank[as0 + i] : 0;
    }
    const int32_t ex0 = threadIdx.x < sa.S ? slot_expert[threadIdx.x] : 0, q0 = threadIdx.x < sa.S ? slot_copy[threadIdx.x] : 0;
    for (int32_t p = threadIdx.x; p < sa.S; p += kDirectThreads) slots_of[p] = (uint16_t)eslots[p];
    if (threadIdx.x == 0) list_len = 0;
    if constexpr (ROUTE) {
        for (int32_t e = threadIdx.x; e < a.E; e += kDirectThreads) {
            ncopies[e] = copies[e];
            first[e] = (uint16_t)efirst[e];
            mask[e] = 0u;
        }
        if (writer && threadIdx.x < CTRL_WORDS) a.ctrl[threadIdx.x] = 0;
        __syncthreads();
        route_block<NQ, PARTS>(ra, tl, tl, writer, mask, cand, my_id);
        __syncthreads();
    }
    for (int32_t e = threadIdx.x; e < a.E; e += kDirectThreads) {
        int32_t total = 0, mine = 0;
        if constexpr (ROUTE) {
            cnt[e] = total = __popc(mask[e]);
            before[e] = 0;
            if (writer) {
                sa.counts[e] = total;
                if (sa.user_counts) sa.user_counts[e] = total;
            }
            continue;
        }
        ncopies[e] = copies[e];
        first[e] = (uint16_t)efirst[e];
        // Whole eights and a four are requested together, the few left one by one: each request of its own
        // is a round trip, but so is code that is fetched and not needed.  A forward one by one (whole
        // sixteens together) / always eight, the ones past the end masked / this, us, E = 256: 2 blocks
        // 18.76 / 19.33 / 18.98, 3 19.05 / 19.52 / 18.92, 8 21.25 / 20.36 / 19.86, 16 19.99 / 20.85 / 20.20,
        // 32 32.57 / 33.49 / 32.81; 8 chunks of them 57.97 / 56.12 / 55.68.
        int32_t i = 0;
        auto add = [&](auto together) {
            constexpr int G = decltype(together)::value;
            int32_t v[G];
#pragma unroll
            for (int u = 0; u < G; ++u) v[u] = sa.tot[(int64_t)(i + u) * a.E + e];
#pragma unroll
            for (int u = 0; u < G; ++u) {
                mine = i + u == own ? total : mine;
                total += v[u];
            }
            i += G;
        };
#pragma unroll 1
        while (i + 8 <= sa.ntot) add(std::integral_constant<int, 8>{});
        if (i + 4 <= sa.ntot) add(std::integral_constant<int, 4>{});
#pragma unroll 1
        while (i < sa.ntot) add(std::integral_constant<int, 1>{});
        cnt[e] = total;
        before[e] = mine;
        if (writer) {
            sa.counts[e] = total;
            if (sa.user_counts) sa.user_counts[e] = total;
        }
    }
    if (sa.local && !tables)
#pragma unroll
        for (int u = 0; u < kFirst; ++u) {
            const int32_t i = threadIdx.x + u * kDirectThreads;
            if (i < mine_n && as0 + i < A) rank0[u] += a.base[(int64_t)(b + i / per_block) * a.E + e0[u]];
        }
    __syncthreads();
    int32_t carry = 0;
    for (int32_t base = 0; base < sa.S; base += kDirectThreads) {
        const int32_t p = base + threadIdx.x;
        int32_t r = 0;
        if (p < sa.S) {
            const int32_t ex = base ? slot_expert[p] : ex0, q = base ? slot_copy[p] : q0;
            const int32_t n = cnt[ex], c = ncopies[ex];
            r = n > q ? (n - q + c - 1) / c : 0;
        }
        int32_t chunk_total;
        const int32_t off = carry + block_exclusive_scan<kDirectThreads / 64>(r, wsum, &chunk_total);
        if (p < sa.S) {
            soff[p] = off;
            if (writer) {
                sa.slot_cnt[p] = r;
                sa.slot_off_out[p] = off;
                if (sa.user_slot_cnt) sa.user_slot_cnt[p] = r;
                if (sa.user_slot_off) sa.user_slot_off[p] = off;
            }
        }
        carry += chunk_total;
    }
    if (threadIdx.x == 0) soff[sa.S] = carry;
    __syncthreads();
    const int32_t lo = soff[a.s_lo], hi = soff[a.s_hi];
    const bool ovf = (int64_t)(hi - lo) > sa.max_rows;
    if (tables) {
        if (threadIdx.x == 0) {
            sa.slot_off_out[sa.S] = carry;
            if (sa.user_slot_off) sa.user_slot_off[sa.S] = carry;
            a.ctrl[CTRL_ROWS] = hi - lo;
            a.ctrl[CTRL_OVERFLOW] = ovf ? 1 : 0;
        }
        build_tile_tables<kDirectThreads>(a, ovf, [&](int32_t sl) { return soff[a.s_lo + sl + 1] - soff[a.s_lo + sl]; });
        return;
    }

    auto place = [&](int32_t i, int32_t e, int32_t rank) {
        const int64_t as = as0 + i;
        const int32_t idx = before[e] + rank;
        const int32_t c = ncopies[e];
        const int32_t p = slots_of[first[e] + idx % c];
        const int32_t row = idx / c, d = soff[p] + row;
        if (slice == 0) {
            a.dest[as] = d;
            a.src[d] = (int32_t)as;
            if (a.user_dest) a.user_dest[as] = d;
            if (a.user_src) a.user_src[d] = (int32_t)as;
        }
        if (COPY && !ovf && p >= a.s_lo && p < a.s_hi) {
            const int32_t at = atomicAdd(&list_len, 1);    // the order of the copies does not matter
            list[2 * at] = (int32_t)(as / a.k);
            list[2 * at + 1] = stream_fragment(soff[p] - lo, p - a.s_lo, row) * 16 + (row & 15);
        }
    };
    if constexpr (ROUTE) {
#pragma unroll
        for (int s = 0; s < kMaxPickSlots; ++s)
            if (tl < a.T && s * 16 + sub < a.k)
                place(tl * a.k + s * 16 + sub, my_id[s], __popc(mask[my_id[s]] & ((1u << tl) - 1u)));
    } else {
#pragma unroll
        for (int u = 0; u < kFirst; ++u) {
            const int32_t i = threadIdx.x + u * kDirectThreads;
            if (i < mine_n && as0 + i < A) place(i, e0[u], rank0[u]);
        }
        for (int32_t i = threadIdx.x + kFirst * kDirectThreads; i < mine_n && as0 + i < A; i += kDirectThreads) {
            const int32_t e = a.ids[as0 + i];
            place(i, e, (int32_t)a.lrank[as0 + i] + (sa.local ? a.base[(int64_t)(b + i / per_block) * a.E + e] : 0));
        }
    }
    if (!COPY) return;
    __syncthreads();
    const int32_t pieces = sa.H >> 3;                      // 16-byte pieces of a row, this slice's share of them
    const int32_t c0 = (int32_t)((int64_t)pieces * slice / sa.slices), nc = (int32_t)((int64_t)pieces * (slice + 1) / sa.slices) - c0;
    const int64_t frag_bytes = (int64_t)((sa.H + 63) / 64) * 2048;
    const int32_t n = list_len * nc;
    for (int32_t i = threadIdx.x; i < n; i += kDirectThreads) {
        const int32_t at = i / nc, c = c0 + i % nc;
        const int32_t row = list[2 * at + 1];
        const uint4 v = reinterpret_cast<const uint4 *>(static_cast<const unsigned char *>(sa.x) + (int64_t)list[2 * at] * sa.H * 2)[c];
        *reinterpret_cast<uint4 *>(sa.xpk + (row >> 4) * frag_bytes + stream_piece((uint32_t)c, (uint32_t)row & 15u)) = v;
    }
}

}  // namespace

bool small_dispatch(int64_t T, int32_t S) { return T > 0 && T <= (int64_t)kSmallBlocks * kTokPerBlock && S <= kDirectSlots; }
// Up to 16 chunks: every workgroup reads all of their totals.  But every workgroup also goes over all the
// slots, 512 at a time, and where a single workgroup scans a batch quickly (one group of experts, one chunk
// of blocks) four such passes in each are the dearer way.  A forward scanned / direct, us (mean of both
// orders on one machine): E = 64, 1537 slots, T = 2048 27.5 / 28.1, 8192 38.0 / 39.2; 2044 slots, 4096 28.5 /
// 29.3; 1536 slots, 2048 27.2 / 27.3, 4096 27.7 / 27.9; 513 slots, 2048 24.6 / 24.7; 512 slots, 2048 24.4 /
// 23.8; 72 slots, 2048 33.3 / 32.9; E = 96, 1996 slots, 2048 29.9 / 29.4.
bool direct_dispatch(int64_t T, int32_t E, int32_t S) {
    if (small_dispatch(T, S)) return true;
    if (E <= 64 && S > 3 * kDirectThreads && T <= (int64_t)kScanChunk * kTokPerBlock) return false;
    return T > 0 && T <= 16ll * kDirectChunk * kTokPerBlock && S <= kDirectSlots;
}

hipError_t launch_prefix(int32_t *hist, int32_t *chunk_tot, int32_t NB, int32_t E, hipStream_t s) {
    if (NB <= kSmallBlocks) return hipSuccess;
    const unsigned grid = (unsigned)((NB + kDirectChunk - 1) / kDirectChunk) * (unsigned)((E + 63) / 64);
    hipLaunchKernelGGL(prefix_kernel, dim3(grid), dim3(64 * kDirectWaves), 0, s, hist, chunk_tot, NB, E);
    return hipGetLastError();
}

// One block: more would be routed one after the other by every workgroup.  E: up to what the scores of a
// lane fit registers beside the rest (and a gate's parts are added for).  Any number of picks and parts:
// over 137 forwards of 1, 8 and 32 tokens, E = 8 to 384, k = 1 to 64 it takes 0.79 to 1.00 of the time (one
// of them 0.97 and 1.02 in two runs).
bool routed_dispatch(int64_t T, int32_t E, int32_t S) { return T <= kTokPerBlock && E <= 384 && small_dispatch(T, S); }

hipError_t launch_dispatch_direct(DirectDispatchArgs a, const int32_t *chunk_tot, const RouteArgs *route, hipStream_t s) {
    const int32_t NB = (int32_t)((a.d.T + kTokPerBlock - 1) / kTokPerBlock);
    a.local = NB > kSmallBlocks;
    a.chunk_blocks = a.local ? kDirectChunk : 1;
    a.ntot = (NB + a.chunk_blocks - 1) / a.chunk_blocks;
    a.tot = a.local ? chunk_tot : a.d.base;
    // enough workgroups to copy at memory speed, at least a few hundred columns each
    a.slices = a.xpk ? std::max(1, std::min({256 / NB, a.H / 256, 16})) : 1;
    // what a workgroup derives for itself is worth a few blocks where there are enough of them
    a.span = 1;
    while (a.local && a.span < 8 && NB / (a.span * 2) >= 256) a.span *= 2;
    const int32_t spans = (NB + a.span - 1) / a.span;
    const dim3 grid((unsigned)((a.slices > 1 ? spans * a.slices : (spans + 7) / 8 * 8) + 1)), block(kDirectThreads);
    if (route) {
        const dim3 grid((unsigned)a.slices + 1);           // no workgroup without a share of the block
        auto go = [&](auto nq) {
            auto with = [&](auto copy) {
                if (route->nparts > 1) hipLaunchKernelGGL((dispatch_direct_kernel<copy.value, nq.value, true>), grid, block, 0, s, a, *route);
                else hipLaunchKernelGGL((dispatch_direct_kernel<copy.value, nq.value, false>), grid, block, 0, s, a, *route);
            };
            if (a.xpk) with(std::true_type{});
            else with(std::false_type{});
        };
        const int nq = (route->E + 63) / 64;
        if (nq <= 1) go(std::integral_constant<int, 1>{});
        else if (nq <= 2) go(std::integral_constant<int, 2>{});
        else if (nq <= 4) go(std::integral_constant<int, 4>{});
        else go(std::integral_constant<int, 6>{});
        return hipGetLastError();
    }
    if (a.xpk) hipLaunchKernelGGL(dispatch_direct_kernel<true>, grid, block, 0, s, a, RouteArgs{});
    else hipLaunchKernelGGL(dispatch_direct_kernel<false>, grid, block, 0, s, a, RouteArgs{});
    return hipGetLastError();
}

hipError_t launch_scan(const ScanArgs &a, hipStream_t s) {
    // one chunk of token blocks: one workgroup does everything; more: one per chunk and 64 experts
    const unsigned chunks = (unsigned)((a.NB + kScanChunk - 1) / kScanChunk);
    const unsigned blocks = chunks <= 1 ? 1u : chunks * (unsigned)((a.E + 63) / 64);
    hipLaunchKernelGGL(scan_kernel, dim3(blocks), dim3(kScanThreads), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_dispatch(const DispatchArgs &a, hipStream_t s) {
    if (a.T == 0) return hipSuccess;
    const int64_t nb = (a.T + kTokPerBlock - 1) / kTokPerBlock;
    hipLaunchKernelGGL(dispatch_kernel, dim3((unsigned)nb + 1), dim3(256), 0, s, a);
    return hipGetLastError();
}

}  // namespace craft
