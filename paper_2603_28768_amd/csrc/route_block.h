// Routing of one block of 32 tokens by a workgroup of eight waves, a 16-lane row per token.
#pragma once

#include <type_traits>
#include <utility>

#include "kernels.h"

namespace craft {

constexpr int kRouteThreads = 16 * kTokPerBlock;   // a 16-lane row per token of the block
constexpr int kRouteMaxE = 1024;
constexpr int kMaxPickSlots = 4;     // k <= 64 picks, 16 lanes per token

typedef float score4_t __attribute__((ext_vector_type(4)));

template <int CTRL>
static __device__ __forceinline__ float dpp_f(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}
template <int CTRL>
static __device__ __forceinline__ int dpp_i(int v) {
    return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, true);
}
// lane exchange patterns that together reach every lane of a 16-lane row
constexpr int kXor1 = 0xB1, kXor2 = 0x4E, kHalfMirror = 0x141, kMirror = 0x140;

static __device__ __forceinline__ bool beats(float va, int ia, float vb, int ib) {
    return va > vb || (va == vb && ia < ib);
}

template <int CTRL>
static __device__ __forceinline__ void argmax_step(float &v, int &i) {
    const float ov = dpp_f<CTRL>(v);
    const int oi = dpp_i<CTRL>(i);
    if (beats(ov, oi, v, i)) { v = ov; i = oi; }
}

static __device__ __forceinline__ float row_sum(float v) {
    v += dpp_f<kXor1>(v);
    v += dpp_f<kXor2>(v);
    v += dpp_f<kHalfMirror>(v);
    v += dpp_f<kMirror>(v);
    return v;
}

static __device__ __forceinline__ uint64_t row_rotate(uint64_t v) {
    constexpr int kRor1 = 0x121;
    return (uint64_t)(uint32_t)dpp_i<kRor1>((int)(v >> 32)) << 32 | (uint32_t)dpp_i<kRor1>((int)v);
}
template <typename F, int... N>
static __device__ __forceinline__ void each_rotation(F &&f, std::integer_sequence<int, N...>) {
    (f(std::integral_constant<int, N>{}), ...);
}
// Score and expert as one integer that is larger for the better pick: the float's bits made
// monotone (-0 counts as 0), then the lower id.
static __device__ __forceinline__ uint64_t pick_key(float v, int id) {
    const uint32_t u = __float_as_uint(v + 0.0f);
    return (uint64_t)(u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u)) << 32 | (uint32_t)~id;
}
static __device__ __forceinline__ float key_score(uint64_t key) {
    const uint32_t u = (uint32_t)(key >> 32);
    return __uint_as_float(u ^ (((int32_t)u >> 31 ? 0u : ~0u) | 0x80000000u));
}
// How many of the row's 16 NC candidates beat the lane's own ones.  The row goes round one lane at a
// time: rotations by every distance at once take registers that cost waves.
template <int NC>
static __device__ __forceinline__ void row_rank(const uint64_t (&key)[NC], int (&rank)[NC]) {
    uint64_t at[NC];
#pragma unroll
    for (int i = 0; i < NC; ++i) { at[i] = key[i]; rank[i] = 0; }
#pragma unroll 1
    for (int n = 0; n < 16; n += 4) {
#pragma unroll
        for (int m = 0; m < 4; ++m) {
#pragma unroll
            for (int i = 0; i < NC; ++i)
#pragma unroll
                for (int j = 0; j < NC; ++j) rank[j] += at[i] > key[j] ? 1 : 0;
#pragma unroll
            for (int i = 0; i < NC; ++i) at[i] = row_rotate(at[i]);
        }
    }
}

// Token t of the block (place tl in it, live: it exists): its k picks and their weights, written where
// `write`; my_id[s] is the expert of pick 16 s + sub of the lane's token, or -1.  mask: per expert the
// block's tokens that chose it, cleared beforehand; may be null.
// NQ = 16-byte score chunks per lane (each chunk = 4 experts; a row covers 64 experts per chunk).
// PARTS: the scores come as partial sums of the gating network.
template <int NQ, bool PARTS>
static __device__ __forceinline__ void route_block(const RouteArgs &a, int64_t t, int tl, bool write, uint32_t *mask,
                                                   uint64_t (*cand)[32], int (&my_id)[kMaxPickSlots]) {
    const int sub = threadIdx.x & 15;              // lane inside the token's row
    // 16-byte loads need every row 16-byte aligned; otherwise the scores are read one by one
    const bool vec_ok = (a.E & 3) == 0 && (reinterpret_cast<uintptr_t>(a.logits) & 15) == 0;
#pragma unroll
    for (int s = 0; s < kMaxPickSlots; ++s) my_id[s] = -1;
    const bool live = t < a.T;                 // uniform over the row
    const float *row = a.logits + (live ? t : 0) * a.E;

    // Experts past E and experts already picked hold -inf: a finite score always beats
    // them (k <= E, and scores are finite by contract).
    constexpr float kGone = -__builtin_huge_valf();
    float v[NQ][4];
    // no branch around a load, only one around all of them: they travel together
    auto load_row = [&](const float *from, float (&to)[NQ][4]) {
        if (vec_ok) {
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                // (a vector type, not float4: four loads of a struct are merged with the other branch's)
                const score4_t f = *reinterpret_cast<const score4_t *>(from + min(q * 64 + sub * 4, a.E - 4));
                to[q][0] = f[0]; to[q][1] = f[1]; to[q][2] = f[2]; to[q][3] = f[3];
            }
        } else {
#pragma unroll
            for (int q = 0; q < NQ; ++q)
#pragma unroll
                for (int c = 0; c < 4; ++c) to[q][c] = from[min(q * 64 + sub * 4 + c, a.E - 1)];
        }
    };
    auto load_scores = [&]() {
        load_row(row, v);
        // the gate's partial scores, added in ascending order of the split; a few parts are
        // requested together, one by one each would cost a round trip
        constexpr int G = NQ <= 4 ? 7 : 3;
        if (PARTS)
            for (int z0 = 1; z0 < a.nparts; z0 += G) {
                float f[G][NQ][4];
#pragma unroll
                for (int g = 0; g < G; ++g) load_row(row + (int64_t)min(z0 + g, a.nparts - 1) * a.T * a.E, f[g]);
#pragma unroll
                for (int g = 0; g < G; ++g)
                    if (z0 + g < a.nparts)
#pragma unroll
                        for (int q = 0; q < NQ; ++q)
#pragma unroll
                            for (int c = 0; c < 4; ++c) v[q][c] += f[g][q][c];
            }
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (q * 64 + sub * 4 + c >= a.E) v[q][c] = kGone;
    };
    load_scores();

    float pick_v[kMaxPickSlots];
    float first_v = 0.0f;
#pragma unroll
    for (int s = 0; s < kMaxPickSlots; ++s) pick_v[s] = 0.0f;

    // Few of the row's scores can be among its k best: the k-th largest of the 16 lanes' maxima
    // is a bound that k of them reach, and a dozen or so reach in all.  Those are gathered
    // through LDS, one or two to a lane, and each finds its place by being compared with
    // every other.  Not for few picks, which the rounds make sooner, the fewer scores a lane has;
    // not where fewer lanes than picks have a score, or from 14 picks on (15 of one chunk): there
    // some row of nearly every wave has more than 32 above its bound, and the rounds come on top.
    // T = 131072, against k arg-max rounds: E = 64, k = 4 17.8 / 15.8 us, k = 5 0.99 of their time,
    // k = 8 0.74; E = 128, k = 2 1.36, 4 1.00, 8 0.64, 13 0.72; E = 256, k = 2 1.07, 3 0.96, 8 0.54;
    // E = 384, k = 1 0.97, 8 0.54, 14 1.05.
    constexpr int kFewest = NQ == 1 ? 5 : NQ == 2 ? 4 : NQ <= 4 ? 3 : NQ <= 6 ? 2 : 1, kMost = NQ == 1 ? 14 : 13;
    const bool few = NQ <= 8 && a.k >= kFewest && a.k <= kMost && 4 * a.k <= a.E + 3;   // (more than 512 scores: no registers)
    int n_cand = 0;
    float bound = kGone;
    if (few) {
        float top = v[0][0];
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
            for (int c = 0; c < 4; ++c) top = fmaxf(top, v[q][c]);
        int above = 0;
        each_rotation([&](auto n) {
            if constexpr (n.value > 0) above += dpp_f<0x120 + n.value>(top) > top ? 1 : 0;
        }, std::make_integer_sequence<int, 16>{});
        bound = above < a.k ? top : __builtin_huge_valf();
        bound = fminf(bound, dpp_f<kXor1>(bound));
        bound = fminf(bound, dpp_f<kXor2>(bound));
        bound = fminf(bound, dpp_f<kHalfMirror>(bound));
        bound = fminf(bound, dpp_f<kMirror>(bound));
        first_v = fmaxf(top, dpp_f<kXor1>(top));
        first_v = fmaxf(first_v, dpp_f<kXor2>(first_v));
        first_v = fmaxf(first_v, dpp_f<kHalfMirror>(first_v));
        first_v = fmaxf(first_v, dpp_f<kMirror>(first_v));
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
            for (int c = 0; c < 4; ++c) n_cand += v[q][c] >= bound ? 1 : 0;
    }
    int upto = n_cand;                         // candidates of this lane and the ones before it
    upto += dpp_i<0x111>(upto);
    upto += dpp_i<0x112>(upto);
    upto += dpp_i<0x114>(upto);
    upto += dpp_i<0x118>(upto);
    const int row_cands = __shfl(upto, 15, 16);
    if (few && __ballot(row_cands > 32 || row_cands < a.k) == 0) {
        int at = upto - n_cand;
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (v[q][c] >= bound) cand[tl][at++] = pick_key(v[q][c], q * 64 + sub * 4 + c);
        __builtin_amdgcn_wave_barrier();       // one wave's own rows: LDS keeps its order
        const bool wide = __ballot(row_cands > 16) != 0;
        uint64_t key[2] = {sub < row_cands ? cand[tl][sub] : 0, 0};
        int rank[2] = {0, 32};
        if (wide) {
            key[1] = 16 + sub < row_cands ? cand[tl][16 + sub] : 0;
            row_rank(key, rank);
        } else {
            const uint64_t one[1] = {key[0]};
            int r[1];
            row_rank(one, r);
            rank[0] = r[0];
        }
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int i = 0; i < 2; ++i)
            if (key[i] && rank[i] < a.k) cand[tl][rank[i]] = key[i];
        __builtin_amdgcn_wave_barrier();
        if (sub < a.k) {
            const uint64_t mine = cand[tl][sub];
            pick_v[0] = key_score(mine);
            my_id[0] = (int)~(uint32_t)mine;
        }
    } else {
#pragma unroll
        for (int s = 0; s < kMaxPickSlots; ++s) {
            const int jn = min(16, a.k - s * 16);  // picks that land in slot s
            for (int j = 0; j < jn; ++j) {
                // the lane's best, in ascending expert order: a later one wins only when
                // strictly greater, so equal scores keep the lower id
                float bv = v[0][0];
                int bi = sub * 4;
                if (NQ == 2) {
                    // as a tournament: a shorter chain (64 picks of 128 scores, 4096 tokens: 20.2 -> 19.4 us);
                    // more scores would take registers that cost waves
                    float tv[8];
                    int ti[8];
#pragma unroll
                    for (int i = 0; i < 8; ++i) { tv[i] = v[i / 4 < NQ ? i / 4 : 0][i % 4]; ti[i] = i / 4 * 64 + sub * 4 + i % 4; }
#pragma unroll
                    for (int width = 1; width < 8; width *= 2)
#pragma unroll
                        for (int i = 0; i + width < 8; i += 2 * width)
                            if (tv[i + width] > tv[i]) { tv[i] = tv[i + width]; ti[i] = ti[i + width]; }
                    bv = tv[0];
                    bi = ti[0];
                } else {
#pragma unroll
                    for (int q = 0; q < NQ; ++q)
#pragma unroll
                        for (int c = 0; c < 4; ++c)
                            if (v[q][c] > bv) { bv = v[q][c]; bi = q * 64 + sub * 4 + c; }
                }
                argmax_step<kXor1>(bv, bi);
                argmax_step<kXor2>(bv, bi);
                argmax_step<kHalfMirror>(bv, bi);
                argmax_step<kMirror>(bv, bi);
                // the owner retires the pick; lane j of the row keeps it for the output
#pragma unroll
                for (int q = 0; q < NQ; ++q)
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        if (bi == q * 64 + sub * 4 + c) v[q][c] = kGone;
                if (j == sub) { pick_v[s] = bv; my_id[s] = bi; }
                if (s == 0 && j == 0) first_v = bv;       // the row maximum
            }
        }
    }
    // softmax weight of the picks
    float ex[kMaxPickSlots], part = 0.0f;
#pragma unroll
    for (int s = 0; s < kMaxPickSlots; ++s) {
        ex[s] = s * 16 + sub < a.k ? expf(pick_v[s] - first_v) : 0.0f;
        part += ex[s];
    }
    if (!a.renorm) {
        load_scores();                         // the picks were blanked out: read the row again
        part = 0.0f;
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (q * 64 + sub * 4 + c < a.E) part += expf(v[q][c] - first_v);
    }
    const float den = row_sum(part);
    if (live) {
#pragma unroll
        for (int s = 0; s < kMaxPickSlots; ++s) {
            const int j = s * 16 + sub;
            if (j < a.k) {
                if (write) {
                    a.ids[t * a.k + j] = my_id[s];
                    a.w[t * a.k + j] = ex[s] / den;
                }
                if (mask) atomicOr(&mask[my_id[s]], 1u << tl);
            }
        }
    } else {
#pragma unroll
        for (int s = 0; s < kMaxPickSlots; ++s) my_id[s] = -1;
    }
}

}  // namespace craft
