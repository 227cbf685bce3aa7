// Greedy disjoint choice among adjacent layer pairs (Alg. 1, second loop; Sec. 4.2) for one
// conversation, run by all threads of a workgroup: shared by the selection kernel and by the
// kernel that averages heads and selects in one launch.
//
// The order of the candidates (adjacent pairs whose two layers are eligible): higher score first, equal
// scores lower index first.  A pair whose score is NaN has no place in that order: it is no candidate.
// Taking pairs in that order iff both layers are still free, until n_select are held, is what the algorithm asks for.
//
// Up to 128 layers it is found without the order: a pair that comes before both its neighbours, as far as they are still
// free, will be taken whatever else is, so all such pairs are taken at once, their neighbours drop out, and so on.  The pairs are
// bits of a mask, "the next pair comes first" another, and a round is a few scalar operations in every wave.  The first n_select of
// the pairs taken are those that the algorithm stops at; a pair's place among them is the number of taken pairs before it.
// (Ranked first and scanned by one wave, three barriers and a step per candidate: a call of 20 tokens
// over 300 keys that takes 16 pairs of 32 layers 27.6 us, 23.8 so.)
//
// Beyond, the candidates are ranked by counting -- rank(l) = number of candidates that come before l, 64 comparisons at a time (a wave
// per candidate, a lane per other candidate), the stable descending sort with no
// data-dependent control flow --, and one thread scans the ranked list.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace krul {

// The value of the lane OFF places on (lane ^ OFF), by vector instructions: a shuffle goes through LDS and takes ten times
// as long, and sums of this kind stand one after the other.
template <int OFF>
__device__ inline float across(float v)
{
    static_assert(OFF == 1 || OFF == 2 || OFF == 4 || OFF == 8 || OFF == 16 || OFF == 32, "a power of two below 64");
    const int i = __builtin_bit_cast(int, v);
    if constexpr (OFF >= 16) {   // (the lower and the upper rows' values, in every lane)
        const auto r = OFF == 32 ? __builtin_amdgcn_permlane32_swap((unsigned)i, (unsigned)i, false, false)
                                 : __builtin_amdgcn_permlane16_swap((unsigned)i, (unsigned)i, false, false);
        return __uint_as_float(__lane_id() & OFF ? r[0] : r[1]);
    }
    int o;
    if constexpr (OFF == 8) o = __builtin_amdgcn_mov_dpp(i, 0x128, 0xF, 0xF, true);        // row_ror 8
    else if constexpr (OFF == 2) o = __builtin_amdgcn_mov_dpp(i, 0x4E, 0xF, 0xF, true);    // quad_perm 2 3 0 1
    else if constexpr (OFF == 1) o = __builtin_amdgcn_mov_dpp(i, 0xB1, 0xF, 0xF, true);    // quad_perm 1 0 3 2
    else o = __builtin_amdgcn_mov_dpp(__builtin_amdgcn_mov_dpp(i, 0x141, 0xF, 0xF, true), 0x1B, 0xF, 0xF, true);   // row_half_mirror (7), quad_perm 3 2 1 0
    return __builtin_bit_cast(float, o);
}

// Average of a pair's Hq head values (times scale) by the 32 lanes of a half-wave: lane k takes heads k, k + 32, ... in
// order, a butterfly adds the lanes' sums.  The one order in which heads are averaged, whichever kernel does it.
// out: the scaled values go there, if anywhere; it may be head (every value is read once).
__device__ inline float pair_average(const float *head, int Hq, float scale, int lane, float *out = nullptr)
{
    float s = 0.f;
    for (int h = lane; h < Hq; h += 32) {
        const float v = head[h] * scale;
        if (out) out[h] = v;
        s += v;
    }
    s += across<16>(s);
    s += across<8>(s);
    s += across<4>(s);
    s += across<2>(s);
    s += across<1>(s);
    return s / (float)Hq;
}

// LDS bytes select_adjacent needs beside the scores: order [NP] int32, cand [NP], used [n_layers]
__host__ __device__ inline size_t select_scratch_bytes(int n_layers)
{
    return (size_t)(n_layers - 1) * (sizeof(int32_t) + 1) + (size_t)n_layers;
}

// score: the conversation's NP = n_layers - 1 pair scores in LDS (written before the call; the
// function starts with a barrier).  el: its eligibility bytes in global memory, or null.
// scratch: select_scratch_bytes(n_layers) bytes of LDS, 4-byte aligned.  out_pairs: n_select entries.
__device__ inline void select_adjacent(const float *score, const uint8_t *el, int n_layers, int n_select,
                                       int32_t *out_pairs, int32_t *out_count, void *scratch)
{
    const int NP = n_layers - 1;
    const int nt = blockDim.x;
    if (n_layers <= 128) {
        typedef unsigned __int128 Mask;   // bit l: pair l
        const int lane = threadIdx.x & 63;
        __syncthreads();   // (the scores)
        float s[2];
        Mask free = 0, next_first = 0;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int l = lane + 64 * i, at = min(l, NP - 1);
            s[i] = score[at];
            const bool candidate = l < NP && s[i] == s[i] && (!el || (el[at] && el[at + 1]));
            free |= (Mask)__ballot(candidate) << (64 * i);
            next_first |= (Mask)__ballot(score[min(l + 1, NP - 1)] > s[i]) << (64 * i);
        }
        Mask taken = 0;
        while (free) {   // (its best pair is taken in every round)
            const Mask now = free & ~((next_first & (free >> 1)) | ((~next_first & free) << 1));
            taken |= now;
            free &= ~(now | (now << 1) | (now >> 1));
        }
        for (int l = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); l < NP; l += nt >> 6) {
            if (!((taken >> l) & 1)) continue;
            const float sl = score[l];
            int place = 0;
#pragma unroll
            for (int i = 0; i < 2; ++i)
                place += __popcll(__ballot(s[i] > sl || (s[i] == sl && lane + 64 * i < l)) & (unsigned long long)(taken >> (64 * i)));
            if (place < n_select && lane == 0) out_pairs[place] = l;
        }
        if (threadIdx.x < 64) {
            const int all = __popcll((unsigned long long)taken) + __popcll((unsigned long long)(taken >> 64)), cnt = min(all, n_select);
            if (lane == 0) *out_count = cnt;
            for (int i = cnt + lane; i < n_select; i += 64) out_pairs[i] = -1;
        }
        __syncthreads();   // (the scores' place may be used again)
        return;
    }

    int32_t *order = static_cast<int32_t *>(scratch);            // [NP] candidate at each rank
    uint8_t *cand = reinterpret_cast<uint8_t *>(order + NP);     // [NP]
    uint8_t *used = cand + NP;                                   // [n_layers]
    for (int l = threadIdx.x; l < NP; l += nt) {
        cand[l] = (!el || (el[l] && el[l + 1])) ? 1 : 0;
        order[l] = -1;
    }
    for (int l = threadIdx.x; l < n_layers; l += nt) used[l] = 0;
    __syncthreads();

    for (int l = threadIdx.x >> 6; l < NP; l += nt >> 6) {   // (uniform over the wave)
        const float s = score[l];
        if (!cand[l] || s != s) continue;
        int rank = 0;
        for (int j0 = 0; j0 < NP; j0 += 64) {
            const int j = j0 + (threadIdx.x & 63);
            const float sj = score[min(j, NP - 1)];
            // j precedes l unless l's score is strictly higher, or equal with l first
            const bool before = j < NP && cand[min(j, NP - 1)] && sj == sj && (sj > s || (!(sj < s) && j < l));
            rank += __popcll(__ballot(before));
        }
        if ((threadIdx.x & 63) == 0) order[rank] = l;
    }
    __syncthreads();

    if (threadIdx.x == 0) {
        int cnt = 0;
        for (int i = 0; i < NP && cnt < n_select; ++i) {
            const int l = order[i];
            if (l < 0) break;
            if (used[l] || used[l + 1]) continue;
            used[l] = used[l + 1] = 1;
            out_pairs[cnt++] = l;
        }
        *out_count = cnt;
        for (int i = cnt; i < n_select; ++i) out_pairs[i] = -1;
    }
    __syncthreads();   // the scratch may be reused
}

}  // namespace krul
