// Device helpers for keeping the CAND smallest (score, index) pairs, shared
// by the dense and the sparse indexing kernels: per-thread sorted lists in
// registers (CAND 16, 32) and a wave-wide list of 64.  Order: ascending
// score, equal scores by ascending index.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

namespace ar {

__device__ __forceinline__ bool pair_less(float as, int ai, float bs, int bi)
{
    return as < bs || (as == bs && ai < bi);
}

// Sorted ascending by (score, index); insertion keeps the CAND smallest.
template <int CAND>
struct TopList {
    float s[CAND];
    int i[CAND];
    __device__ __forceinline__ void init()
    {
#pragma unroll
        for (int j = 0; j < CAND; ++j) {
            s[j] = INFINITY;
            i[j] = 0x7fffffff;
        }
    }
    __device__ __forceinline__ void insert(float cs, int ci)
    {
        if (!pair_less(cs, ci, s[CAND - 1], i[CAND - 1])) return;
#pragma unroll
        for (int j = 0; j < CAND; ++j) {
            const bool lt = pair_less(cs, ci, s[j], i[j]);
            const float ts = lt ? s[j] : cs;
            const int ti = lt ? i[j] : ci;
            s[j] = lt ? cs : s[j];
            i[j] = lt ? ci : i[j];
            cs = ts;
            ci = ti;
        }
    }
    // entry `head` (INFINITY past the end), selected without dynamic indexing
    __device__ __forceinline__ void at(int head, float &hs, int &hi) const
    {
        hs = INFINITY;
        hi = 0x7fffffff;
#pragma unroll
        for (int q = 0; q < CAND; ++q)
            if (q == head) {
                hs = s[q];
                hi = i[q];
            }
    }
};

// The smaller of this lane's pair and that of the lane a DPP pattern names.
template <int CTRL> __device__ __forceinline__ void min_pair_dpp(float &bs, int &bi)
{
    const float os = __int_as_float(
        __builtin_amdgcn_update_dpp(__float_as_int(bs), __float_as_int(bs), CTRL, 0xF, 0xF, false));
    const int oi = __builtin_amdgcn_update_dpp(bi, bi, CTRL, 0xF, 0xF, false);
    if (pair_less(os, oi, bs, bi)) {
        bs = os;
        bi = oi;
    }
}

// Wave-wide minimum of (score, index) pairs, the same on every lane: within
// rows of 16 lanes by DPP (xor 1, xor 2, half-row and row mirrors), then over
// the four rows by lane reads.  The chain is what a selection of 16 waits for:
// k_select of 16 rows of 1024 scores takes 13.4 us, with twelve LDS
// permutations per minimum 21.2.
__device__ __forceinline__ void wave_min_pair(float &bs, int &bi)
{
    min_pair_dpp<0xB1>(bs, bi);
    min_pair_dpp<0x4E>(bs, bi);
    min_pair_dpp<0x141>(bs, bi);
    min_pair_dpp<0x140>(bs, bi);
    const int s = __float_as_int(bs), i = bi;
    bs = __int_as_float(__builtin_amdgcn_readlane(s, 0));
    bi = __builtin_amdgcn_readlane(i, 0);
#pragma unroll
    for (int l = 16; l < 64; l += 16) {
        const float os = __int_as_float(__builtin_amdgcn_readlane(s, l));
        const int oi = __builtin_amdgcn_readlane(i, l);
        if (pair_less(os, oi, bs, bi)) {
            bs = os;
            bi = oi;
        }
    }
}

// The wave's CAND smallest pairs over every lane's sorted list t (each list
// holds at most CAND valid entries): CAND rounds of an argmin over the list
// heads.  Round j's result is passed to emit(j, score, index) on every lane.
template <int CAND, int LEN, typename Emit>
__device__ __forceinline__ void wave_select(const TopList<LEN> &t, Emit emit)
{
    int head = 0;
    for (int j = 0; j < CAND; ++j) {
        float hs;
        int hi;
        t.at(head, hs, hi);
        float bs = hs;
        int bi = hi;
        wave_min_pair(bs, bi);
        if (hs == bs && hi == bi && head < LEN) ++head;
        emit(j, bs, bi);
    }
}

// The k first of CAND <= 64 entries (ds, di) in LDS by (score, index), by one
// wavefront: each lane counts the entries before its own (equal ones, which
// hold no candidate, in place).  Index 0x7fffffff stands for none and is
// written as -1.
template <int CAND>
__device__ __forceinline__ void rank_candidates(float *ds, int *di, int lane, int k, int32_t *__restrict__ top_idx,
                                                float *__restrict__ top_score)
{
    const float ms = lane < CAND ? ds[lane] : 0.0f;
    const int mi = lane < CAND ? di[lane] : 0;
    if (!__any(ms != ms)) {
        int rank = 0;
#pragma unroll
        for (int j = 0; j < CAND; ++j) {
            const float s = ds[j];
            const int i = di[j];
            rank += pair_less(s, i, ms, mi) || (s == ms && i == mi && j < lane) ? 1 : 0;
        }
        if (lane < CAND && rank < k) {
            top_idx[rank] = mi == 0x7fffffff ? -1 : mi;
            top_score[rank] = ms;
        }
    } else if (lane == 0) {
        // a score that is not a number: an insertion sort, whose order is defined there too
        for (int a = 1; a < CAND; ++a) {
            const float vs = ds[a];
            const int vi = di[a];
            int b = a - 1;
            while (b >= 0 && pair_less(vs, vi, ds[b], di[b])) {
                ds[b + 1] = ds[b];
                di[b + 1] = di[b];
                --b;
            }
            ds[b + 1] = vs;
            di[b + 1] = vi;
        }
        for (int j = 0; j < k; ++j) {
            top_idx[j] = di[j] == 0x7fffffff ? -1 : di[j];
            top_score[j] = ds[j];
        }
    }
}

// ---------------------------------------------------------------------------
// Wave-wide sorted list of 64 (score, index) pairs: lane j holds the j-th
// smallest.  A batch of 64 new pairs (one per lane) enters by a bitonic
// merge: the batch is sorted ascending across the lanes, reversed and
// combined lane by lane with the list by min (which leaves the 64 smallest
// of the 128 as a bitonic sequence), then sorted by the six half-cleaner
// steps.  Keys (score, index) are distinct except for the empty-slot
// sentinel, so the result is the exact 64 smallest whatever the order of
// arrival.

// Compare-exchange with the lane at distance `mask`: keep the smaller pair
// if keep_min, else the larger.
__device__ __forceinline__ void wave_cmpx(float &s, int &i, int mask, bool keep_min)
{
    const float os = __shfl_xor(s, mask);
    const int oi = __shfl_xor(i, mask);
    const bool other_less = pair_less(os, oi, s, i);
    if (keep_min == other_less) {
        s = os;
        i = oi;
    }
}

// Sort one pair per lane ascending across the 64 lanes.
__device__ __forceinline__ void wave_sort64(float &s, int &i, int lane)
{
#pragma unroll
    for (int k = 2; k <= 64; k <<= 1)
#pragma unroll
        for (int j = k >> 1; j > 0; j >>= 1) wave_cmpx(s, i, j, ((lane & j) == 0) == ((lane & k) == 0));
}

// Merge the batch (bs, bi) into the sorted list (ls, li).  Lanes whose pair
// does not beat the list's last entry are dropped first; when none does,
// the list is unchanged and the merge is skipped.
__device__ __forceinline__ void wave_merge64(float &ls, int &li, float bs, int bi, int lane)
{
    const float ts = __shfl(ls, 63);
    const int ti = __shfl(li, 63);
    const bool enters = pair_less(bs, bi, ts, ti);
    if (!__any(enters)) return;
    if (!enters) {
        bs = INFINITY;
        bi = 0x7fffffff;
    }
    wave_sort64(bs, bi, lane);
    const float rs = __shfl(bs, 63 - lane);
    const int ri = __shfl(bi, 63 - lane);
    if (pair_less(rs, ri, ls, li)) {
        ls = rs;
        li = ri;
    }
#pragma unroll
    for (int j = 32; j > 0; j >>= 1) wave_cmpx(ls, li, j, (lane & j) == 0);
}

}  // namespace ar
