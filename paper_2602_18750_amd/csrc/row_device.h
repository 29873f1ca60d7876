// Exact top-k of one importance row by one 1024-thread workgroup, the row's
// keys in registers: the selection of short rows (row.hip, and the pool pass
// in bkp.hip).  Wave w holds 64 * TPT consecutive tokens in groups of GS per
// lane: element e of lane l is token row_token<TPT, GS>(e), so that the lanes
// of a load read consecutive groups (TPT consecutive tokens per thread read
// each line TPT / 4 times: row_topk at 2 x 16K 19.8 us).
#pragma once

#include "hill_device.h"
#include "hill_internal.h"

namespace hill {

constexpr int kRowThreads = 1024;
constexpr int kRowWaves = kRowThreads / 64;
// The digits are counted in LDS in COPIES interleaved copies, lane l into copy
// l % COPIES: S values cluster in a few dozen bins, and lanes of one
// instruction that add to the same word take their turns.
constexpr int row_bin_words(int copies) { return kHistBins * copies; }

constexpr int kRowBins = kHistBins;   // the radix digits are 12 (as elsewhere: the streamed bound) + 10 + 10 bits

template <int TPT, int GS>
__device__ __forceinline__ int row_token(int e)
{
    static_assert(TPT % GS == 0, "whole groups");
    return ((int)threadIdx.x >> 6) * 64 * TPT + (e / GS) * 64 * GS + ((int)threadIdx.x & 63) * GS + e % GS;
}

// Positions in token order: c[i] counts of this lane's groups -> how many are
// counted in the row before each of them.  One barrier; the wave totals stay
// in wave[], which must not be rewritten before the next.
template <int NG>
__device__ __forceinline__ void row_positions(const uint32_t (&c)[NG], uint32_t* wave, uint32_t (&pos)[NG])
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint32_t run = 0u;
#pragma unroll
    for (int i = 0; i < NG; ++i) {
        const uint32_t inc = wave_incl_scan(c[i]);
        pos[i] = run + inc - c[i];
        run += (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
    }
    if (lane == 0) wave[w] = run;
    __syncthreads();
    const uint32_t t = lane < kRowWaves ? wave[lane] : 0u;
    const uint32_t ti = wave_incl_scan(t);
    const uint32_t base = (uint32_t)__shfl((int)(ti - t), w, 64);
#pragma unroll
    for (int i = 0; i < NG; ++i) pos[i] += base;
}

struct RowLds {
    uint32_t wave[2][kRowWaves];   // wave totals of the scans, used alternately
    uint32_t res[4];
};

// Exclusive prefix sum over the workgroup with one barrier; the wave totals
// stay in wave[], which must not be rewritten before the next barrier.
__device__ __forceinline__ uint32_t row_scan(uint32_t v, uint32_t* wave, uint32_t* total)
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint32_t inc = wave_incl_scan(v);
    if (lane == 63) wave[w] = inc;
    __syncthreads();
    const uint32_t t = lane < kRowWaves ? wave[lane] : 0u;   // every wave sums the totals by itself
    const uint32_t ti = wave_incl_scan(t);
    *total = (uint32_t)__builtin_amdgcn_readlane((int)ti, kRowWaves - 1);
    const uint32_t base = (uint32_t)__shfl((int)(ti - t), w, 64);
    return base + inc - v;
}

// The bin that holds the need-th largest counted key, with NB bins of COPIES
// words each (thread t sums NB / kRowThreads of them, from the top):
// L.res[0] = bin, L.res[1] = keys still needed from it, L.res[2] = keys in it.
// Ends with a barrier.
template <int NB, int COPIES>
__device__ __forceinline__ void row_find_bin(const uint32_t* bins, RowLds& L, uint32_t need, uint32_t* wave)
{
    constexpr int PER = NB / kRowThreads;
    static_assert(COPIES % 4 == 0, "16-byte loads");
    const int t = kRowThreads - 1 - (int)threadIdx.x;   // this thread's bins are PER * t onward
    uint32_t c[PER], sum = 0u, total;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        c[i] = 0u;
#pragma unroll
        for (int q = 0; q < COPIES / 4; ++q) {
            const uint4 v = reinterpret_cast<const uint4*>(bins)[(PER * t + i) * (COPIES / 4) + q];
            c[i] += (v.x + v.y) + (v.z + v.w);
        }
        sum += c[i];
    }
    const uint32_t above = row_scan(sum, wave, &total);
    if (above < need && above + sum >= need) {
        uint32_t a = above;
        bool found = false;
#pragma unroll
        for (int i = PER - 1; i >= 0; --i) {
            if (!found && a + c[i] >= need) {
                L.res[0] = (uint32_t)(PER * t + i);
                L.res[1] = need - a;
                L.res[2] = c[i];
                found = true;
            }
            a += c[i];
        }
    }
    __syncthreads();
}

// First digit of the row's threshold: its bin, keys needed from it, keys in it.
struct RowBound {
    uint32_t b1, need1, in1;
};

// The keys of this thread's tokens to select, k of the row's n (1 <= k <= n):
// sel[e] for token row_token(e); before[i]: tokens selected in the row before
// this lane's group i.  ok[e]: the token exists (j < n).  bins: row_bin_words(COPIES)
// words of LDS, 16-byte aligned, free again when it returns.  Every thread of
// the workgroup calls it.
template <int TPT, int GS, int COPIES>
__device__ __forceinline__ RowBound row_select(const uint32_t (&key)[TPT], const bool (&ok)[TPT], uint32_t k, RowLds& L,
                                               uint32_t* bins, bool (&sel)[TPT], uint32_t (&before)[TPT / GS])
{
    const int tid = threadIdx.x;
    const uint32_t copy = tid & (COPIES - 1);
#pragma unroll
    for (int i = 0; i < kRowBins * COPIES / 4 / kRowThreads; ++i)
        reinterpret_cast<uint4*>(bins)[i * kRowThreads + tid] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
#pragma unroll
    for (int e = 0; e < TPT; ++e)
        if (ok[e]) atomicAdd(&bins[(key[e] >> 20) * COPIES + copy], 1u);
    __syncthreads();
    row_find_bin<kRowBins, COPIES>(bins, L, k, L.wave[0]);
    const RowBound bound{L.res[0], L.res[1], L.res[2]};
    uint32_t prefix = bound.b1, need = bound.need1;
    int shift = 20;
    bool all_eq = need == bound.in1;
#pragma unroll
    for (int round = 1; round < 3; ++round) {
        if (all_eq) continue;   // block-uniform
        // the last reads of the bins lie before row_find_bin's barriers
#pragma unroll
        for (int i = 0; i < COPIES / 4; ++i)
            reinterpret_cast<uint4*>(bins)[i * kRowThreads + tid] = make_uint4(0u, 0u, 0u, 0u);
        __syncthreads();
#pragma unroll
        for (int e = 0; e < TPT; ++e)
            if (ok[e] && (key[e] >> shift) == prefix)
                atomicAdd(&bins[((key[e] >> (shift - 10)) & 1023u) * COPIES + copy], 1u);
        __syncthreads();
        row_find_bin<kRowThreads, COPIES>(bins, L, need, L.wave[round & 1]);
        prefix = (prefix << 10) | L.res[0];
        shift -= 10;
        need = L.res[1];
        all_eq = need == L.res[2];
    }
    // keys above the threshold's prefix, and of those equal to it all or, when
    // the budget cuts through them, the first `need` in token order
    constexpr int NG = TPT / GS;
    uint32_t cnt[NG];
    bool eq[TPT];
#pragma unroll
    for (int i = 0; i < NG; ++i) cnt[i] = 0u;
#pragma unroll
    for (int e = 0; e < TPT; ++e) {
        const uint32_t kd = key[e] >> shift;
        sel[e] = ok[e] && kd > prefix;
        eq[e] = ok[e] && kd == prefix;
        cnt[e / GS] += eq[e] ? 1u : 0u;
    }
    uint32_t rank[NG];
#pragma unroll
    for (int i = 0; i < NG; ++i) rank[i] = 0u;
    if (!all_eq) row_positions<NG>(cnt, L.wave[1], rank);   // the last round's scan used wave[0]
#pragma unroll
    for (int i = 0; i < NG; ++i) cnt[i] = 0u;
#pragma unroll
    for (int e = 0; e < TPT; ++e) {
        sel[e] = sel[e] || (eq[e] && (all_eq || rank[e / GS] < need));
        rank[e / GS] += eq[e] ? 1u : 0u;
        cnt[e / GS] += sel[e] ? 1u : 0u;
    }
    __syncthreads();   // earlier reads of the wave totals are done
    row_positions<NG>(cnt, L.wave[0], before);
    return bound;
}

// This thread's floats of a row (16-byte aligned, its stride a multiple of 4
// and at least n: a group of four that begins below n lies inside it); groups
// past the row's end read its last one.  GS is 4, or 2 where TPT is.
template <int TPT, int GS>
__device__ __forceinline__ void row_load(const float* srow, int n, float (&x)[TPT])
{
    static_assert(GS == 4 || (GS == 2 && TPT == 2), "16- or 8-byte groups");
    if constexpr (GS == 2) {
        const float2 v = *reinterpret_cast<const float2*>(srow + min(row_token<TPT, GS>(0), (n - 1) & ~1));
        x[0] = v.x;
        x[1] = v.y;
    } else {
#pragma unroll
        for (int i = 0; i < TPT / 4; ++i) {
            const float4 v = *reinterpret_cast<const float4*>(srow + min(row_token<TPT, GS>(4 * i), (n - 1) & ~3));
            x[4 * i] = v.x;
            x[4 * i + 1] = v.y;
            x[4 * i + 2] = v.z;
            x[4 * i + 3] = v.w;
        }
    }
}

template <int TPT, int GS>
__device__ __forceinline__ void row_keys(const float (&x)[TPT], int n, int lo, int hi, uint32_t (&key)[TPT], bool (&ok)[TPT])
{
#pragma unroll
    for (int e = 0; e < TPT; ++e) {
        const int j = row_token<TPT, GS>(e);
        ok[e] = j < n;
        key[e] = ok[e] ? select_key(x[e], j, lo, hi) : 0u;
    }
}

}  // namespace hill
