// Exact top-k of one importance row by one 1024-thread workgroup, the row's
// keys in registers: the selection of short rows (row.hip, and the pool pass
// in bkp.hip).  Thread t holds TPT consecutive tokens, TPT * t onward, so that
// one block scan gives positions in token order.
#pragma once

#include "hill_device.h"
#include "hill_internal.h"

namespace hill {

constexpr int kRowThreads = 1024;
constexpr int kRowWaves = kRowThreads / 64;
constexpr int kRowBins = kHistBins;   // the radix digits are 12 (as elsewhere: the streamed bound) + 10 + 10 bits

struct RowLds {
    alignas(16) uint32_t bins[kRowBins];
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

// The bin that holds the need-th largest counted key, with NB bins in L.bins
// (NB / kRowThreads per thread, thread t from the top): L.res[0] = bin,
// L.res[1] = keys still needed from it, L.res[2] = keys in it.  Ends with a
// barrier.
template <int NB>
__device__ __forceinline__ void row_find_bin(RowLds& L, uint32_t need, uint32_t* wave)
{
    constexpr int PER = NB / kRowThreads;
    static_assert(PER == 1 || PER == 4, "one word or one 16-byte load per thread");
    const int t = kRowThreads - 1 - (int)threadIdx.x;   // this thread's bins are PER * t onward
    uint32_t c[PER], sum = 0u, total;
    if constexpr (PER == 4) {
        const uint4 v = reinterpret_cast<const uint4*>(L.bins)[t];
        c[0] = v.x;
        c[1] = v.y;
        c[2] = v.z;
        c[3] = v.w;
    } else {
        c[0] = L.bins[t];
    }
#pragma unroll
    for (int i = 0; i < PER; ++i) sum += c[i];
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
// sel[e] for token TPT * t + e; `before`: tokens selected in the row before
// this thread's.  ok[e]: the token exists (j < n).  Every thread of the
// workgroup calls it.
template <int TPT>
__device__ __forceinline__ RowBound row_select(const uint32_t (&key)[TPT], const bool (&ok)[TPT], uint32_t k, RowLds& L,
                                               bool (&sel)[TPT], uint32_t& before)
{
    const int tid = threadIdx.x;
    uint32_t total;
    reinterpret_cast<uint4*>(L.bins)[tid] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
#pragma unroll
    for (int e = 0; e < TPT; ++e)
        if (ok[e]) atomicAdd(&L.bins[key[e] >> 20], 1u);
    __syncthreads();
    row_find_bin<kRowBins>(L, k, L.wave[0]);
    const RowBound bound{L.res[0], L.res[1], L.res[2]};
    uint32_t prefix = bound.b1, need = bound.need1;
    int shift = 20;
    bool all_eq = need == bound.in1;
#pragma unroll
    for (int round = 1; round < 3; ++round) {
        if (all_eq) continue;   // block-uniform
        L.bins[tid] = 0u;       // the last reads of the bins and of res lie before row_find_bin's barriers
        __syncthreads();
#pragma unroll
        for (int e = 0; e < TPT; ++e)
            if (ok[e] && (key[e] >> shift) == prefix) atomicAdd(&L.bins[(key[e] >> (shift - 10)) & 1023u], 1u);
        __syncthreads();
        row_find_bin<kRowThreads>(L, need, L.wave[round & 1]);
        prefix = (prefix << 10) | L.res[0];
        shift -= 10;
        need = L.res[1];
        all_eq = need == L.res[2];
    }
    // keys above the threshold's prefix, and of those equal to it all or, when
    // the budget cuts through them, the first `need` in token order
    uint32_t neq = 0u;
    bool eq[TPT];
#pragma unroll
    for (int e = 0; e < TPT; ++e) {
        const uint32_t kd = key[e] >> shift;
        sel[e] = ok[e] && kd > prefix;
        eq[e] = ok[e] && kd == prefix;
        neq += eq[e] ? 1u : 0u;
    }
    uint32_t rank = 0u;
    if (!all_eq) rank = row_scan(neq, L.wave[1], &total);   // the last round's scan used wave[0]
    uint32_t nsel = 0u;
#pragma unroll
    for (int e = 0; e < TPT; ++e) {
        sel[e] = sel[e] || (eq[e] && (all_eq || rank < need));
        rank += eq[e] ? 1u : 0u;
        nsel += sel[e] ? 1u : 0u;
    }
    __syncthreads();   // earlier reads of the wave totals are done
    before = row_scan(nsel, L.wave[0], &total);
    return bound;
}

// This thread's TPT floats of a row (16-byte aligned, its stride a multiple of
// 4 and at least n: a group of four that begins below n lies inside it);
// groups past the row's end read its last one.
template <int TPT>
__device__ __forceinline__ void row_load(const float* srow, int n, float (&x)[TPT])
{
    const int j = TPT * (int)threadIdx.x;
    if constexpr (TPT == 2) {
        const float2 v = *reinterpret_cast<const float2*>(srow + min(j, (n - 1) & ~1));
        x[0] = v.x;
        x[1] = v.y;
    } else {
#pragma unroll
        for (int i = 0; i < TPT / 4; ++i) {
            const float4 v = *reinterpret_cast<const float4*>(srow + min(j + 4 * i, (n - 1) & ~3));
            x[4 * i] = v.x;
            x[4 * i + 1] = v.y;
            x[4 * i + 2] = v.z;
            x[4 * i + 3] = v.w;
        }
    }
}

template <int TPT>
__device__ __forceinline__ void row_keys(const float (&x)[TPT], int n, int lo, int hi, uint32_t (&key)[TPT], bool (&ok)[TPT])
{
    const int j = TPT * (int)threadIdx.x;
#pragma unroll
    for (int e = 0; e < TPT; ++e) {
        ok[e] = j + e < n;
        key[e] = ok[e] ? select_key(x[e], j + e, lo, hi) : 0u;
    }
}

}  // namespace hill
