// Exact top-k token selection on gfx950 (Sec. 3.1 top-alpha; Sec. 4.2 global
// top-alpha indices) as a radix select on order-preserving 32-bit keys, split
// over 512-token chunks of each importance row so that every step runs on
// many CUs -- the GPU form of the paper's chunked evaluation whose per-chunk
// results are merged into one global threshold (Sec. 4.2, HIE).
//
//  topk_hist    first-digit (bits 31..20) histogram of every row; in hill_step
//               the importance update counts it as it writes S.
//  topk_refine  per chunk: finds the first-digit bin holding the k-th key,
//               histograms the second digit (bits 19..8) of the chunk's keys
//               inside that bin and keeps those keys in a compact candidate
//               list.
//  topk_emit    per chunk: resolves the exact threshold key from the row's
//               second-digit histogram (and, when keys still tie on 24 bits,
//               the third digit from the candidate lists), marks the chunk's
//               selected tokens -- every key above the threshold plus, among
//               keys equal to it, the lowest token indices that fit the
//               budget -- and stores them in token order with their count.
//               With attention, the workgroup then attends over the chunk's
//               selected tokens for one or more KV heads (fused gather +
//               softmax over the list, attn_device.h; the logits are the
//               scan's own when it read the 16-bit keys, so only V rows are
//               gathered) and writes one partial per query head.  The
//               streamed variant takes the first two digits from the
//               update's histograms (the second from its window above the
//               previous step's threshold) and, when those do not settle the
//               threshold, walks the update's candidate pairs instead of
//               refine's lists; it writes the bound for the next step.
//  topk_write   places each chunk's list at its ascending-order offset (the
//               counts of the chunks before it) in the output; in hill_step
//               this runs inside merge_write, with the merge of the attention
//               partials.
//
// Every histogram is a 12-bit digit whose top 6 bits are also counted, so the
// bin of the k-th key is found in registers: every wave scans the 64 coarse
// bins (one per lane), and the wave that holds the 64 fine bins of the chosen
// coarse bin finishes.  Cross-chunk results always pass through a kernel
// boundary: on this multi-XCD part an agent-scope fence per workgroup (needed
// by a last-workgroup-done merge) costs far more than a launch.  The
// selection is exactly the k largest S with ties to the lower index: keys are
// integers, so no floating-point rounding takes part.
#include <hip/hip_ext.h>

#include "topk_device.h"

namespace hill {

namespace {

__global__ __launch_bounds__(256) void topk_hist_kernel(const float* __restrict__ s, int64_t s_sb, int64_t s_sr,
                                                        int R, int n, int pin_lo, int pin_hi,
                                                        uint32_t* __restrict__ hist)
{
    __shared__ uint32_t lds_hist[kHistRow];
    __shared__ uint32_t list[kHistRow];
    __shared__ uint32_t nlist;
    const int row = blockIdx.y;
    const int b = row / R, r = row % R;
    for (int i = threadIdx.x; i < kHistRow; i += 256) lds_hist[i] = 0u;
    if (threadIdx.x == 0) nlist = 0u;
    __syncthreads();
    const float* srow = s + (int64_t)b * s_sb + (int64_t)r * s_sr;
    constexpr int kPer = kHistChunk / 256;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        const int j = blockIdx.x * kHistChunk + i * 256 + threadIdx.x;
        if (j < n) {
            const uint32_t kk = select_key(srow[j], j, pin_lo, pin_hi);
            hist_add(lds_hist, list, &nlist, kk >> (32 - kHistBits));
            hist_add(lds_hist, list, &nlist, kHistBins + (kk >> 26));
        }
    }
    __syncthreads();
    hist_flush(lds_hist, list, nlist, hist + (int64_t)row * kHistRow);
}

// find_digit over a histogram in `parts` copies of a row: the coarse bins of
// all copies in one round trip, then the 64 fine bins of the chosen coarse bin
// in another (loading every copy whole would cost more than that round trip).
// Every wave finds the same; the first publishes.
__device__ __forceinline__ void find_digit_parts(const uint32_t* h, int parts, uint32_t need, uint32_t* res)
{
    const int lane = threadIdx.x & 63;
    auto sum = [&](int at) {
        uint32_t v[kMaxHistParts], t = 0u;
#pragma unroll
        for (int p = 0; p < kMaxHistParts; ++p) v[p] = h[(int64_t)min(p, parts - 1) * kHistRow + at + lane];
#pragma unroll
        for (int p = 0; p < kMaxHistParts; ++p) t += p < parts ? v[p] : 0u;
        return t;
    };
    int C, L;
    uint32_t above_c, above_f;
    wave_find_bin(sum(kHistBins), need, C, above_c);
    const uint32_t v = sum(64 * C);
    wave_find_bin(v, need - above_c, L, above_f);
    const uint32_t in_bin = __shfl(v, L, 64);
    if (threadIdx.x == 0) {
        res[0] = (uint32_t)(64 * C + L);
        res[1] = need - above_c - above_f;
        res[2] = in_bin;
    }
}

__global__ __launch_bounds__(kThreads) void topk_refine_kernel(RefineArgs a, int parts)
{
    __shared__ uint32_t hist[kHistRow];
    __shared__ uint32_t list[2 * kSelChunk];
    __shared__ uint32_t res[3];
    __shared__ uint32_t n_cand, nlist;

    const int tid = threadIdx.x, lane = tid & 63;
    const int c = blockIdx.x, row = blockIdx.y;
    const float* srow = row_ptr(a, row);

    // the chunk's S and the row's first-digit histogram are loaded together
    const float2 sx = load_s_pair(srow, c, a.n);
    const uint32_t* h1p = a.hist1 + (int64_t)row * parts * kHistRow;
    DigitHist h1;
    if (parts == 1) load_digit_hist(h1p, h1);
    uint32_t key[kPerThread];
    bool ok[kPerThread];
    keys_of(sx, c, a.n, a.pin_lo, a.pin_hi, key, ok);
    for (int i = tid; i < kHistRow; i += kThreads) hist[i] = 0u;
    if (tid == 0) n_cand = nlist = 0u;
    // first digit: the bin of the k-th key
    if (parts == 1) find_digit(h1, (uint32_t)a.k, res);
    else find_digit_parts(h1p, parts, (uint32_t)a.k, res);
    __syncthreads();
    const uint32_t b1 = res[0] & (kHistBins - 1);
    const uint32_t need1 = res[1];
    const uint32_t in1 = res[2];
    const bool refine = need1 < in1;
    if (c == 0 && tid == 0) a.state[row] = make_uint4(b1, need1, in1, 0u);

    // keys inside the bin are the candidates: their second digit is
    // histogrammed and they are appended (wave-compacted) to the chunk's
    // candidate list, whose order does not matter
    uint32_t* cand = a.cand_key + (int64_t)row * a.n + (int64_t)c * kSelChunk;
#pragma unroll
    for (int e = 0; e < kPerThread; ++e) {
        const bool is_c = ok[e] && (key[e] >> 20) == b1;
        if (is_c && refine) {
            hist_add(hist, list, &nlist, (key[e] >> 8) & (kHistBins - 1));
            hist_add(hist, list, &nlist, kHistBins + ((key[e] >> 14) & (kCoarseBins - 1)));
        }
        const uint64_t mask = __ballot(is_c);
        if (mask) {
            const int leader = __ffsll((unsigned long long)mask) - 1;
            uint32_t base = 0;
            if (lane == leader) base = atomicAdd(&n_cand, (uint32_t)__popcll(mask));
            base = __shfl(base, leader, 64);
            if (is_c) cand[base + __popcll(mask & ((1ull << lane) - 1ull))] = key[e];
        }
    }
    __syncthreads();
    if (refine) hist_flush(hist, list, nlist, a.hist2 + (int64_t)row * kHistRow);
    if (tid == 0) a.cand_n[(int64_t)row * a.nchunks + c] = n_cand;
}

// Copies the list of chunk c of a row to the output at its ascending-order
// offset (the selected counts of the chunks before it).  Every load is issued
// before the first wait: the counts before c, this chunk's count and its list
// entries (two per thread, at most kSelChunk; positions past the chunk's
// tokens are clamped into it and never stored).
__device__ __forceinline__ void write_chunk(const RefineArgs& r, int row, int c, int32_t* idx, float* val,
                                            uint32_t* red)
{
    const int tid = threadIdx.x, lane = tid & 63;
    const uint32_t* sn = r.sel_n + (int64_t)row * r.nchunks;
    const int32_t* list = r.sel_list + (int64_t)row * r.n + (int64_t)c * kSelChunk;
    const int last = min(kSelChunk, r.n - c * kSelChunk) - 1;   // the chunk's last slot
    const int32_t e0 = list[min(tid, last)];
    const int32_t e1 = list[min(tid + kThreads, last)];
    const uint32_t m = sn[c];
    uint32_t before = 0;
    for (int cc = tid; cc < c; cc += kThreads) before += sn[cc];
    before = wave_sum_u32(before);
    if (lane == 0) red[tid >> 6] = before;
    __syncthreads();
    uint32_t base = 0;
    for (int i = 0; i < kThreads / 64; ++i) base += red[i];
    const float* srow = row_ptr(r, row);
    static_assert(kSelChunk == 2 * kThreads, "two list entries per thread");
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const uint32_t i = (uint32_t)(tid + e * kThreads);
        const uint32_t p = base + i;
        if (i < m && p < (uint32_t)r.k) {
            const int32_t j = e == 0 ? e0 : e1;
            idx[(int64_t)row * r.k + p] = j;
            if (val) val[(int64_t)row * r.k + p] = srow[j];
        }
    }
}

__global__ __launch_bounds__(kThreads) void topk_write_kernel(RefineArgs r, int32_t* idx, float* val)
{
    __shared__ uint32_t red[kThreads / 64];
    write_chunk(r, blockIdx.y, blockIdx.x, idx, val, red);
}

// hill_step's last kernel: workgroups [0, B*Hq*kMergeSlices) merge the chunk
// partials of one slice of kHeadDim / kMergeSlices output dimensions of one
// query head each (a slice's loads are one 128-byte line per slot; more,
// shorter workgroups finish sooner than one per head); the rest copy one
// chunk list each into the index output.
constexpr int kMergeSlices = 4;

__global__ __launch_bounds__(kThreads) void merge_write_kernel(RefineArgs r, AttnArgs at, int32_t* idx)
{
    constexpr int DS = kHeadDim / kMergeSlices;
    __shared__ float red[kThreads / 64 + kThreads / DS];
    __shared__ float osum[kThreads];
    __shared__ uint32_t ured[kThreads / 64];
    const int nmerge = at.B * at.Hq * kMergeSlices;
    if ((int)blockIdx.x < nmerge) {
        const int bh = blockIdx.x / kMergeSlices, sl = blockIdx.x % kMergeSlices;
        merge_head<kThreads, DS>(at, bh / at.Hq, bh % at.Hq, sl * DS, r.nchunks, red, osum);
    } else {
        const int t = blockIdx.x - nmerge;
        write_chunk(r, t / r.nchunks, t % r.nchunks, idx, nullptr, ured);
    }
}

}  // namespace

hipError_t launch_topk_hist(const float* s, int64_t s_sb, int64_t s_sr, int B, int R, int n, int pin_lo, int pin_hi,
                            uint32_t* hist, hipStream_t st, Stamp ts)
{
    dim3 grid((n + kHistChunk - 1) / kHistChunk, B * R);
    hipExtLaunchKernelGGL(topk_hist_kernel, grid, dim3(256), 0, st, ts.start, ts.stop, 0, s, s_sb, s_sr, R, n, pin_lo,
                          pin_hi, hist);
    return hipGetLastError();
}

hipError_t launch_topk_refine(const RefineArgs& a, int rows, int parts, hipStream_t st, Stamp ts)
{
    dim3 grid(a.nchunks, rows);
    hipExtLaunchKernelGGL(topk_refine_kernel, grid, dim3(kThreads), 0, st, ts.start, ts.stop, 0, a, parts);
    return hipGetLastError();
}

hipError_t launch_topk_emit_indices(const RefineArgs& r, int rows, int32_t* idx, float* val, hipStream_t st, Stamp ts)
{
    dim3 grid(r.nchunks, rows);
    hipExtLaunchKernelGGL((topk_emit_kernel<0, 1, false>), grid, dim3(kThreads), 0, st, ts.start, nullptr, 0, r,
                          AttnArgs{});
    hipExtLaunchKernelGGL(topk_write_kernel, grid, dim3(kThreads), 0, st, nullptr, ts.stop, 0, r, idx, val);
    return hipGetLastError();
}

hipError_t launch_topk_emit_lists(const RefineArgs& r, int rows, hipStream_t st)
{
    hipLaunchKernelGGL((topk_emit_kernel<0, 1, false>), dim3(r.nchunks, rows), dim3(kThreads), 0, st, r, AttnArgs{});
    return hipGetLastError();
}

hipError_t launch_topk_emit_attn_stream(const RefineArgs& r, const AttnArgs& at, int dtype, hipStream_t st, Stamp ts)
{
    return at.logits ? launch_emit_logits(r, at, dtype, true, st, ts) : launch_emit_gather(r, at, dtype, true, st, ts);
}

hipError_t launch_topk_emit_attn(const RefineArgs& r, const AttnArgs& at, int dtype, hipStream_t st, Stamp ts)
{
    return at.logits ? launch_emit_logits(r, at, dtype, false, st, ts) : launch_emit_gather(r, at, dtype, false, st, ts);
}

hipError_t launch_merge_write(const RefineArgs& r, const AttnArgs& at, int32_t* idx, int rows, hipStream_t st,
                              Stamp ts)
{
    const int blocks = at.B * at.Hq * kMergeSlices + rows * r.nchunks;
    hipExtLaunchKernelGGL(merge_write_kernel, dim3(blocks), dim3(kThreads), 0, st, ts.start, ts.stop, 0, r, at, idx);
    return hipGetLastError();
}

}  // namespace hill
