// Standalone sparse decode attention over a caller-given index set (Eq. 1
// restricted to the selected set I, softmax renormalised over I; Sec. 4.1
// workflow step 6: only the selected tokens' original 16-bit K and V rows are
// read, in place).  hill_step does not use these two kernels: its attention
// is fused into the selection's emit kernel (topk.hip).
//
//  attn_split    one workgroup per (sequence, KV head, split of I); each K
//                and V row is read once for all G query heads of the group.
//  attn_combine  merges the split partials of each query head.
#include <hip/hip_ext.h>

#include "attn_device.h"

namespace hill {

namespace {

template <int DT, int GC, bool MASK>
__global__ __launch_bounds__(256) void attn_split_kernel(AttnArgs a)
{
    __shared__ AttnLds<GC> sh;
    const int split = blockIdx.x;
    const int b = blockIdx.y / a.Hkv, g = blockIdx.y % a.Hkv;
    const int r = a.R == 1 ? 0 : g;
    const int32_t* I = a.idx + ((int64_t)b * a.R + r) * a.ksel;
    const int t0 = split * a.per_split;
    const int t1 = min(t0 + a.per_split, a.ksel);
    for (int hc = 0; hc < a.G; hc += GC) {
        uint4 qv[GC];
        load_queries<GC, MASK>(a, b, g, hc, qv);
        AttnAcc<GC> acc;
        attn_begin<GC>(acc, sh);
        for (int tb = t0; tb < t1; tb += kAttnBlock) {
            const int cnt = min(kAttnBlock, t1 - tb);
            __syncthreads();   // the previous block's list reads are done
            for (int i = threadIdx.x; i < cnt; i += 256) sh.tok[i] = I[tb + i];
            __syncthreads();
            attn_block<DT, GC>(a, b, g, qv, cnt, acc, sh);
        }
        attn_finish<GC, MASK>(a, b, g, hc, acc, split, a.nsplit, sh);
    }
}

__global__ __launch_bounds__(kHeadDim) void attn_combine_kernel(AttnArgs a)
{
    __shared__ float red[kHeadDim / 64 + 1];
    __shared__ float osum[kHeadDim];
    merge_head<kHeadDim>(a, blockIdx.x / a.Hq, blockIdx.x % a.Hq, 0, a.nsplit, red, osum);
}

template <int DT>
hipError_t launch_attn_dt(const AttnArgs& a, dim3 grid, hipStream_t st)
{
    const bool mask = masked_pass(a.G);
    auto kernel = attn_split_kernel<DT, 1, false>;
    switch (heads_per_pass(a.G)) {
    case 8: kernel = mask ? attn_split_kernel<DT, 8, true> : attn_split_kernel<DT, 8, false>; break;
    case 4: kernel = mask ? attn_split_kernel<DT, 4, true> : attn_split_kernel<DT, 4, false>; break;
    case 2: kernel = attn_split_kernel<DT, 2, false>; break;
    }
    hipLaunchKernelGGL(kernel, grid, dim3(256), 0, st, a);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_attn_split(const AttnArgs& a, int dtype, hipStream_t st)
{
    dim3 grid(a.nsplit, a.B * a.Hkv);
    if (dtype == 1) return launch_attn_dt<1>(a, grid, st);
    return launch_attn_dt<0>(a, grid, st);
}

hipError_t launch_attn_combine(const AttnArgs& a, hipStream_t st, Stamp ts)
{
    hipExtLaunchKernelGGL(attn_combine_kernel, dim3(a.B * a.Hq), dim3(kHeadDim), 0, st, ts.start, ts.stop, 0, a);
    return hipGetLastError();
}

}  // namespace hill
