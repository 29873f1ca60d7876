// Short rows: the selection and all that follows it in one launch, by one
// workgroup (or two) per KV head instead of a refine, an emit and a merge
// launch over 512-token chunks.
//
//  row_attend  hill_step on rows of at most kRowTokens tokens and kRowPicks
//              selected ones: the exact top-k of the row (row_device.h), the
//              ordered index list, and the attention of the KV head's query
//              heads over it, written as the final output.  What bounds such
//              a step is the chain of launches (2 to 5 us each with its
//              boundary, for microseconds of work), so repeating the row's
//              selection in every KV head's workgroup is cheaper than sharing
//              it.
//  row_topk    hill_topk on rows of at most kRowTopkTokens tokens.
#include <hip/hip_ext.h>

#include "attn_device.h"
#include "row_device.h"

namespace hill {

namespace {

constexpr int kRowV = 4;         // output dimensions per lane: 8-byte loads of a V row
constexpr int kRowCopies = 4;    // of the digit counts: they lie where the weights and outputs go later
constexpr int kRowBatch = 8;     // V loads in flight per lane and buffer (two buffers)

template <int GC>
struct RowAttnLds {
    int32_t tok[kRowPicks];
    union {
        alignas(16) uint32_t bins[row_bin_words(kRowCopies)];   // the selection's
        float p[kRowPicks][GC];                      // logits, then weights
        float o[kRowWaves * kHeadDim * GC];          // the waves' outputs, once every weight has been read
    };
    float m[kRowWaves][GC], l[kRowWaves][GC];        // per-wave maxima and sums
};

// Sum of N values pairwise: the partial sums of one output or softmax
// normaliser.  One after another their roundings add up instead (against 64
// bits, 1021 tokens with 204 picks, whole step: 2.1e-7 serial, 1.7e-7 in the
// chunked kernels).
template <int N>
__device__ __forceinline__ float sum_pairwise(float (&v)[N])
{
#pragma unroll
    for (int m = N / 2; m > 0; m /= 2)
#pragma unroll
        for (int i = 0; i < m; ++i) v[i] += v[i + m];
    return v[0];
}

// DSPLIT: 2 workgroups per KV head, each for half of the output dimensions
// (a 128-byte line of every V row), where few KV heads leave CUs idle.
// LG: the logits are the scan's own (at.logits); else K rows are gathered.
// TIER: a tiered cache; the list then holds ~slot for a token whose rows lie
// in the hot pool.  With r.state_out (a streamed step's state) the bound is
// written as the refine pass would.
template <int DT, int GC, bool LG, bool TIER, int TPT, int DSPLIT>
__global__ __launch_bounds__(kRowThreads) void row_attend_kernel(RefineArgs r, AttnArgs at, int32_t* idx)
{
    constexpr int LPR = kHeadDim / DSPLIT / kRowV;   // lanes per V row
    constexpr int RPI = 64 / LPR;                    // rows per wave and load
    constexpr int STEP = kRowWaves * RPI;            // list entries per load of the workgroup
    __shared__ RowLds rl;
    __shared__ RowAttnLds<GC> sh;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ds = blockIdx.x % DSPLIT, g = blockIdx.x / DSPLIT, b = blockIdx.y;
    const int row = r.R == 1 ? b : b * at.Hkv + g;
    constexpr int GS = TPT < 4 ? TPT : 4;
    static_assert(TPT == GS, "one group per thread");
    const int j0 = row_token<TPT, GS>(0);

    float sx[TPT];
    row_load<TPT, GS>(r.s + (int64_t)b * r.s_sb + (int64_t)(r.R == 1 ? 0 : g) * r.s_sr, r.n, sx);
    // the first pass's logits of this thread's tokens, in flight during the selection
    float lg[LG ? GC : 1][TPT];
    if constexpr (LG) {
        const float* p = at.logits + ((int64_t)b * at.Hq + g * at.G) * at.ld;
#pragma unroll
        for (int hh = 0; hh < GC; ++hh) {
            row_load<TPT, GS>(p, r.n, lg[hh]);
            p += hh + 1 < at.G ? at.ld : 0;   // heads past G repeat the last (masked below)
        }
    }
    uint32_t key[TPT];
    bool ok[TPT], sel[TPT];
    row_keys<TPT, GS>(sx, r.n, r.pin_lo, r.pin_hi, key, ok);
    uint32_t before[1];
    const RowBound bound = row_select<TPT, GS, kRowCopies>(key, ok, (uint32_t)r.k, rl, sh.bins, sel, before);
    const bool writer = ds == 0 && (r.R != 1 || g == 0);
    if (r.state_out && writer && tid == 0) {
        r.state_out[2 * row] = make_uint4(bound.b1 << 20, (uint32_t)r.k - bound.need1 + bound.in1, (uint32_t)r.n, 1u);
        r.state_out[2 * row + 1] = make_uint4((uint32_t)r.pin_lo, (uint32_t)(r.n - r.pin_hi), 0u, 0u);
    }
    const int cnt = r.k;
    {
        uint32_t p = before[0];
#pragma unroll
        for (int e = 0; e < TPT; ++e)
            if (sel[e] && p < (uint32_t)cnt) {   // exactly k are selected
                int at_row = j0 + e;
                if constexpr (TIER) {
                    const int slot = at.loc[(int64_t)row * at.loc_sr + j0 + e];
                    at_row = slot >= 0 ? ~slot : at_row;
                }
                sh.tok[p] = at_row;
                if (writer) idx[(int64_t)row * r.k + p] = j0 + e;
                if constexpr (LG) {
#pragma unroll
                    for (int hh = 0; hh < GC; ++hh) sh.p[p][hh] = at.s2 * lg[hh][e];
                }
                ++p;
            }
    }
    __syncthreads();

    const int sub = lane / LPR, d0 = ds * (kHeadDim / DSPLIT) + (lane % LPR) * kRowV;
    const uint16_t* vb = at.v + (int64_t)b * at.v_sb + (int64_t)g * at.v_sh + d0;
    const uint16_t* vhot = TIER ? at.v_hot + (int64_t)b * at.hv_sb + (int64_t)g * at.hv_sh + d0 : vb;
    // list entry t's row: of the cache (or cold pool), or of the hot pool
    auto row_of = [&](int t, const uint16_t* cold, int64_t cold_sn, const uint16_t* hot, int64_t hot_sn) {
        const int j = sh.tok[t];
        if constexpr (TIER) {
            if (j < 0) return hot + row_off(~j, at.cap, hot_sn);
        }
        return cold + row_off(j, at.n, cold_sn);
    };
    const int e0 = w * RPI + sub;   // this lane's entries: e0, e0 + STEP, ...
    auto load_v = [&](int i0, uint2 (&v)[kRowBatch]) {
#pragma unroll
        for (int i = 0; i < kRowBatch; ++i) {
            const int e = min(e0 + (i0 + i) * STEP, cnt - 1);   // past the list: its last row, weighing 0
            v[i] = *reinterpret_cast<const uint2*>(row_of(e, vb, at.v_sn, vhot, at.hv_sn));
        }
    };
    for (int hc = 0; hc < at.G; hc += GC) {
        uint2 va[kRowBatch], vn[kRowBatch];
        if constexpr (LG) {
            if (hc > 0) {   // further passes take their logits by token
                const float* lp = at.logits + ((int64_t)b * at.Hq + g * at.G + hc) * at.ld;
                for (int t = tid; t < cnt; t += kRowThreads) {
                    const int j = sh.tok[t];
#pragma unroll
                    for (int hh = 0; hh < GC; ++hh) sh.p[t][hh] = at.s2 * lp[min(hh, at.G - 1 - hc) * at.ld + j];
                }
            }
            load_v(0, va);
        } else {
            // 16-lane row groups: K rows of entries rg, rg + 64, ...
            uint4 qv[GC];
            load_queries<GC, true>(at, b, g, hc, qv);
            const int rg = tid >> 4, l16 = tid & 15;
            const uint16_t* kb = at.k + (int64_t)b * at.k_sb + (int64_t)g * at.k_sh + l16 * 8;
            const uint16_t* khot = TIER ? at.k_hot + (int64_t)b * at.hk_sb + (int64_t)g * at.hk_sh + l16 * 8 : kb;
            constexpr int kNB = GC <= 4 ? 4 : 2, kGroups = kRowThreads / 16;   // 8 heads' queries leave registers for two
            for (int t0 = rg; t0 - rg < cnt; t0 += kGroups * kNB) {   // workgroup-uniform trips
                uint4 kr[kNB];
#pragma unroll
                for (int u = 0; u < kNB; ++u)
                    kr[u] = *reinterpret_cast<const uint4*>(
                        row_of(min(t0 + u * kGroups, cnt - 1), kb, at.k_sn, khot, at.hk_sn));
                if (t0 == rg) load_v(0, va);   // behind the first K rows
#pragma unroll
                for (int u = 0; u < kNB; ++u) {
                    const int t = t0 + u * kGroups;
                    float mine = 0.0f;
#pragma unroll
                    for (int hh = 0; hh < GC; ++hh) {
                        const float d = sum16(dot8<DT>(kr[u], qv[hh]));
                        mine = l16 == hh ? d : mine;
                    }
                    if (l16 < GC && t < cnt) sh.p[t][l16] = at.s2 * mine;
                }
            }
        }
        if (!LG || hc > 0) __syncthreads();
        // softmax over the list: thread t weighs entries t, t + 1024, ... for every head
        constexpr int kPer = kRowPicks / kRowThreads;
        float x[kPer][GC], mx[GC], lsum[GC];
#pragma unroll
        for (int hh = 0; hh < GC; ++hh) mx[hh] = -INFINITY;
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int t = tid + i * kRowThreads;
#pragma unroll
            for (int hh = 0; hh < GC; ++hh) {
                x[i][hh] = t < cnt ? sh.p[t][hh] : -INFINITY;
                mx[hh] = fmaxf(mx[hh], x[i][hh]);
            }
        }
#pragma unroll
        for (int hh = 0; hh < GC; ++hh) {
            mx[hh] = wave_max(mx[hh]);
            if (lane == 0) sh.m[w][hh] = mx[hh];
        }
        __syncthreads();
#pragma unroll
        for (int hh = 0; hh < GC; ++hh) {
            mx[hh] = max16(sh.m[lane & (kRowWaves - 1)][hh]);
            lsum[hh] = 0.0f;
#pragma unroll
            for (int i = 0; i < kPer; ++i) {
                const float e = exp2_ftz(x[i][hh] - mx[hh]);
                const int t = tid + i * kRowThreads;
                if (t < cnt) sh.p[t][hh] = e;
                lsum[hh] += t < cnt ? e : 0.0f;
            }
            lsum[hh] = wave_sum(lsum[hh]);
            if (lane == 0) sh.l[w][hh] = lsum[hh];
        }
        __syncthreads();
        // weight * V of this lane's entries, the next batch in flight
        float acc[GC][kRowV];
#pragma unroll
        for (int hh = 0; hh < GC; ++hh)
#pragma unroll
            for (int d = 0; d < kRowV; ++d) acc[hh][d] = 0.0f;
        const int steps = (cnt + STEP - 1) / STEP;   // loads that hold an entry of any lane
        for (int i0 = 0; i0 < steps; i0 += kRowBatch) {
            const bool more = i0 + kRowBatch < steps;
            if (more) load_v(i0 + kRowBatch, vn);
#pragma unroll
            for (int i = 0; i < kRowBatch; ++i) {
                if (i0 + i >= steps) break;   // workgroup-uniform
                const int e = e0 + (i0 + i) * STEP;
                const int ec = min(e, cnt - 1);
                float v[kRowV];
                widen2<DT>(va[i].x, v[0], v[1]);
                widen2<DT>(va[i].y, v[2], v[3]);
#pragma unroll
                for (int hh = 0; hh < GC; ++hh) {
                    const float pw = e < cnt ? sh.p[ec][hh] : 0.0f;
#pragma unroll
                    for (int d = 0; d < kRowV; ++d) acc[hh][d] += pw * v[d];
                }
            }
            if (more) {
#pragma unroll
                for (int i = 0; i < kRowBatch; ++i) va[i] = vn[i];
            }
        }
        __syncthreads();   // every weight has been read
        // The sums of a wave's RPI rows per load are added in registers, each swap serving two of the lane's
        // GC * kRowV sums, after which lanes of row group `sub` hold the sub-th part of them; into
        // o[wave][head][dimension]
        constexpr int DW = kHeadDim / DSPLIT, NV = GC * kRowV, PV = NV / RPI, VW = PV < kRowV ? PV : kRowV;
        static_assert(RPI == 2 || RPI == 4, "lanes l ^ 32, or l ^ 16 and l ^ 32, hold the same dimensions");
        float sv[NV];
#pragma unroll
        for (int i = 0; i < NV / 2; ++i) {
            const int j = i + NV / 2;
            sv[i] = sum2_x32(acc[i / kRowV][i % kRowV], acc[j / kRowV][j % kRowV]);
        }
        if constexpr (RPI == 4) {
#pragma unroll
            for (int i = 0; i < NV / 4; ++i) sv[i] = sum2_x16(sv[i], sv[i + NV / 4]);
        }
#pragma unroll
        for (int i = 0; i < PV; i += VW) {
            const int f = sub * PV + i;   // the sum's head and dimension of four
            float* p = &sh.o[(w * GC + f / kRowV) * DW + (lane % LPR) * kRowV + f % kRowV];
            if constexpr (VW == 4) *reinterpret_cast<float4*>(p) = make_float4(sv[i], sv[i + 1], sv[i + 2], sv[i + 3]);
            else if constexpr (VW == 2) *reinterpret_cast<float2*>(p) = make_float2(sv[i], sv[i + 1]);
            else *p = sv[i];
        }
        __syncthreads();
        for (int t = tid; t < DW * GC; t += kRowThreads) {
            const int d = t % DW, hh = t / DW;
            float o[kRowWaves], l[kRowWaves];
#pragma unroll
            for (int i = 0; i < kRowWaves; ++i) {
                o[i] = sh.o[i * DW * GC + t];
                l[i] = sh.l[i][hh];
            }
            const float ov = sum_pairwise(o) / sum_pairwise(l);
            if (hc + hh < at.G) at.out[((int64_t)b * at.Hq + g * at.G + hc + hh) * kHeadDim + ds * DW + d] = ov;
        }
        __syncthreads();   // p is written again by the next pass
    }
}

template <int TPT>
__global__ __launch_bounds__(kRowThreads) void row_topk_kernel(RefineArgs r, int32_t* idx, float* val)
{
    __shared__ RowLds rl;
    __shared__ __attribute__((aligned(16))) uint32_t bins[row_bin_words(8)];
    const int row = blockIdx.x, b = row / r.R;
    const float* srow = r.s + (int64_t)b * r.s_sb + (int64_t)(row % r.R) * r.s_sr;
    constexpr int GS = 4;
    uint32_t key[TPT];
    bool ok[TPT], sel[TPT];
    {
        float sx[TPT];
        row_load<TPT, GS>(srow, r.n, sx);
        row_keys<TPT, GS>(sx, r.n, r.pin_lo, r.pin_hi, key, ok);
    }
    uint32_t p[TPT / GS];
    row_select<TPT, GS, 8>(key, ok, (uint32_t)r.k, rl, bins, sel, p);
#pragma unroll
    for (int e = 0; e < TPT; ++e)
        if (sel[e] && p[e / GS] < (uint32_t)r.k) {
            const int j = row_token<TPT, GS>(e);
            idx[(int64_t)row * r.k + p[e / GS]] = j;
            if (val) val[(int64_t)row * r.k + p[e / GS]] = srow[j];   // read again: the keys fill the registers
            ++p[e / GS];
        }
}

template <int DT, int GC, bool LG, bool TIER>
hipError_t launch_row_gc(const RefineArgs& r, const AttnArgs& at, int32_t* idx, hipStream_t st, Stamp ts)
{
    // half of the dimensions per workgroup while that leaves at most one per CU; gathering K is not split
    const bool split = LG && (int64_t)at.B * at.Hkv <= 128;
    const dim3 grid(at.Hkv * (split ? 2 : 1), at.B), wg(kRowThreads);
    auto kernel = r.n <= 2 * kRowThreads ? row_attend_kernel<DT, GC, LG, TIER, 2, 1>
                                         : row_attend_kernel<DT, GC, LG, TIER, 4, 1>;
    if constexpr (LG) {
        if (split)
            kernel = r.n <= 2 * kRowThreads ? row_attend_kernel<DT, GC, LG, TIER, 2, 2>
                                            : row_attend_kernel<DT, GC, LG, TIER, 4, 2>;
    }
    hipExtLaunchKernelGGL(kernel, grid, wg, 0, st, ts.start, ts.stop, 0, r, at, idx);
    return hipGetLastError();
}

template <int DT, bool LG, bool TIER>
hipError_t launch_row_dt(const RefineArgs& r, const AttnArgs& at, int32_t* idx, hipStream_t st, Stamp ts)
{
    switch (heads_per_pass(at.G)) {
    case 8: return launch_row_gc<DT, 8, LG, TIER>(r, at, idx, st, ts);
    case 4: return launch_row_gc<DT, 4, LG, TIER>(r, at, idx, st, ts);
    case 2: return launch_row_gc<DT, 2, LG, TIER>(r, at, idx, st, ts);
    default: return launch_row_gc<DT, 1, LG, TIER>(r, at, idx, st, ts);
    }
}

template <int DT>
hipError_t launch_row_any(const RefineArgs& r, const AttnArgs& at, int32_t* idx, hipStream_t st, Stamp ts)
{
    if (at.loc) return launch_row_dt<DT, false, true>(r, at, idx, st, ts);
    if (at.logits) return launch_row_dt<DT, true, false>(r, at, idx, st, ts);
    return launch_row_dt<DT, false, false>(r, at, idx, st, ts);
}

}  // namespace

hipError_t launch_row_attend(const RefineArgs& r, const AttnArgs& at, int dtype, int32_t* idx, hipStream_t st, Stamp ts)
{
    return dtype == 1 ? launch_row_any<1>(r, at, idx, st, ts) : launch_row_any<0>(r, at, idx, st, ts);
}

hipError_t launch_row_topk(const RefineArgs& r, int rows, int32_t* idx, float* val, hipStream_t st)
{
    auto kernel = r.n <= 8 * kRowThreads ? row_topk_kernel<8> : r.n <= 16 * kRowThreads ? row_topk_kernel<16> : row_topk_kernel<32>;
    hipLaunchKernelGGL(kernel, dim3(rows), dim3(kRowThreads), 0, st, r, idx, val);
    return hipGetLastError();
}

}  // namespace hill
