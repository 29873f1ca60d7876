// Scoring sketch of the key cache (Sec. 4.4 asymmetric precision: the
// evaluation runs in low precision while attention keeps the 16-bit K and V).
//
//  sketch_keys  casts key rows [t0, t1) of every (sequence, KV head) to int8
//               (BITS 8) or int4 (BITS 4) codes with one power-of-two
//               exponent per row: the smallest e with max|x| * 2^-e <= qmax
//               (127 or 7), codes x * 2^-e rounded to nearest (ties to even).
//               Every operation is exact, so the sketch does not depend on
//               the order of evaluation.  In a decode loop it runs once per
//               appended token; the scan then reads 128 + 1 (int8) or 64 + 1
//               (int4) bytes per key row instead of 256.
//
// Layout: 16 lanes per row, lane l16 reads elements [8*l16, 8*l16+8) with one
// 16-byte load and writes their 8 codes with one 8-byte store (int8) or one
// 4-byte word (int4: byte i = (code i + 8) | (code i+4 + 8) << 4).  A wave
// covers 4 rows per load, a workgroup 16; it takes kSketchBatch such groups at
// once, so that enough loads are in flight, of one (sequence, KV head), so that
// no row number is divided.  The bound is a copy's (reads and writes mixed):
// 8 x 32768 rows, 101 MB, in 21.9 us (4.6 TB/s; a 2 GiB copy reaches 4.9),
// 23.3 with one row per lane group and 64-bit divisions.
#include <hip/hip_ext.h>

#include "hill_device.h"
#include "hill_internal.h"

namespace hill {

namespace {

constexpr int kSketchBatch = 4;                     // rows per lane group
constexpr int kSketchRows = 16 * kSketchBatch;      // rows per workgroup

template <int DT, int BITS>
__global__ __launch_bounds__(256) void sketch_keys_kernel(SketchArgs a)
{
    constexpr int kQmax = BITS == 8 ? 127 : 7;
    const int l16 = threadIdx.x & 15;
    const int j0 = a.t0 + blockIdx.x * kSketchRows + (threadIdx.x >> 4);   // then + 16, ...
    for (int bg = blockIdx.y; bg < a.B * a.Hkv; bg += gridDim.y) {
        const int b = bg / a.Hkv, g = bg % a.Hkv;
        const uint16_t* kb = a.k + (int64_t)b * a.k_sb + (int64_t)g * a.k_sh + l16 * 8;
        uint4 w[kSketchBatch];
        // every lane takes part in the row maxima (rows past the range repeat its last and are not stored)
#pragma unroll
        for (int u = 0; u < kSketchBatch; ++u) w[u] = load_stream16(kb + (int64_t)min(j0 + 16 * u, a.t1 - 1) * a.k_sn);
#pragma unroll
        for (int u = 0; u < kSketchBatch; ++u) {
            const int j = j0 + 16 * u;
            const uint32_t pw[4] = {w[u].x, w[u].y, w[u].z, w[u].w};
            float x[8];
            float amax = 0.0f;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                widen2<DT>(pw[i], x[2 * i], x[2 * i + 1]);
                amax = fmaxf(amax, fmaxf(fabsf(x[2 * i]), fabsf(x[2 * i + 1])));
            }
            const int e = sketch_exponent<kQmax>(max16(amax));
            const int64_t row = (int64_t)bg * a.cap + j;
            if constexpr (BITS == 8) {
                uint32_t lo = 0u, hi = 0u;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    lo |= ((uint32_t)sketch_code<kQmax>(x[i], e) & 0xffu) << (8 * i);
                    hi |= ((uint32_t)sketch_code<kQmax>(x[4 + i], e) & 0xffu) << (8 * i);
                }
                if (j < a.t1) *reinterpret_cast<uint2*>(a.k8 + row * kHeadDim + l16 * 8) = make_uint2(lo, hi);
            } else {
                uint32_t word = 0u;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t lo = (uint32_t)(sketch_code<kQmax>(x[i], e) + 8);
                    const uint32_t hi = (uint32_t)(sketch_code<kQmax>(x[4 + i], e) + 8);
                    word |= (lo | (hi << 4)) << (8 * i);
                }
                if (j < a.t1) *reinterpret_cast<uint32_t*>(a.k8 + row * (kHeadDim / 2) + l16 * 4) = word;
            }
            if (j < a.t1 && l16 == 0) a.k_exp[row] = (int8_t)e;
        }
    }
}

}  // namespace

hipError_t launch_sketch_keys(const SketchArgs& a, int dtype, hipStream_t st)
{
    if (a.t1 <= a.t0) return hipSuccess;
    const int64_t bg = (int64_t)a.B * a.Hkv;
    const dim3 grid((a.t1 - a.t0 + kSketchRows - 1) / kSketchRows, (unsigned)(bg < 65535 ? bg : 65535));
    if (a.bits == 4) {
        if (dtype == 1) hipLaunchKernelGGL((sketch_keys_kernel<1, 4>), grid, dim3(256), 0, st, a);
        else hipLaunchKernelGGL((sketch_keys_kernel<0, 4>), grid, dim3(256), 0, st, a);
    } else {
        if (dtype == 1) hipLaunchKernelGGL((sketch_keys_kernel<1, 8>), grid, dim3(256), 0, st, a);
        else hipLaunchKernelGGL((sketch_keys_kernel<0, 8>), grid, dim3(256), 0, st, a);
    }
    return hipGetLastError();
}

}  // namespace hill
