// Device helpers shared by the gx kernels (block scans and reductions, the
// saturating add of the min-plus relaxation).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "gx_internal.h"

namespace gx {

__device__ __forceinline__ uint32_t sat_add(uint32_t a, uint32_t b) {
    uint32_t s = a + b;
    return s < a ? INF : s;
}

// Exclusive prefix sum of a 64-bit value over a 256-thread block.
__device__ __forceinline__ unsigned long long block_excl_scan_u64(unsigned long long v, unsigned long long *total,
                                                                  unsigned long long *lds) {
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nw = blockDim.x >> 6;
    unsigned long long x = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        unsigned long long y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    if (lane == 63) lds[wid] = x;
    __syncthreads();
    unsigned long long pre = 0, tot = 0;
    for (int i = 0; i < nw; i++) {
        unsigned long long t = lds[i];
        if (i < wid) pre += t;
        tot += t;
    }
    *total = tot;
    __syncthreads();
    return pre + x - v;
}

// Sum over a block in a fixed tree (deterministic for floating point).
template <class T>
__device__ __forceinline__ T block_sum(T v, T *lds) {
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nw = blockDim.x >> 6;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
    if (lane == 0) lds[wid] = v;
    __syncthreads();
    T r = 0;
    if (wid == 0) {
        r = lane < nw ? lds[lane] : T(0);
#pragma unroll
        for (int o = 8; o > 0; o >>= 1) r += __shfl_down(r, o, 16);
    }
    __syncthreads();
    return r;  // valid in thread 0
}

// In-place inclusive max-scan of s[0..n) (n <= blockDim * VT), VT contiguous
// elements per thread.
template <int VT>
__device__ __forceinline__ void block_max_scan(int32_t *s, int n, int32_t *lds) {
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6, nw = blockDim.x >> 6;
    int32_t loc[VT];
    int32_t run = 0;
#pragma unroll
    for (int i = 0; i < VT; i++) {
        int p = tid * VT + i;
        int32_t v = p < n ? s[p] : 0;
        run = max(run, v);
        loc[i] = run;
    }
    int32_t x = run;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        int32_t y = __shfl_up(x, o, 64);
        if (lane >= o) x = max(x, y);
    }
    if (lane == 63) lds[wid] = x;
    __syncthreads();
    int32_t pre = 0;
    for (int i = 0; i < wid; i++) pre = max(pre, lds[i]);
    (void)nw;
    int32_t excl = __shfl_up(x, 1, 64);
    if (lane == 0) excl = 0;
    excl = max(excl, pre);
#pragma unroll
    for (int i = 0; i < VT; i++) {
        int p = tid * VT + i;
        if (p < n) s[p] = max(loc[i], excl);
    }
    __syncthreads();
}


// The XCD (accelerator complex die) the calling wave runs on: bits 3:0 of
// the XCC_ID hardware register.
__device__ __forceinline__ uint32_t xcc_id() { return __builtin_amdgcn_s_getreg((3 << 11) | 20) & 15u; }

}  // namespace gx
