// Grouped products: every workgroup takes one output tile of one of many independent products
// (GemmArgs in a device table), so that a dependency level of a small or middle-sized program costs
// one launch instead of one per product.
//
// What bounds it: at these sizes a product alone has a few workgroups and waits on launch, address
// table and operand latency; side by side the products of a level fill the chip.  The molecular-limit
// sigma (o=4, v=12, 9 right-hand sides, complex128) went from 0.65 ms in 53 launches to 0.09 ms in 11 by
// this (0.064 now), the three-k chain (o=4, v=20, 12 right-hand sides) from 3.53 to 0.87 ms (0.61 now), Nk=4,
// o=6, v=26 (6 right-hand sides, forward and backward) from 17.0 to 9.6 ms (7.4 now).
#include "tile.hpp"

namespace lrcc {

template <typename T, int TM, int TN, int WTM, int WTN>
__device__ __forceinline__ void group_tile(const GemmArgs &g, const GroupItem &it, void *lds) {
    TileLds<T, TM, TN> &l = *reinterpret_cast<TileLds<T, TM, TN> *>(lds);
    if (g.sk.tri) tile_product<T, TM, TN, WTM, WTN, true>(g, l, it.m0, it.n0, it.sb, it.t0, it.t1, it.js, it.beta, it.C, nullptr);
    else tile_product<T, TM, TN, WTM, WTN, false>(g, l, it.m0, it.n0, it.sb, it.t0, it.t1, it.js, it.beta, it.C, nullptr);
}

// LARGE 0: the tiles of one fragment per wave, which share a launch (a launch per tile would queue
// short launches behind each other); 1: 64x64
template <typename T, int LARGE>
__global__ void __launch_bounds__(kTileThreads, 2) gemm_group_kernel(const GemmArgs *__restrict__ ops,
                                                        const GroupItem *__restrict__ items) {
    constexpr size_t bytes = LARGE ? sizeof(TileLds<T, 64, 64>) : sizeof(TileLds<T, 16, 64>);
    __shared__ __attribute__((aligned(16))) char lds[bytes];
    const GroupItem it = items[blockIdx.x];
    const GemmArgs &g = ops[it.op];
    if constexpr (LARGE) {
        group_tile<T, 64, 64, 32, 32>(g, it, lds);
    } else {
        static_assert(sizeof(TileLds<T, 32, 32>) <= bytes && sizeof(TileLds<T, 64, 16>) <= bytes, "LDS of the small tiles");
        if (it.tile == 0) group_tile<T, 32, 32, 16, 16>(g, it, lds);
        else if (it.tile == 2) group_tile<T, 16, 64, 16, 16>(g, it, lds);
        else group_tile<T, 64, 16, 16, 16>(g, it, lds);
    }
}

template <typename T>
hipError_t launch_gemm_group(int cls, const GemmArgs *ops, const GroupItem *items, int n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    if (cls == 2) {
        if constexpr (sizeof(T) == 4) return launch_split_group(ops, items, n, s);
        return hipErrorInvalidValue;
    }
    if (cls == 1) hipLaunchKernelGGL((gemm_group_kernel<T, 1>), dim3(n), dim3(kTileThreads), 0, s, ops, items);
    else hipLaunchKernelGGL((gemm_group_kernel<T, 0>), dim3(n), dim3(kTileThreads), 0, s, ops, items);
    return hipGetLastError();
}

// Sums of arrays, many tensors in one launch (bound by memory; the arrays are small or still cached).
// The order of the summands is fixed, so results do not vary.
template <typename T>
__global__ void k_sums(const SumSeg *__restrict__ segs, const void *const *__restrict__ src,
                       const int2 *__restrict__ work) {
    typedef typename Cx<T>::type C2;
    const int2 w = work[blockIdx.x];
    const SumSeg g = segs[w.x];
    const i64 e0 = (i64)w.y * kSumChunk;
    const i64 e1 = e0 + kSumChunk < g.n ? e0 + kSumChunk : g.n;
    C2 *dst = reinterpret_cast<C2 *>(g.dst);
    for (i64 e = e0 + threadIdx.x; e < e1; e += blockDim.x) {
        double2 a = make_double2(0, 0);          // summed in double, rounded once
        int q = 0;
        for (; q + 4 <= g.nsrc; q += 4) {       // four loads in flight
            C2 v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = reinterpret_cast<const C2 *>(src[g.src0 + q + u])[e];
#pragma unroll
            for (int u = 0; u < 4; ++u) { a.x += (double)v[u].x; a.y += (double)v[u].y; }
        }
        for (; q < g.nsrc; ++q) {
            const C2 v = reinterpret_cast<const C2 *>(src[g.src0 + q])[e];
            a.x += (double)v.x;
            a.y += (double)v.y;
        }
        C2 w2;
        w2.x = (T)a.x;
        w2.y = (T)a.y;
        dst[e] = w2;
    }
}

template <typename T>
hipError_t launch_sums(const SumSeg *segs, const void *const *src, const int2 *work, int n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_sums<T>, dim3(n), dim3(256), 0, s, segs, src, work);
    return hipGetLastError();
}

template hipError_t launch_gemm_group<double>(int, const GemmArgs *, const GroupItem *, int, hipStream_t);
template hipError_t launch_gemm_group<float>(int, const GemmArgs *, const GroupItem *, int, hipStream_t);
template hipError_t launch_sums<double>(const SumSeg *, const void *const *, const int2 *, int, hipStream_t);
template hipError_t launch_sums<float>(const SumSeg *, const void *const *, const int2 *, int, hipStream_t);

}  // namespace lrcc
