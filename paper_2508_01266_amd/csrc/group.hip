// Grouped products: every workgroup takes one output tile of one of many independent products
// (GemmArgs in a device table), so that a dependency level of a small or middle-sized program costs
// one launch instead of one per product.
//
// What bounds it: at these sizes a product alone has a few workgroups and waits on launch, address
// table and operand latency; side by side the products of a level fill the chip.  The molecular-limit
// sigma (o=4, v=12, 9 right-hand sides, complex128) takes 0.09 ms in 11 launches against 0.65 ms in
// 53, the three-k chain (o=4, v=20, 12 right-hand sides) 0.87 ms against 3.53 ms, Nk=4, o=6, v=26
// (6 right-hand sides, forward and backward) 9.6 ms against 17.0 ms.
#include "group.hpp"

namespace lrcc {

namespace {
template <typename T> struct GM;
template <> struct GM<double> {
    typedef double v4 __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ v4 mma(double a, double b, v4 c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int lane, int r) { return (lane >> 4) + 4 * r; }
};
template <> struct GM<float> {
    typedef float v4 __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ v4 mma(float a, float b, v4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int lane, int r) { return 4 * (lane >> 4) + r; }
};
constexpr int NT = 256;
}  // namespace

// The products of one tile over reduction steps [t0, t1): four waves, each WTM x WTN; complex
// elements stay interleaved in LDS (one wide read gives both parts of an operand).  Two LDS buffers,
// one barrier per step; operands are loaded two steps ahead, since one step of a small tile
// (16 to 64 matrix instructions per wave) is shorter than a trip to memory.
template <typename T, int TM, int TN, int WTM, int WTN, bool TRI>
__device__ __forceinline__ void group_tile(const GemmArgs &g, const GroupItem &it, typename Cx<T>::type *lds) {
    typedef typename Cx<T>::type C2;
    typedef typename GM<T>::v4 v4;
    constexpr int TK = kGroupTK;
    constexpr int WGM = TM / WTM, FM = WTM / 16, FN = WTN / 16;
    constexpr int LA = TM * TK / NT, LB = TK * TN / NT;
    constexpr int SA = TM + 1, SB = TN + 1;
    static_assert((TM / WTM) * (TN / WTN) == 4, "4 waves per block");
    C2 *const bufA[2] = {lds, lds + TK * SA};
    C2 *const bufB[2] = {lds + 2 * TK * SA, lds + 2 * TK * SA + TK * SB};
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = (wave % WGM) * WTM, wn = (wave / WGM) * WTN;
    const C2 *A = reinterpret_cast<const C2 *>(g.A);
    const C2 *B = reinterpret_cast<const C2 *>(g.B);
    const bool aM = g.aMfast != 0, bN = g.bNfast != 0;
    const int ak0 = (int)g.Ak.s[0], ak1 = (int)g.Ak.s[1], ak2 = (int)g.Ak.s[2];
    const int bk0 = (int)g.Bk.s[0], bk1 = (int)g.Bk.s[1], bk2 = (int)g.Bk.s[2];
    int am[LA], ak[LA], bk[LB], bn[LB], arow[LA], bcol[LB];
    bool aok[LA], bok[LB];
#pragma unroll
    for (int q = 0; q < LA; ++q) {
        const int idx = tid + NT * q;
        if (aM) { am[q] = idx % TM; ak[q] = idx / TM; } else { ak[q] = idx % TK; am[q] = idx / TK; }
        const int gm = it.m0 + am[q];
        aok[q] = gm < g.M;
        arow[q] = aok[q] ? split_off32(gm, g.sm, (int)g.Am.s[0], (int)g.Am.s[1], (int)g.Am.s[2]) : 0;
    }
#pragma unroll
    for (int q = 0; q < LB; ++q) {
        const int idx = tid + NT * q;
        if (bN) { bn[q] = idx % TN; bk[q] = idx / TN; } else { bk[q] = idx % TK; bn[q] = idx / TK; }
        const int gn = it.n0 + bn[q];
        bok[q] = gn < g.N;
        bcol[q] = bok[q] ? split_off32(gn, g.sn, (int)g.Bn.s[0], (int)g.Bn.s[1], (int)g.Bn.s[2]) : 0;
    }
    v4 accr[FM][FN], acci[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) { accr[i][j] = v4{0, 0, 0, 0}; acci[i][j] = v4{0, 0, 0, 0}; }
    // complex64: the running sums move to a second set every kFlush steps (128 elements), so that the
    // rounding of a long reduction grows with its pieces and not with its length
    constexpr bool FLUSH = sizeof(T) == 4;
    constexpr int kFlush = 8;
    v4 sumr[FLUSH ? FM : 1][FLUSH ? FN : 1], sumi[FLUSH ? FM : 1][FLUSH ? FN : 1];
    auto flush = [&](bool first) {
        if constexpr (FLUSH) {
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j) {
                    sumr[i][j] = first ? accr[i][j] : sumr[i][j] + accr[i][j];
                    sumi[i][j] = first ? acci[i][j] : sumi[i][j] + acci[i][j];
                    accr[i][j] = v4{0, 0, 0, 0};
                    acci[i][j] = v4{0, 0, 0, 0};
                }
        }
    };
    flush(true);
    const int ksteps = (g.K + TK - 1) / TK;
    C2 va[2][LA], vb[2][LB];
    auto fetch = [&](int t, C2 *ra, C2 *rb) {
        const int s = it.sb + t / ksteps, k0 = (t % ksteps) * TK;
        const C2 *As = A + g.segA[s];
        const C2 *Bs = B + g.segB[s];
#pragma unroll
        for (int q = 0; q < LA; ++q) {
            const int gk = k0 + ak[q];
            if (aok[q] && gk < g.K) ra[q] = As[arow[q] + split_off32<TRI>(gk, g.sk, ak0, ak1, ak2)];
            else { ra[q].x = 0; ra[q].y = 0; }
        }
#pragma unroll
        for (int q = 0; q < LB; ++q) {
            const int gk = k0 + bk[q];
            if (bok[q] && gk < g.K) rb[q] = Bs[bcol[q] + split_off32<TRI>(gk, g.sk, bk0, bk1, bk2)];
            else { rb[q].x = 0; rb[q].y = 0; }
        }
    };
    auto step = [&](const C2 *ra, const C2 *rb, C2 *la, C2 *lb, int tnext, C2 *na, C2 *nb) {
#pragma unroll
        for (int q = 0; q < LA; ++q) la[ak[q] * SA + am[q]] = ra[q];
#pragma unroll
        for (int q = 0; q < LB; ++q) lb[bk[q] * SB + bn[q]] = rb[q];
        __syncthreads();
        if (tnext < it.t1) fetch(tnext, na, nb);
#pragma unroll
        for (int kk = 0; kk < TK; kk += 4) {
            const int kr = kk + (lane >> 4), c = lane & 15;
            C2 a[FM], b[FN];
#pragma unroll
            for (int i = 0; i < FM; ++i) a[i] = la[kr * SA + wm + 16 * i + c];
#pragma unroll
            for (int j = 0; j < FN; ++j) b[j] = lb[kr * SB + wn + 16 * j + c];
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j) {
                    accr[i][j] = GM<T>::mma(a[i].x, b[j].x, accr[i][j]);
                    acci[i][j] = GM<T>::mma(a[i].x, b[j].y, acci[i][j]);
                    accr[i][j] = GM<T>::mma(-a[i].y, b[j].y, accr[i][j]);
                    acci[i][j] = GM<T>::mma(a[i].y, b[j].x, acci[i][j]);
                }
        }
    };
    if (it.t0 < it.t1) fetch(it.t0, va[0], vb[0]);
    if (it.t0 + 1 < it.t1) fetch(it.t0 + 1, va[1], vb[1]);
    // a buffer is rewritten two steps later, after the barrier of the step between, which every
    // wave reaches only once it has finished reading it
    for (int t = it.t0; t < it.t1; t += 2) {
        step(va[0], vb[0], bufA[0], bufB[0], t + 2, va[0], vb[0]);
        if (t + 1 < it.t1) step(va[1], vb[1], bufA[1], bufB[1], t + 3, va[1], vb[1]);
        if (FLUSH && (t - it.t0) % kFlush == kFlush - 2) flush(false);
    }
    if constexpr (FLUSH) {
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j) { accr[i][j] += sumr[i][j]; acci[i][j] += sumi[i][j]; }
    }
    const T alr = (T)it.js * (T)g.alpha_re, ali = (T)it.js * (T)g.alpha_im;
    C2 *Cj = reinterpret_cast<C2 *>(it.C);
    i64 coff[FN];
    bool cok[FN];
#pragma unroll
    for (int j = 0; j < FN; ++j) {
        const int gn = it.n0 + wn + 16 * j + (lane & 15);
        cok[j] = gn < g.N;
        coff[j] = cok[j] ? split_off(gn, g.sn, g.Cn) : 0;
    }
#pragma unroll
    for (int i = 0; i < FM; ++i) {
        i64 roff[4];
        bool rok[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int gm = it.m0 + wm + 16 * i + GM<T>::row(lane, r);
            rok[r] = gm < g.M;
            roff[r] = rok[r] ? split_off(gm, g.sm, g.Cm) : 0;
        }
        C2 old[FN][4];
        if (it.beta) {
            // all reads before the first write (a write may alias a later read as far as the
            // compiler knows); outside elements read the block's first in range
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) old[j][r] = Cj[rok[r] && cok[j] ? roff[r] + coff[j] : 0];
        }
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                if (!(rok[r] && cok[j])) continue;
                const T xr = accr[i][j][r], xi = acci[i][j][r];
                C2 w;
                w.x = alr * xr - ali * xi;
                w.y = alr * xi + ali * xr;
                if (it.beta) { w.x += old[j][r].x; w.y += old[j][r].y; }
                Cj[roff[r] + coff[j]] = w;
            }
    }
}

template <typename T, int TM, int TN, int WTM, int WTN>
__device__ __forceinline__ void group_tile_any(const GemmArgs &g, const GroupItem &it, typename Cx<T>::type *lds) {
    if (g.sk.tri) group_tile<T, TM, TN, WTM, WTN, true>(g, it, lds);
    else group_tile<T, TM, TN, WTM, WTN, false>(g, it, lds);
}

constexpr int group_lds(int tm, int tn) { return 2 * kGroupTK * (tm + 1 + tn + 1); }

// LARGE 0: the tiles of one fragment per wave, which share a launch (a launch per tile would queue
// short launches behind each other); 1: 64x64
template <typename T, int LARGE>
__global__ void __launch_bounds__(NT) gemm_group_kernel(const GemmArgs *__restrict__ ops,
                                                        const GroupItem *__restrict__ items) {
    __shared__ typename Cx<T>::type lds[LARGE ? group_lds(64, 64) : group_lds(16, 64)];
    const GroupItem it = items[blockIdx.x];
    const GemmArgs &g = ops[it.op];
    if constexpr (LARGE) {
        group_tile_any<T, 64, 64, 32, 32>(g, it, lds);
    } else {
        if (it.tile == 0) group_tile_any<T, 32, 32, 16, 16>(g, it, lds);
        else if (it.tile == 2) group_tile_any<T, 16, 64, 16, 16>(g, it, lds);
        else group_tile_any<T, 64, 16, 16, 16>(g, it, lds);
    }
}

template <typename T>
hipError_t launch_gemm_group(int large, const GemmArgs *ops, const GroupItem *items, int n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    if (large) hipLaunchKernelGGL((gemm_group_kernel<T, 1>), dim3(n), dim3(NT), 0, s, ops, items);
    else hipLaunchKernelGGL((gemm_group_kernel<T, 0>), dim3(n), dim3(NT), 0, s, ops, items);
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
        C2 a;
        a.x = 0;
        a.y = 0;
        for (int q = 0; q < g.nsrc; ++q) {
            const C2 v = reinterpret_cast<const C2 *>(src[g.src0 + q])[e];
            a.x += v.x;
            a.y += v.y;
        }
        dst[e] = a;
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
