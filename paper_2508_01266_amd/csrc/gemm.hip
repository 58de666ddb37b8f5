// Batched strided complex GEMM on the gfx950 matrix cores.
//
// A complex product is four real MFMA products on the real and imaginary
// parts: Cre += Are*Bre - Aim*Bim, Cim += Are*Bim + Aim*Bre (tile_product).
// Operand addresses use the three-level index splits of GemmArgs so that k-blocked
// tensors are read in place (no permute passes); the thread->element map of each
// tile load runs along the unit-stride index when one exists, for coalesced loads.
// The large complex64 products run on the bf16 matrix cores instead (split.hip).
#include "tile.hpp"

#include <algorithm>
#include <vector>

namespace lrcc {

// One tile per workgroup, jobs along grid.y, reduction splits along grid.z (their raw sums go to g.part).
// KIND 1: the ladder products over integral blocks (a kernel symbol of their own for profiles).
template <typename T, int TM, int TN, int WTM, int WTN, int KIND, bool TRI>
__global__ void __launch_bounds__(kTileThreads, 2) gemm_kernel(GemmArgs g) {
    __shared__ TileLds<T, TM, TN> lds;
    typedef typename Cx<T>::type C2;
    const int job = blockIdx.y, split = blockIdx.z;
    const int tilesM = (g.M + TM - 1) / TM;
    int tm, tn;
    tile_of(blockIdx.x, tilesM, gridDim.x / tilesM, tm, tn);
    const int m0 = tm * TM, n0 = tn * TN;
    if (tile_skipped(g, g.job0 + job, m0, n0, TM, TN)) return;
    const int sb = g.segBeg[job], se = g.segBeg[job + 1];
    const i64 nsteps = (i64)(se - sb) * ((g.K + kGroupTK - 1) / kGroupTK);
    const int t0 = (int)(nsteps * split / g.ksplit), t1 = (int)(nsteps * (split + 1) / g.ksplit);
    const float js = g.jscale ? g.jscale[g.job0 + job] : 1.0f;
    C2 *dense = g.ksplit > 1 ? reinterpret_cast<C2 *>(g.part) + ((i64)split * g.njobs_all + g.job0 + job) * g.M * g.N
                             : nullptr;
    tile_product<T, TM, TN, WTM, WTN, TRI>(g, lds, m0, n0, sb, t0, t1, js, g.beta,
                                           reinterpret_cast<C2 *>(g.C) + g.offC[job], dense);
}

template <typename T, int TM, int TN, int WTM, int WTN>
hipError_t launch_shape(const GemmArgs &g, hipStream_t s) {
    const int tilesM = (g.M + TM - 1) / TM, tilesN = (g.N + TN - 1) / TN;
    // grid.y is limited to 65535: launch the job list in chunks
    for (int j0 = 0; j0 < g.njobs; j0 += 65535) {
        GemmArgs c = g;
        c.njobs = (g.njobs - j0 < 65535) ? g.njobs - j0 : 65535;
        c.offC = g.offC + j0;
        c.segBeg = g.segBeg + j0;
        c.job0 = j0;
        const dim3 grid(tilesM * tilesN, c.njobs, g.ksplit);
        auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(kTileThreads), 0, s, c); };
        if (g.kind == 1) {
            if (g.sk.tri) go(gemm_kernel<T, TM, TN, WTM, WTN, 1, true>);
            else go(gemm_kernel<T, TM, TN, WTM, WTN, 1, false>);
        } else {
            if (g.sk.tri) go(gemm_kernel<T, TM, TN, WTM, WTN, 0, true>);
            else go(gemm_kernel<T, TM, TN, WTM, WTN, 0, false>);
        }
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// C[job](m, n) = alpha * sum_split part[split][job][m][n] (+ C), splits summed in order
template <typename T>
__global__ void k_gemm_reduce(GemmArgs g) {
    typedef typename Cx<T>::type C2;
    const C2 *P = reinterpret_cast<const C2 *>(g.part);
    C2 *C = reinterpret_cast<C2 *>(g.C);
    const i64 per = (i64)g.M * g.N, n = (i64)g.njobs * per;
    for (i64 t = blockIdx.x * (i64)blockDim.x + threadIdx.x; t < n; t += (i64)gridDim.x * blockDim.x) {
        const int job = (int)(t / per);
        const T js = g.jscale ? (T)g.jscale[job] : (T)1;
        const T alr = js * (T)g.alpha_re, ali = js * (T)g.alpha_im;
        const int gm = (int)((t % per) / g.N), gn = (int)(t % g.N);
        T xr = 0, xi = 0;
        for (int z = 0; z < g.ksplit; ++z) {
            const C2 v = P[(i64)z * n + t];
            xr += v.x;
            xi += v.y;
        }
        T vr = alr * xr - ali * xi, vi = alr * xi + ali * xr;
        const i64 off = g.offC[job] + split_off(gm, g.sm, g.Cm) + split_off(gn, g.sn, g.Cn);
        if (g.beta) { C2 o = C[off]; vr += o.x; vi += o.y; }
        C2 w; w.x = vr; w.y = vi;
        C[off] = w;
    }
}

int gemm_shape(const GemmArgs &g, bool fp64) {
    return g.shape >= 0 ? g.shape : best_tile(g.M, g.N, g.K, 1, fp64, false);
}

// The tile with the least work, edges included: a step costs its matrix instructions and, once per step,
// about half a fragment's time for loads and the barrier; 64x64 first, which reads its operands half as
// often, unless another saves a tenth.
int best_tile(int M, int N, int K, i64 jobs, bool fp64, bool fill) {
    // complex64: the bf16 products need a reduction that fills most of a 32-deep step and tiles that are
    // not mostly edge (Nk=5, o=8, v=40, 48 right-hand sides: M=3072 N=1600 K=28 0.43 against 0.49 ms of
    // 64x64, M=122880 N=40 K=40 3.4 against 4.6, M=3072 N=28 K=1600 0.44 against 0.52; but
    // M=2560 N=1920 K=8 2.2 against 2.0, M=64 N=76800 K=64 1.17 against 1.13)
    const GroupTile &sp = kGroupTiles[kSplitTile];
    if (!fp64 && K >= 24 && M >= 96 && N >= 24 && !(fill && jobs * ((M + sp.m - 1) / sp.m) * ((N + sp.n - 1) / sp.n) < 256))
        return kSplitTile;
    int tile = -1;
    double best = 0;
    for (int t : {1, 0, 2, 3}) {
        const GroupTile &gt = kGroupTiles[t];
        const i64 n = jobs * ((M + gt.m - 1) / gt.m) * ((N + gt.n - 1) / gt.n);
        const double w = (double)n * (gt.frags + 0.5);
        // fill: 64x64 only where its tiles fill the 256 compute units by themselves
        if (fill && gt.frags > 1 && n < 512) continue;
        if (tile >= 0 && w >= 0.9 * best) continue;
        best = w;
        tile = t;
    }
    return tile;
}

std::vector<int> gemm_candidates(const GemmArgs &g, bool fp64) {
    GemmArgs h = g;
    h.shape = -1;
    std::vector<int> c{gemm_shape(h, fp64)};
    for (int s : {(int)kSplitTile, 1, 0, 2, 3}) {
        if (s == kSplitTile && (fp64 || g.M < 32 || g.N < 16)) continue;
        if (c.size() < 3 && std::find(c.begin(), c.end(), s) == c.end()) c.push_back(s);
    }
    return c;
}

template <typename T>
hipError_t launch_gemm(const GemmArgs &g, hipStream_t s) {
    if (g.njobs <= 0 || g.M <= 0 || g.N <= 0) return hipSuccess;
    constexpr bool f64 = sizeof(T) == 8;
    hipError_t e;
    switch (gemm_shape(g, f64)) {
    case 0: e = launch_shape<T, 32, 32, 16, 16>(g, s); break;
    case 1: e = launch_shape<T, 64, 64, 32, 32>(g, s); break;
    case 2: e = launch_shape<T, 16, 64, 16, 16>(g, s); break;
    case 3: e = launch_shape<T, 64, 16, 16, 16>(g, s); break;
    case kSplitTile:
        if constexpr (f64) e = hipErrorInvalidValue;
        else e = launch_gemm_split(g, s);
        break;
    default: return hipErrorInvalidValue;
    }
    if (e != hipSuccess || g.ksplit <= 1) return e;
    const i64 n = (i64)g.njobs * g.M * g.N;
    const unsigned blocks = (unsigned)std::min<i64>((n + 255) / 256, 65535);
    hipLaunchKernelGGL(k_gemm_reduce<T>, dim3(blocks), dim3(256), 0, s, g);
    return hipGetLastError();
}

template hipError_t launch_gemm<double>(const GemmArgs &, hipStream_t);
template hipError_t launch_gemm<float>(const GemmArgs &, hipStream_t);

}  // namespace lrcc
