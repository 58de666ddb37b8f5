// One output tile of a strided complex product on the matrix cores (device code shared by the single and
// the grouped launches).
#pragma once
#include "group.hpp"

namespace lrcc {

template <typename T> struct Mfma;
template <> struct Mfma<double> {
    typedef double v4 __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ v4 mma(double a, double b, v4 c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    // output row of accumulator register r held by `lane` (column = lane % 16)
    static __device__ __forceinline__ int row(int lane, int r) { return (lane >> 4) + 4 * r; }
};
template <> struct Mfma<float> {
    typedef float v4 __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ v4 mma(float a, float b, v4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int lane, int r) { return 4 * (lane >> 4) + r; }
};

constexpr int kTileThreads = 256;

// LDS of a tile: two buffers of each operand, complex elements interleaved (one wide read gives both
// parts), rows one element apart from a multiple of the banks; and the offsets of the reduction index.
template <typename T, int TM, int TN> struct TileLds {
    typename Cx<T>::type a[2][kGroupTK * (TM + 1)], b[2][kGroupTK * (TN + 1)];
    int koff[2][2][kGroupTK];
};

// Reduction steps [t0, t1) of the (segment, k) range that starts at segment sb, then the tile's outputs:
// C = js alpha sum (+ C with beta), or with `dense` the raw sums into dense[m][n].
//
// Four waves, each WTM x WTN; one barrier per step; operands are loaded two steps ahead, since one step of
// a small tile (16 to 64 matrix instructions per wave) is shorter than a trip to memory.  The offset of a
// reduction index (two divisions by the extents of its split) is formed once per step by 16 threads per
// operand and read from LDS: formed by every thread for every load it took 4.2 vector instructions per
// matrix instruction, and the fp64 matrix cores (64 cycles per instruction) were busy 64% of the time on
// the largest product.  Rows and columns outside the operands read row 0 instead of being masked: their
// sums are not stored.
template <typename T, int TM, int TN, int WTM, int WTN, bool TRI>
__device__ __forceinline__ void tile_product(const GemmArgs &g, TileLds<T, TM, TN> &lds, int m0, int n0, int sb, int t0,
                                             int t1, float js, int beta, void *Cblock, typename Cx<T>::type *dense) {
    typedef typename Cx<T>::type C2;
    typedef typename Mfma<T>::v4 v4;
    constexpr int TK = kGroupTK, NT = kTileThreads;
    constexpr int WGM = TM / WTM, FM = WTM / 16, FN = WTN / 16;
    constexpr int LA = TM * TK / NT, LB = TK * TN / NT;
    constexpr int SA = TM + 1, SB = TN + 1;
    static_assert((TM / WTM) * (TN / WTN) == 4, "4 waves per block");
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = (wave % WGM) * WTM, wn = (wave / WGM) * WTN;
    const C2 *A = reinterpret_cast<const C2 *>(g.A);
    const C2 *B = reinterpret_cast<const C2 *>(g.B);
    const bool aM = g.aMfast != 0, bN = g.bNfast != 0;
    int am[LA], ak[LA], bk[LB], bn[LB], arow[LA], bcol[LB];
#pragma unroll
    for (int q = 0; q < LA; ++q) {
        const int idx = tid + NT * q;
        if (aM) { am[q] = idx % TM; ak[q] = idx / TM; } else { ak[q] = idx % TK; am[q] = idx / TK; }
        const int gm = m0 + am[q];
        arow[q] = gm < g.M ? split_off32(gm, g.sm, (int)g.Am.s[0], (int)g.Am.s[1], (int)g.Am.s[2]) : 0;
    }
#pragma unroll
    for (int q = 0; q < LB; ++q) {
        const int idx = tid + NT * q;
        if (bN) { bn[q] = idx % TN; bk[q] = idx / TN; } else { bk[q] = idx % TK; bn[q] = idx / TK; }
        const int gn = n0 + bn[q];
        bcol[q] = gn < g.N ? split_off32(gn, g.sn, (int)g.Bn.s[0], (int)g.Bn.s[1], (int)g.Bn.s[2]) : 0;
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
    const bool ragged = g.K % TK != 0;
    int ps = sb + t0 / (ksteps > 0 ? ksteps : 1), pk = t0 % (ksteps > 0 ? ksteps : 1);   // next step to load
    C2 va[2][LA], vb[2][LB];
    // offsets of the step (ps, pk)'s reduction indices (0 past the end) into table `par`
    auto offsets = [&](int par) {
        if (tid < TK) {
            const int k = pk * TK + tid;
            lds.koff[par][0][tid] =
                k < g.K ? split_off32<TRI>(k, g.sk, (int)g.Ak.s[0], (int)g.Ak.s[1], (int)g.Ak.s[2]) : 0;
        } else if (tid >= 64 && tid < 64 + TK) {
            const int k = pk * TK + tid - 64;
            lds.koff[par][1][tid - 64] =
                k < g.K ? split_off32<TRI>(k, g.sk, (int)g.Bk.s[0], (int)g.Bk.s[1], (int)g.Bk.s[2]) : 0;
        }
    };
    // loads of step (ps, pk), then on to the next step
    auto fetch = [&](int par, C2 *ra, C2 *rb) {
        const C2 *As = A + g.segA[ps];
        const C2 *Bs = B + g.segB[ps];
#pragma unroll
        for (int q = 0; q < LA; ++q) ra[q] = As[arow[q] + lds.koff[par][0][ak[q]]];
#pragma unroll
        for (int q = 0; q < LB; ++q) rb[q] = Bs[bcol[q] + lds.koff[par][1][bk[q]]];
        if (ragged && pk == ksteps - 1) {
            const int left = g.K - pk * TK;
#pragma unroll
            for (int q = 0; q < LA; ++q)
                if (ak[q] >= left) { ra[q].x = 0; ra[q].y = 0; }
#pragma unroll
            for (int q = 0; q < LB; ++q)
                if (bk[q] >= left) { rb[q].x = 0; rb[q].y = 0; }
        }
        if (++pk == ksteps) { pk = 0; ++ps; }
    };
    // step t: its operands (loaded two steps before) to LDS, the offsets of step t + 2, the barrier, the
    // loads of step t + 2, the products
    auto step = [&](int par, bool more) {
        C2 *la = lds.a[par], *lb = lds.b[par];
#pragma unroll
        for (int q = 0; q < LA; ++q) la[ak[q] * SA + am[q]] = va[par][q];
#pragma unroll
        for (int q = 0; q < LB; ++q) lb[bk[q] * SB + bn[q]] = vb[par][q];
        if (more) offsets(par);
        __syncthreads();
        if (more) fetch(par, va[par], vb[par]);
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
                    accr[i][j] = Mfma<T>::mma(a[i].x, b[j].x, accr[i][j]);
                    acci[i][j] = Mfma<T>::mma(a[i].x, b[j].y, acci[i][j]);
                }
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j) {
                    accr[i][j] = Mfma<T>::mma(-a[i].y, b[j].y, accr[i][j]);
                    acci[i][j] = Mfma<T>::mma(a[i].y, b[j].x, acci[i][j]);
                }
        }
    };
    // LDS buffer and offset table `par` are written before the barrier of step t (t of parity par) and read
    // after it; the next writes come before the barrier of step t + 2, which a wave reaches only after
    // the barrier of step t + 1 and so after every wave's reads of step t
    if (t0 < t1) {
        offsets(0);
        __syncthreads();
        fetch(0, va[0], vb[0]);
        if (t0 + 1 < t1) {
            offsets(1);
            __syncthreads();
            fetch(1, va[1], vb[1]);
        }
        __syncthreads();
    }
    for (int t = t0; t < t1; t += 2) {
        step(0, t + 2 < t1);
        if (t + 1 < t1) step(1, t + 3 < t1);
        if (FLUSH && (t - t0) % kFlush == kFlush - 2) flush(false);
    }
    if constexpr (FLUSH) {
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j) { accr[i][j] += sumr[i][j]; acci[i][j] += sumi[i][j]; }
    }

    if (dense) {
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int gm = m0 + wm + 16 * i + Mfma<T>::row(lane, r);
                    const int gn = n0 + wn + 16 * j + (lane & 15);
                    if (gm < g.M && gn < g.N) {
                        C2 w;
                        w.x = accr[i][j][r];
                        w.y = acci[i][j][r];
                        dense[(i64)gm * g.N + gn] = w;
                    }
                }
        return;
    }
    const T alr = (T)js * (T)g.alpha_re, ali = (T)js * (T)g.alpha_im;
    C2 *Cj = reinterpret_cast<C2 *>(Cblock);
    i64 coff[FN];
    bool cok[FN];
#pragma unroll
    for (int j = 0; j < FN; ++j) {
        const int gn = n0 + wn + 16 * j + (lane & 15);
        cok[j] = gn < g.N;
        coff[j] = cok[j] ? split_off(gn, g.sn, g.Cn) : 0;
    }
    // one row of fragments at a time.  With beta all reads of C come, unconditionally, before the first
    // write: a write may alias a later read as far as the compiler knows, so read-add-write element by
    // element would wait out one memory round trip per element, which bounds the short-K products
#pragma unroll
    for (int i = 0; i < FM; ++i) {
        i64 roff[4];
        bool rok[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int gm = m0 + wm + 16 * i + Mfma<T>::row(lane, r);
            rok[r] = gm < g.M;
            roff[r] = rok[r] ? split_off(gm, g.sm, g.Cm) : 0;
        }
        C2 old[FN][4];
        if (beta) {
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r)   // (0, 0) of the block stands in for outside elements
                    old[j][r] = Cj[rok[r] && cok[j] ? roff[r] + coff[j] : 0];
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
                if (beta) { w.x += old[j][r].x; w.y += old[j][r].y; }
                Cj[roff[r] + coff[j]] = w;
            }
    }
}

}  // namespace lrcc
