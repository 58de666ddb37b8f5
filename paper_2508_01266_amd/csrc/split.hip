// complex64 products on the bf16 matrix cores.
//
// Every fp32 operand x is the sum of three bf16 numbers, x = h + m + l, up to 2^-25 |x| (h, m, l the
// roundings of x and of what is left), and a product is formed from six bf16 products with fp32
// accumulation, small ones first: h l + l h + m m + m h + h m + h h.  The terms left out (m l, l m, l l)
// are below 2^-24 |a b|.  The matrix cores run bf16 16 times as fast as fp32, so six products leave a
// factor of 2.7; a complex product takes 24 of them.  An operand that rounds to an infinite bf16 number (above
// 3.396e38, or infinite) has no such parts and leaves NaN: a tile with a sum that is not finite is formed again
// by tile_product, so that it holds what the fp32 matrix cores give (all NaN, Nk=2, o=8, v=40, 24 vectors: 5.4 ms
// against 3.1 of ordinary numbers).  An operand below 2^-110 = 8e-34 loses the bits of its parts under the
// smallest bf16 number, 2^-133.
#include "tile.hpp"

namespace lrcc {

namespace {
constexpr int NT = 256;
typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef float f2 __attribute__((ext_vector_type(2)));
typedef float v4 __attribute__((ext_vector_type(4)));
typedef unsigned u4 __attribute__((ext_vector_type(4)));
struct __attribute__((aligned(8))) c64x2 { float2 a, b; };   // two elements, 8-byte aligned

__device__ __forceinline__ v4 mma(bf8 a, bf8 b, v4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ unsigned bits(bf2 x) { return __builtin_bit_cast(unsigned, x); }

// the three bf16 parts of eight values (pairs packed in order)
__device__ __forceinline__ void split8(const float *x, u4 &h, u4 &m, u4 &l) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const f2 v = {x[2 * i], x[2 * i + 1]};
        const bf2 a = __builtin_convertvector(v, bf2);
        const f2 r = v - __builtin_convertvector(a, f2);
        const bf2 b = __builtin_convertvector(r, bf2);
        const f2 q = r - __builtin_convertvector(b, f2);
        h[i] = bits(a);
        m[i] = bits(b);
        l[i] = bits(__builtin_convertvector(q, bf2));
    }
}
}  // namespace

// 128x64 tiles, 32-deep steps, four waves of 64x32; an LDS unit is eight consecutive reduction elements
// of one row of one part (re/im x h/m/l), the operand of one 16x16x32 instruction per lane.  75 KB of LDS
// and under 256 registers: two workgroups per compute unit, so that one converts while the other
// multiplies.  Operands are loaded one step ahead, eight elements of a row per thread.
// RUN: every unit lies in one run of the reduction index (its innermost extent is a multiple of 8).
// Steps [t0, t1) of the (segment, k) range that starts at segment sb, then the outputs as tile_product's.
constexpr int STM = 128, STN = 64, STK = 32, SKG = STK / 8;
// the k groups of a row start 8 banks apart
constexpr int SSA = STM + 2, SSB = STN + 2;
struct SplitLds { u4 a[6 * SKG * SSA], b[6 * SKG * SSB]; };
static_assert(sizeof(TileLds<float, 64, 64>) <= sizeof(SplitLds), "LDS of the tiles formed again");

// The tile on the fp32 matrix cores.  A function of its own, never inlined: in the kernels' body it costs the
// main loop its scalar registers (Nk=3, o=10, v=60, 6 vectors, transposed: 24.1 ms inlined, 22.2 so, 22.0 without
// the check; Nk=5, o=8, v=40, 48 vectors: 112.6, 107.2 and 106.9).
__device__ __attribute__((noinline)) void form_again(const GemmArgs *gp, SplitLds *lds, int m0, int n0, int sb, int tbeg,
                                                     int tend, float js, int beta, void *Cblock, float2 *dense) {
    const GemmArgs &g = *gp;
    const int ksteps = (g.K + STK - 1) / STK, k16 = (g.K + kGroupTK - 1) / kGroupTK;
    auto at = [&](int t) {                          // step t of 32 in steps of 16
        const int s = t / (ksteps > 0 ? ksteps : 1), left = 2 * (t - s * ksteps);
        return s * k16 + (left < k16 ? left : k16);
    };
    for (int h = 0; h < STM; h += 64) {
        tile_product<float, 64, 64, 32, 32, true>(g, *reinterpret_cast<TileLds<float, 64, 64> *>(lds), m0 + h, n0, sb,
                                                  at(tbeg), at(tend), js, beta, Cblock, dense);
        __syncthreads();
    }
}

template <bool RUN>
__device__ __forceinline__ void split_tile(const GemmArgs &g, const GemmArgs *gp, SplitLds &lds, int m0, int n0, int sb, int tbeg, int tend,
                                           float js, int beta, void *Cblock, float2 *dense) {
    constexpr int TM = STM, TN = STN, TK = STK, KG = SKG, SA = SSA, SB = SSB;
    constexpr int FM = 4, FN = 2, UA = TM * KG / NT, UB = TN * KG / NT;
    u4 *const lA = lds.a, *const lB = lds.b;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = (wave & 1) * 64, wn = (wave >> 1) * 32;
    const float2 *A = reinterpret_cast<const float2 *>(g.A);
    const float2 *B = reinterpret_cast<const float2 *>(g.B);
    const int ak0 = (int)g.Ak.s[0], ak1 = (int)g.Ak.s[1], ak2 = (int)g.Ak.s[2];
    const int bk0 = (int)g.Bk.s[0], bk1 = (int)g.Bk.s[1], bk2 = (int)g.Bk.s[2];
    int arow[UA], akg[UA], am[UA], bcol[UB], bkg[UB], bn[UB];
    bool aok[UA], bok[UB];
#pragma unroll
    for (int q = 0; q < UA; ++q) {
        const int idx = tid + NT * q;
        if (g.aMfast) { am[q] = idx % TM; akg[q] = idx / TM; } else { akg[q] = idx % KG; am[q] = idx / KG; }
        const int gm = m0 + am[q];
        aok[q] = gm < g.M;
        arow[q] = aok[q] ? split_off32(gm, g.sm, (int)g.Am.s[0], (int)g.Am.s[1], (int)g.Am.s[2]) : 0;
    }
#pragma unroll
    for (int q = 0; q < UB; ++q) {
        const int idx = tid + NT * q;
        if (g.bNfast) { bn[q] = idx % TN; bkg[q] = idx / TN; } else { bkg[q] = idx % KG; bn[q] = idx / KG; }
        const int gn = n0 + bn[q];
        bok[q] = gn < g.N;
        bcol[q] = bok[q] ? split_off32(gn, g.sn, (int)g.Bn.s[0], (int)g.Bn.s[1], (int)g.Bn.s[2]) : 0;
    }
    v4 accr[FM][FN], acci[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) { accr[i][j] = v4{0, 0, 0, 0}; acci[i][j] = v4{0, 0, 0, 0}; }

    const int ksteps = (g.K + TK - 1) / TK;
    float2 va[UA][8], vb[UB][8];
    auto unit = [&](const float2 *P, int row, bool ok, int k, int s0, int s1, int s2, float2 *v) {
        if (RUN) {
            if (ok && k < g.K) {
                const float2 *p = P + row + split_off32<false>(k, g.sk, s0, s1, s2);
                if (s2 == 1) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const c64x2 w = *reinterpret_cast<const c64x2 *>(p + 2 * i);
                        v[2 * i] = w.a;
                        v[2 * i + 1] = w.b;
                    }
                } else {
#pragma unroll
                    for (int i = 0; i < 8; ++i) v[i] = p[i * s2];
                }
            } else {
#pragma unroll
                for (int i = 0; i < 8; ++i) v[i] = make_float2(0, 0);
            }
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i)
                v[i] = ok && k + i < g.K ? P[row + split_off32<true>(k + i, g.sk, s0, s1, s2)] : make_float2(0, 0);
        }
    };
    int ps = sb + tbeg / (ksteps > 0 ? ksteps : 1), pk = tbeg % (ksteps > 0 ? ksteps : 1);   // next step to load
    auto fetch = [&]() {
        const int k0 = pk * TK;
        const float2 *As = A + g.segA[ps];
        const float2 *Bs = B + g.segB[ps];
        if (++pk == ksteps) { pk = 0; ++ps; }
#pragma unroll
        for (int q = 0; q < UA; ++q) unit(As, arow[q], aok[q], k0 + 8 * akg[q], ak0, ak1, ak2, va[q]);
#pragma unroll
        for (int q = 0; q < UB; ++q) unit(Bs, bcol[q], bok[q], k0 + 8 * bkg[q], bk0, bk1, bk2, vb[q]);
    };
    auto put = [&](const float2 *v, u4 *l, int stride, int at) {
        float x[8], y[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) { x[i] = v[i].x; y[i] = v[i].y; }
        u4 p[3];
        split8(x, p[0], p[1], p[2]);
#pragma unroll
        for (int c = 0; c < 3; ++c) l[c * KG * stride + at] = p[c];
        split8(y, p[0], p[1], p[2]);
#pragma unroll
        for (int c = 0; c < 3; ++c) l[(3 + c) * KG * stride + at] = p[c];
    };
    if (tbeg < tend) fetch();
    for (int t = tbeg; t < tend; ++t) {
#pragma unroll
        for (int q = 0; q < UA; ++q) put(va[q], lA, SA, akg[q] * SA + am[q]);
#pragma unroll
        for (int q = 0; q < UB; ++q) put(vb[q], lB, SB, bkg[q] * SB + bn[q]);
        __syncthreads();
        if (t + 1 < tend) fetch();
        const int kg = lane >> 4, c = lane & 15;
        bf8 b[FN][6];
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int p = 0; p < 6; ++p)
                b[j][p] = __builtin_bit_cast(bf8, lB[(p * KG + kg) * SB + wn + 16 * j + c]);
#pragma unroll
        for (int i = 0; i < FM; ++i) {
            bf8 a[6], na[3];
#pragma unroll
            for (int p = 0; p < 6; ++p) {
                const u4 w = lA[(p * KG + kg) * SA + wm + 16 * i + c];
                a[p] = __builtin_bit_cast(bf8, w);
                if (p >= 3) na[p - 3] = __builtin_bit_cast(bf8, w ^ u4{0x80008000u, 0x80008000u, 0x80008000u, 0x80008000u});
            }
            // The six products of a step, small ones first, are summed apart and added to the running sum once: an
            // instruction rounds its accumulator every four elements, 16 times a step, and at the size of one
            // step's sum those roundings do not count.  Relative error of a random reduction of 40, 1600 and 98304
            // elements: 5.0e-8, 1.4e-7, 1.0e-6; with h h added to the running sum directly 5.8e-8, 3.6e-7,
            // 3.1e-6; on the fp32 tiles, whose running sums move to a second set every 128 elements, 1.6e-7, 2.9e-7,
            // 5.9e-7 (here the second set would not fit the registers), and without that 1.6e-7, 1.0e-6, 7.8e-6.
            constexpr int pa[6] = {0, 2, 1, 1, 0, 0}, pb[6] = {2, 0, 1, 0, 1, 0};
            v4 lr[FN], li[FN];
#pragma unroll
            for (int j = 0; j < FN; ++j) { lr[j] = v4{0, 0, 0, 0}; li[j] = v4{0, 0, 0, 0}; }
#pragma unroll
            for (int q = 0; q < 6; ++q) {
#pragma unroll
                for (int j = 0; j < FN; ++j) {
                    lr[j] = mma(a[pa[q]], b[j][pb[q]], lr[j]);
                    li[j] = mma(a[pa[q]], b[j][3 + pb[q]], li[j]);
                }
#pragma unroll
                for (int j = 0; j < FN; ++j) {
                    lr[j] = mma(na[pa[q]], b[j][3 + pb[q]], lr[j]);
                    li[j] = mma(a[3 + pa[q]], b[j][pb[q]], li[j]);
                }
            }
#pragma unroll
            for (int j = 0; j < FN; ++j) { accr[i][j] += lr[j]; acci[i][j] += li[j]; }
        }
        __syncthreads();
    }
    // 0 unless some sum is not finite; the LDS is free (the loop ends with a barrier)
    float nan = 0;
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) nan += accr[i][j][r] * 0.0f + acci[i][j][r] * 0.0f;
    unsigned *const again = reinterpret_cast<unsigned *>(lds.a);
    const bool any = __any(nan != 0.0f);            // (true for NaN)
    if (lane == 0) again[wave] = any;
    __syncthreads();
    if (again[0] | again[1] | again[2] | again[3]) {
        __syncthreads();
        form_again(gp, &lds, m0, n0, sb, tbeg, tend, js, beta, Cblock, dense);
        return;
    }
    if (dense) {
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int gm = m0 + wm + 16 * i + 4 * (lane >> 4) + r;
                    const int gn = n0 + wn + 16 * j + (lane & 15);
                    if (gm < g.M && gn < g.N) dense[(i64)gm * g.N + gn] = make_float2(accr[i][j][r], acci[i][j][r]);
                }
        return;
    }
    const float alr = js * (float)g.alpha_re, ali = js * (float)g.alpha_im;
    float2 *Cj = reinterpret_cast<float2 *>(Cblock);
    i64 coff[FN];
    bool cok[FN];
#pragma unroll
    for (int j = 0; j < FN; ++j) {
        const int gn = n0 + wn + 16 * j + (lane & 15);
        cok[j] = gn < g.N;
        coff[j] = cok[j] ? split_off(gn, g.sn, g.Cn) : 0;
    }
#pragma unroll
    for (int i = 0; i < FM; ++i) {
        i64 roff[4];
        bool rok[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int gm = m0 + wm + 16 * i + 4 * (lane >> 4) + r;
            rok[r] = gm < g.M;
            roff[r] = rok[r] ? split_off(gm, g.sm, g.Cm) : 0;
        }
        float2 old[FN][4];
        if (beta) {
            // all reads before the first write; (0, 0) of the block stands in for outside elements
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
                const float xr = accr[i][j][r], xi = acci[i][j][r];
                float2 w = make_float2(alr * xr - ali * xi, alr * xi + ali * xr);
                if (beta) { w.x += old[j][r].x; w.y += old[j][r].y; }
                Cj[roff[r] + coff[j]] = w;
            }
    }
}

template <bool RUN>
__global__ void __launch_bounds__(NT, 2) gemm_split_kernel(GemmArgs g) {
    __shared__ SplitLds lds;
    const int job = blockIdx.y, split = blockIdx.z;
    const int tilesM = (g.M + STM - 1) / STM;
    int tm, tn;
    tile_of(blockIdx.x, tilesM, gridDim.x / tilesM, tm, tn);
    const int m0 = tm * STM, n0 = tn * STN;
    if (tile_skipped(g, g.job0 + job, m0, n0, STM, STN)) return;
    const int sb = g.segBeg[job], se = g.segBeg[job + 1];
    const i64 nsteps = (i64)(se - sb) * ((g.K + STK - 1) / STK);
    const int tbeg = (int)(nsteps * split / g.ksplit), tend = (int)(nsteps * (split + 1) / g.ksplit);
    float2 *dense = g.ksplit > 1 ? reinterpret_cast<float2 *>(g.part) +
                                       ((i64)split * g.njobs_all + g.job0 + job) * g.M * g.N : nullptr;
    // (the arguments where the launch put them: the address of g would be that of a copy)
    const GemmArgs *const gp = (const GemmArgs *)__builtin_amdgcn_kernarg_segment_ptr();
    split_tile<RUN>(g, gp, lds, m0, n0, sb, tbeg, tend,
                    g.jscale ? g.jscale[g.job0 + job] : 1.0f, g.beta, reinterpret_cast<float2 *>(g.C) + g.offC[job], dense);
}

__device__ __host__ inline bool split_run(const GemmArgs &g) { return !g.sk.tri && g.sk.d2 % 8 == 0; }

// the same tiles over a table of work items (GroupItem)
__global__ void __launch_bounds__(NT, 2) gemm_split_group_kernel(const GemmArgs *__restrict__ ops,
                                                                 const GroupItem *__restrict__ items) {
    __shared__ SplitLds lds;
    const GroupItem it = items[blockIdx.x];
    const GemmArgs &g = ops[it.op];
    if (split_run(g)) split_tile<true>(g, &g, lds, it.m0, it.n0, it.sb, it.t0, it.t1, it.js, it.beta, it.C, nullptr);
    else split_tile<false>(g, &g, lds, it.m0, it.n0, it.sb, it.t0, it.t1, it.js, it.beta, it.C, nullptr);
}

hipError_t launch_split_group(const GemmArgs *ops, const GroupItem *items, int n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(gemm_split_group_kernel, dim3(n), dim3(NT), 0, s, ops, items);
    return hipGetLastError();
}

hipError_t launch_gemm_split(const GemmArgs &g, hipStream_t s) {
    const int tilesM = (g.M + STM - 1) / STM, tilesN = (g.N + STN - 1) / STN;
    const bool run = split_run(g);
    // grid.y is limited to 65535: launch the job list in chunks
    for (int j0 = 0; j0 < g.njobs; j0 += 65535) {
        GemmArgs c = g;
        c.njobs = (g.njobs - j0 < 65535) ? g.njobs - j0 : 65535;
        c.offC = g.offC + j0;
        c.segBeg = g.segBeg + j0;
        c.job0 = j0;
        const dim3 grid(tilesM * tilesN, c.njobs, g.ksplit);
        if (run) hipLaunchKernelGGL(gemm_split_kernel<true>, grid, dim3(NT), 0, s, c);
        else hipLaunchKernelGGL(gemm_split_kernel<false>, grid, dim3(NT), 0, s, c);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace lrcc
