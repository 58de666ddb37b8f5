// Streaming (HBM-bound) kernels of the sigma path: layout transposes between
// the caller's rhs-major layout and the internal k-block-major layout, the
// amplitude products entering tau (Eq. t2 and the perturbed analogue), the
// final P_IJ P_AB antisymmetrisation with the -omega shift, Cholesky slices,
// and precision conversion.  Grid-stride loops (over elements, or over rows of
// the doubles arrays for the per-sigma kernels); consecutive threads touch
// consecutive elements of the innermost (unit-stride) index.
#include "common.hpp"
#include "elem.hpp"

#include <algorithm>

namespace lrcc {

namespace {
inline unsigned grid_for(i64 n, int bs = 256) {
    i64 g = (n + bs - 1) / bs;
    if (g > 65536 * 4) g = 65536 * 4;
    if (g < 1) g = 1;
    return (unsigned)g;
}
template <typename T> __device__ inline typename Cx<T>::type mk(T x, T y) {
    typename Cx<T>::type r; r.x = x; r.y = y; return r;
}
// Row-wise launches: a workgroup takes whole rows of `len` consecutive elements, so the
// row index (the same for every lane) is split with 64-bit arithmetic once per row and
// the position inside the row with 32-bit arithmetic; splitting a flat 64-bit element
// index with 64-bit divisions costs more than the memory traffic of these kernels.
// Many short rows (up to 512 elements) go to a wave each: a workgroup of four waves spends longer on starting
// and on splitting the row's index than on its 256 elements.  2x2x2 mesh, o=4, v=16, 12 complex64 vectors (98304
// rows): inputs 0.365 -> 0.155 ms (805 MB), outputs 0.45 -> 0.28 ms.  Few rows leave the device idle that way:
// one k point, o=4, v=12 (144 rows): a product 62 -> 69 us; Nk=3, o=4, v=20 (5184 rows): 601 -> 616 us.
inline bool wave_rows(i64 rows, int v) { return (i64)v * v <= 512 && rows >= 32768; }
inline unsigned rows_grid(i64 rows) {
    return (unsigned)std::max<i64>(1, std::min<i64>(rows, 65536 * 4));
}
}

// out[b][r][e] = scale * in[r][b][e]
template <typename Tin, typename Tout>
__global__ void k_rhs_to_block(const typename Cx<Tin>::type *in, typename Cx<Tout>::type *out,
                               int R, i64 B, i64 E, double scale) {
    // rows (b, r) of the output, E elements each (E < 2^31, checked by the launcher)
    const i64 rows = (i64)R * B;
    for (i64 row = blockIdx.x; row < rows; row += gridDim.x) {
        const int r = (int)(row % R);
        const i64 b = row / R;
        const typename Cx<Tin>::type *src = in + ((i64)r * B + b) * E;
        typename Cx<Tout>::type *dst = out + row * E;
        for (int e = threadIdx.x; e < (int)E; e += blockDim.x) {
            auto v = src[e];
            dst[e] = mk<Tout>((Tout)(scale * v.x), (Tout)(scale * v.y));
        }
    }
}

template <typename Tin, typename Tout>
hipError_t rhs_to_block(const void *in, void *out, int R, i64 B, i64 E, double scale, hipStream_t s) {
    if (E >= ((i64)1 << 31)) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_rhs_to_block<Tin, Tout>), dim3(rows_grid((i64)R * B)), dim3(256), 0, s,
                       (const typename Cx<Tin>::type *)in, (typename Cx<Tout>::type *)out, R, B, E, scale);
    return hipGetLastError();
}

// out = x2 + c * (x_ia t_jb + t_ia x_jb - x_ib t_ja - t_ib x_ja), k-blocked, rhs inside the block.
// x1 [nk][R][o][v], t1 [nk][o][v], x2/out [nk^3][R][o][o][v][v]
template <typename T>
__global__ void k_tau_like(const typename Cx<T>::type *x1, const typename Cx<T>::type *x2,
                           const typename Cx<T>::type *t1, typename Cx<T>::type *out,
                           KMesh km, int R, int o, int v, T c, int x1_has_rhs) {
    const int nk = km.size(), vv = v * v;
    const i64 rows = (i64)nk * nk * nk * R * o * o;
    for (i64 row = blockIdx.x; row < rows; row += gridDim.x) {
        // row = (((ki nk + kj) nk + ka) R + r) o + i) o + j, elements (a, b)
        i64 q = row;
        const int j = take(q, o);
        const int i = take(q, o);
        const int r = take(q, R);
        const int ka = take(q, nk);
        const int kj = take(q, nk);
        const int ki = (int)q;
        const int kb = km.comb(ki, kj, ka);
        const int rx = x1_has_rhs ? r : 0;
        const int Rx = x1_has_rhs ? R : 1;
        auto X = [&](int k, int ii, int aa) { return x1[(((i64)k * Rx + rx) * o + ii) * v + aa]; };
        auto Tt = [&](int k, int ii, int aa) { return t1[((i64)k * o + ii) * v + aa]; };
        const typename Cx<T>::type *src = x2 + row * vv;
        typename Cx<T>::type *dst = out + row * vv;
        for (int e = threadIdx.x; e < vv; e += blockDim.x) {
            const int a = e / v, b = e - a * v;
            auto acc = src[e];
            T sr = 0, si = 0;
            if (ka == ki) {     // x_ia t_jb + t_ia x_jb  (kb == kj)
                auto p = X(ki, i, a), q2 = Tt(kj, j, b), u = Tt(ki, i, a), w = X(kj, j, b);
                sr += p.x * q2.x - p.y * q2.y + u.x * w.x - u.y * w.y;
                si += p.x * q2.y + p.y * q2.x + u.x * w.y + u.y * w.x;
            }
            if (kb == ki) {     // - x_ib t_ja - t_ib x_ja  (ka == kj)
                auto p = X(ki, i, b), q2 = Tt(kj, j, a), u = Tt(ki, i, b), w = X(kj, j, a);
                sr -= p.x * q2.x - p.y * q2.y + u.x * w.x - u.y * w.y;
                si -= p.x * q2.y + p.y * q2.x + u.x * w.y + u.y * w.x;
            }
            dst[e] = mk<T>(acc.x + c * sr, acc.y + c * si);
        }
    }
}

template <typename T>
hipError_t tau_like(const void *x1, const void *x2, const void *t1, void *out, KMesh km, int R, int o, int v,
                    double c, int x1_has_rhs, hipStream_t s) {
    const int nk = km.size();
    const i64 rows = (i64)nk * nk * nk * R * o * o;
    hipLaunchKernelGGL(k_tau_like<T>, dim3(rows_grid(rows)), dim3(256), 0, s,
                       (const typename Cx<T>::type *)x1, (const typename Cx<T>::type *)x2,
                       (const typename Cx<T>::type *)t1, (typename Cx<T>::type *)out, km, R, o, v, (T)c,
                       x1_has_rhs);
    return hipGetLastError();
}

// Inputs of the forward product in one pass over x2: x1 and x2 from the caller's layout into the blocks'
// (doubles scaled by `scale`), and dtau = x2 + x_ia t_jb + t_ia x_jb - x_ib t_ja - t_ib x_ja.  Bound by HBM;
// as three kernels x2 was read twice and the smallest programs waited on three launches (batched complex64
// input, Nk=5, o=8, v=40, 48 right-hand sides: 2.9 + 2.1 ms before, 3.7 ms now).
template <typename T>
__global__ void k_inputs(const double2 *x1, const double2 *x2, const typename Cx<T>::type *t1,
                         typename Cx<T>::type *o1, typename Cx<T>::type *o2, typename Cx<T>::type *dtau, KMesh km,
                         int R, int o, int v, double scale, i64 rows, unsigned b1) {
    const int nk = km.size(), vv = v * v;
    const int lane = threadIdx.x, lanes = blockDim.x, ty = threadIdx.y, ny = blockDim.y;   // ny rows at a time
    if (blockIdx.x < b1) {      // singles
        const i64 E = (i64)o * v, n = (i64)R * nk * E;
        for (i64 t = ((i64)blockIdx.x * ny + ty) * lanes + lane; t < n; t += (i64)b1 * ny * lanes) {
            const i64 e = t % E;
            const int k = (int)((t / E) % nk), r = (int)(t / (E * nk));
            const double2 x = x1[t];
            o1[((i64)k * R + r) * E + e] = mk<T>((T)x.x, (T)x.y);
        }
        return;
    }
    const i64 B = (i64)nk * nk * nk;
    for (i64 row = (i64)(blockIdx.x - b1) * ny + ty; row < rows; row += (i64)(gridDim.x - b1) * ny) {
        // row = (((ki nk + kj) nk + ka) R + r) o + i) o + j of the block layout, elements (a, b)
        i64 q = row;
        const int j = take(q, o);
        const int i = take(q, o);
        const int r = (int)(q % R);
        const i64 blk = q / R;
        const int ka = (int)(blk % nk), kj = (int)((blk / nk) % nk), ki = (int)(blk / (nk * nk));
        const int kb = km.comb(ki, kj, ka);
        auto X = [&](int k, int ii, int aa) {
            const double2 x = x1[(((i64)r * nk + k) * o + ii) * v + aa];
            return mk<T>((T)x.x, (T)x.y);
        };
        auto Tt = [&](int k, int ii, int aa) { return t1[((i64)k * o + ii) * v + aa]; };
        const double2 *src = x2 + ((((i64)r * B + blk) * o + i) * o + j) * vv;
        typename Cx<T>::type *d2 = o2 + row * vv, *dt = dtau + row * vv;
#pragma unroll 4
        for (int e = lane; e < vv; e += lanes) {
            const double2 in = src[e];
            const auto x = mk<T>((T)(scale * in.x), (T)(scale * in.y));
            d2[e] = x;
            const int a = e / v, b = e - a * v;
            T sr = 0, si = 0;
            if (ka == ki) {     // x_ia t_jb + t_ia x_jb  (kb == kj)
                auto p = X(ki, i, a), q2 = Tt(kj, j, b), u = Tt(ki, i, a), w = X(kj, j, b);
                sr += p.x * q2.x - p.y * q2.y + u.x * w.x - u.y * w.y;
                si += p.x * q2.y + p.y * q2.x + u.x * w.y + u.y * w.x;
            }
            if (kb == ki) {     // - x_ib t_ja - t_ib x_ja  (ka == kj)
                auto p = X(ki, i, b), q2 = Tt(kj, j, a), u = Tt(ki, i, b), w = X(kj, j, a);
                sr -= p.x * q2.x - p.y * q2.y + u.x * w.x - u.y * w.y;
                si -= p.x * q2.y + p.y * q2.x + u.x * w.y + u.y * w.x;
            }
            dt[e] = mk<T>(x.x + sr, x.y + si);
        }
    }
}

template <typename T>
hipError_t inputs(const void *x1, const void *x2, const void *t1, void *o1, void *o2, void *dtau, KMesh km, int R,
                  int o, int v, double scale, hipStream_t s) {
    const int nk = km.size();
    const i64 rows = (i64)nk * nk * nk * R * o * o;
    const unsigned b1 = (unsigned)std::min<i64>(((i64)R * nk * o * v + 255) / 256, 1024);
    const dim3 block = wave_rows(rows, v) ? dim3(64, 4) : dim3(256, 1);
    hipLaunchKernelGGL(k_inputs<T>, dim3(b1 + rows_grid((rows + block.y - 1) / block.y)), block, 0, s, (const double2 *)x1,
                       (const double2 *)x2, (const typename Cx<T>::type *)t1, (typename Cx<T>::type *)o1,
                       (typename Cx<T>::type *)o2, (typename Cx<T>::type *)dtau, km, R, o, v, scale, rows, b1);
    return hipGetLastError();
}

// One orbit of the antisymmetriser P(ij)P(ab): the four rows 0: (ki,kj,ka,i,j), 1: (kj,ki,ka,j,i),
// 2: (ki,kj,kb,i,j), 3: (kj,ki,kb,j,i) of an array read by ld(row, e) become A, -A, -A^T and A^T with
// A = row0 - row1 - (row2 - row3)^T (transposes in (a, b)), handed to st(row, e, value).  The workgroup
// takes the rows tile by tile: the differences row0 - row1 of tile (a, b) and row2 - row3 of tile (b, a)
// go through LDS, so every element is read once, along its unit-stride index, and both A and -A^T are
// written along theirs.  Where ka = kb rows 2 and 3 are rows 0 and 1: the tiles a0 <= b0 then make the whole
// row, so that in every orbit an element is read and written in the step of one tile alone and `st` may write
// the array that `ld` reads.  Bound by HBM.  (Reading the transposed elements from memory instead, twice,
// ran at 3.6 TB/s on the batched complex64 output, v = 40, and below 1 TB/s at v = 60 with two summands,
// whose rows do not stay in the L1 cache.)
constexpr int kOrbTile = 32;
// tiles of at most 32x32, the same size over the row, and their LDS (two arrays, rows one element apart
// from the tile's width): as little as the row needs, so that workgroups of short rows share a compute unit
__host__ __device__ inline int orbit_tile(int v) {
    const int nt = (v + kOrbTile - 1) / kOrbTile;
    return (v + nt - 1) / nt;
}
inline size_t orbit_lds(int v) { return (size_t)2 * orbit_tile(v) * (orbit_tile(v) + 1) * sizeof(double2); }
template <typename Ld, typename St>
__device__ __forceinline__ void orbit_rows(double2 *lds, int v, bool two_pairs, bool two_blocks, Ld ld, St st) {
    const int ts = orbit_tile(v), w = ts + 1;
    double2 *const ld0 = lds, *const ld1 = lds + ts * w;
    for (int a0 = 0; a0 < v; a0 += ts)
        for (int b0 = two_blocks ? 0 : a0; b0 < v; b0 += ts) {
            const bool both = two_blocks || a0 != b0;
            const int na = min(ts, v - a0), nb = min(ts, v - b0), n = na * nb;
#pragma unroll 4
            for (int e = threadIdx.x; e < n; e += blockDim.x) {
                const int a = e / nb, b = e - a * nb, at = (a0 + a) * v + b0 + b;
                const double2 p = ld(0, at, a0 + a, b0 + b), q = ld(1, at, a0 + a, b0 + b);
                ld0[a * w + b] = make_double2(p.x - q.x, p.y - q.y);
            }
#pragma unroll 4
            for (int e = threadIdx.x; e < n; e += blockDim.x) {
                const int b = e / na, a = e - b * na, at = (b0 + b) * v + a0 + a;
                const double2 p = ld(2, at, a0 + a, b0 + b), q = ld(3, at, a0 + a, b0 + b);
                ld1[b * w + a] = make_double2(p.x - q.x, p.y - q.y);
            }
            __syncthreads();
#pragma unroll 4
            for (int e = threadIdx.x; e < n; e += blockDim.x) {
                const int a = e / nb, b = e - a * nb, at = (a0 + a) * v + b0 + b;
                const double2 x = ld0[a * w + b], y = ld1[b * w + a];
                const double2 z = make_double2(x.x - y.x, x.y - y.y);
                st(0, at, a0 + a, b0 + b, z);
                if (two_pairs) st(1, at, a0 + a, b0 + b, make_double2(-z.x, -z.y));
            }
            if (both) {
#pragma unroll 4
                for (int e = threadIdx.x; e < n; e += blockDim.x) {
                    const int b = e / na, a = e - b * na, at = (b0 + b) * v + a0 + a;
                    const double2 x = ld0[a * w + b], y = ld1[b * w + a];
                    const double2 z = make_double2(x.x - y.x, x.y - y.y);
                    st(2, at, a0 + a, b0 + b, make_double2(-z.x, -z.y));
                    if (two_pairs) st(3, at, a0 + a, b0 + b, z);
                }
            }
            __syncthreads();
        }
}

// value at `at` of the sum of l.n arrays (NS of them, or any number for NS = 0), summed in double
template <typename T, int NS>
__device__ __forceinline__ double2 slab_sum(const SlabList &l, i64 at) {
    typedef typename Cx<T>::type C2;
    const C2 z0 = reinterpret_cast<const C2 *>(l.p[0])[at];
    double2 z = make_double2((double)z0.x, (double)z0.y);
    if constexpr (NS == 0) {
        int s = 1;
        for (; s + 4 <= l.n; s += 4) {     // four loads in flight
            C2 t[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) t[u] = reinterpret_cast<const C2 *>(l.p[s + u])[at];
#pragma unroll
            for (int u = 0; u < 4; ++u) { z.x += (double)t[u].x; z.y += (double)t[u].y; }
        }
        for (; s < l.n; ++s) {
            const C2 t = reinterpret_cast<const C2 *>(l.p[s])[at];
            z.x += (double)t.x;
            z.y += (double)t.y;
        }
    } else {
#pragma unroll
        for (int s = 1; s < NS; ++s) {
            const C2 t = reinterpret_cast<const C2 *>(l.p[s])[at];
            z.x += (double)t.x;
            z.y += (double)t.y;
        }
    }
    return z;
}

// Outputs of a product in the caller's layout, one launch:
//   y1[r][k][i][a] = s1[k][r][i][a] - omega_r x1[r][k][i][a];
//   y2[r][ki,kj,ka][i][j][a][b] = scale * (P_ij P_ab Z)[ki,kj,ka][r][i][j][a][b] - omega_r * x2[r][...],
// s1 and Z sums of arrays (NS of them in Z, or any number for NS = 0).  diag: the diagonal of
// the one-body terms joins Z, with xs as (diag_a + diag_b - diag_i - diag_j) / 4 times xs (antisymmetric in both
// pairs), else as the products it stands for would form it from an x2 of any symmetry: 1/2 diag_b x_ijab in every
// row, and - diag_j x_ijab on the unique pairs (ka, a) < (kb, b) alone.  These are far the largest terms: they are
// added here, in double (in the products with the other elements they double the rounding of a
// complex64 product's doubles, from 1.0e-7 to 2.1e-7 at Nk=5, o=8, v=40), from the elements of x2 that omega reads
// again a moment later (48 complex64 vectors of that size: 7.2 ms for 41 GB; 6.5 with one read of x2, as an x2 that
// is antisymmetric would allow).  The workgroup of an orbit's first
// row ((ki, i) <= (kj, j), ka <= kb) writes all of its distinct rows; the others return at once.
template <typename T, int NS>
__global__ void k_outputs(SlabList s1, SlabList zs, SlabList xs, const double2 *diag, const double2 *x1,
                          const double2 *x2, double2 *y1, double2 *y2, const double *omega, KMesh km, int R, int o,
                          int v, double scale, unsigned b1) {
    extern __shared__ __attribute__((aligned(16))) double2 lds[];
    const int nk = km.size(), vv = v * v;
    if (blockIdx.x < b1) {      // singles
        const i64 E = (i64)o * v, n = (i64)R * nk * E;
        for (i64 t = blockIdx.x * (i64)blockDim.x + threadIdx.x; t < n; t += (i64)b1 * blockDim.x) {
            const i64 e = t % E;
            const int k = (int)((t / E) % nk), r = (int)(t / (E * nk));
            double2 out = slab_sum<T, 0>(s1, ((i64)k * R + r) * E + e);
            if (omega) {
                const double w = omega[r];
                const double2 xv = x1[t];
                out.x -= w * xv.x;
                out.y -= w * xv.y;
            }
            y1[t] = out;
        }
        return;
    }
    const i64 B = (i64)nk * nk * nk;
    const i64 rows = B * R * o * o;
    for (i64 row = blockIdx.x - b1; row < rows; row += gridDim.x - b1) {
        // row indexes the caller layout [r][blk][i][j], elements (a, b)
        i64 q = row;
        const int j = take(q, o);
        const int i = take(q, o);
        const i64 blk = q % B;
        const int r = (int)(q / B);
        const int ka = (int)(blk % nk), kj = (int)((blk / nk) % nk), ki = (int)(blk / (nk * nk));
        const int kb = km.comb(ki, kj, ka);
        const int pi = ki * o + i, pj = kj * o + j;
        if (pi > pj || ka > kb) continue;
        auto zrow = [&](int k0, int k1, int k2, int p, int q3) {
            return ((((i64)(k0 * nk + k1) * nk + k2) * R + r) * o + p) * o * vv + (i64)q3 * vv;
        };
        auto yrow = [&](int k0, int k1, int k2, int p, int q3) {
            return (((i64)r * B + ((i64)k0 * nk + k1) * nk + k2) * o + p) * o * vv + (i64)q3 * vv;
        };
        const i64 zr[4] = {zrow(ki, kj, ka, i, j), zrow(kj, ki, ka, j, i), zrow(ki, kj, kb, i, j), zrow(kj, ki, kb, j, i)};
        const i64 yr[4] = {row * vv, yrow(kj, ki, ka, j, i), yrow(ki, kj, kb, i, j), yrow(kj, ki, kb, j, i)};
        const double w = omega ? omega[r] : 0.0;
        const double2 *const da = diag + ka * (o + v) + o, *const db = diag + kb * (o + v) + o;
        double2 di = make_double2(0, 0), dj = make_double2(0, 0);
        if (diag) {
            di = diag[ki * (o + v) + i];
            dj = diag[kj * (o + v) + j];
        }
        const double half = 0.5 / scale;
        orbit_rows(lds, v, pi != pj, ka != kb,
                   [&](int rw, int e, int a, int b) {
                       double2 z = slab_sum<T, NS>(zs, zr[rw] + e);
                       if (diag && xs.n) {             // the same factor for the four rows
                           const double2 x = slab_sum<T, 0>(xs, zr[rw] + e), fa = da[a], fb = db[b];
                           const double2 d = make_double2(fa.x + fb.x - di.x - dj.x, fa.y + fb.y - di.y - dj.y);
                           z.x += 0.25 * (d.x * x.x - d.y * x.y);
                           z.y += 0.25 * (d.x * x.y + d.y * x.x);
                       } else if (diag) {              // second virtual and second occupied index of the row
                           const double2 x = x2[yr[rw] + e], fv = rw < 2 ? db[b] : da[a], fo = (rw & 1) ? di : dj;
                           const double u = (rw < 2 ? ka < kb || a < b : ka == kb && b < a) ? 2 : 0;
                           const double2 d = make_double2(half * (fv.x - u * fo.x), half * (fv.y - u * fo.y));
                           z.x += d.x * x.x - d.y * x.y;
                           z.y += d.x * x.y + d.y * x.x;
                       }
                       return z;
                   },
                   [&](int rw, int e, int, int, double2 z) {
                       const i64 at = yr[rw] + e;
                       double2 out = make_double2(scale * z.x, scale * z.y);
                       if (omega) {
                           const double2 xv = x2[at];
                           out.x -= w * xv.x;
                           out.y -= w * xv.y;
                       }
                       y2[at] = out;
                   });
    }
}

template <typename T>
hipError_t outputs(const SlabList &s1, const SlabList &Z, const SlabList &X, const void *diag, const void *x1,
                   const void *x2, void *y1, void *y2, const double *omega, KMesh km, int R, int o, int v,
                   double scale, hipStream_t s) {
    const int nk = km.size();
    const i64 rows = (i64)nk * nk * nk * R * o * o;
    const unsigned b1 = (unsigned)std::min<i64>(((i64)R * nk * o * v + 255) / 256, 1024);
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(b1 + rows_grid(rows)), dim3(wave_rows(rows, v) ? 64 : 256), orbit_lds(v), s, s1, Z, X, (const double2 *)diag,
                           (const double2 *)x1, (const double2 *)x2, (double2 *)y1, (double2 *)y2, omega, km, R, o, v, scale, b1);
    };
    switch (Z.n) {
    case 1: go(k_outputs<T, 1>); break;
    case 2: go(k_outputs<T, 2>); break;
    case 3: go(k_outputs<T, 3>); break;
    case 4: go(k_outputs<T, 4>); break;
    case 5: go(k_outputs<T, 5>); break;
    case 6: go(k_outputs<T, 6>); break;
    case 7: go(k_outputs<T, 7>); break;
    case 8: go(k_outputs<T, 8>); break;
    default: go(k_outputs<T, 0>); break;
    }
    return hipGetLastError();
}

// Slice of Cholesky vectors: out[k1][k2][Q][p][q] = scale * L[k1][k2][Q][p0+p][q0+q]   (conj_pair = 0)
//                            out[k1][k2][Q][p][q] = scale * conj(L[k2][k1][Q][q0+q][p0+p])  (conj_pair = 1)
template <typename Tout>
__global__ void k_chol_slice(const double2 *L, typename Cx<Tout>::type *out, int nk, int naux, int n, int p0,
                             int np, int q0, int nq, double scale, int conj_pair) {
    const i64 n_out = (i64)nk * nk * naux * np * nq;
    for (i64 t = blockIdx.x * (i64)blockDim.x + threadIdx.x; t < n_out; t += (i64)gridDim.x * blockDim.x) {
        i64 q = t;
        const int qq = take(q, nq);
        const int pp = take(q, np);
        const int Q = take(q, naux);
        const int k2 = (int)(q % nk);
        const int k1 = (int)(q / nk);
        double2 v;
        if (!conj_pair) {
            v = L[(((i64)(k1 * nk + k2) * naux + Q) * n + (p0 + pp)) * n + (q0 + qq)];
        } else {
            v = L[(((i64)(k2 * nk + k1) * naux + Q) * n + (q0 + qq)) * n + (p0 + pp)];
            v.y = -v.y;
        }
        out[t] = mk<Tout>((Tout)(scale * v.x), (Tout)(scale * v.y));
    }
}

template <typename Tout>
hipError_t chol_slice(const void *L, void *out, int nk, int naux, int n, int p0, int np, int q0, int nq,
                      double scale, int conj_pair, hipStream_t s) {
    hipLaunchKernelGGL(k_chol_slice<Tout>, dim3(grid_for((i64)nk * nk * naux * np * nq)), dim3(256), 0, s,
                       (const double2 *)L, (typename Cx<Tout>::type *)out, nk, naux, n, p0, np, q0, nq, scale,
                       conj_pair);
    return hipGetLastError();
}

// Strided block copy of the 1E matrices: out[k][p][q] = in[k][p0+p][q0+q] (in: [nk][n][n])
template <typename Tout>
__global__ void k_one_body_slice(const double2 *in, typename Cx<Tout>::type *out, int nk, int n, int p0, int np,
                                 int q0, int nq) {
    const i64 N = (i64)nk * np * nq;
    for (i64 t = blockIdx.x * (i64)blockDim.x + threadIdx.x; t < N; t += (i64)gridDim.x * blockDim.x) {
        const int qq = (int)(t % nq), pp = (int)((t / nq) % np), k = (int)(t / ((i64)nq * np));
        double2 v = in[((i64)k * n + p0 + pp) * n + q0 + qq];
        out[t] = mk<Tout>((Tout)v.x, (Tout)v.y);
    }
}

template <typename Tout>
hipError_t one_body_slice(const void *in, void *out, int nk, int n, int p0, int np, int q0, int nq, hipStream_t s) {
    hipLaunchKernelGGL(k_one_body_slice<Tout>, dim3(grid_for((i64)nk * np * nq)), dim3(256), 0, s,
                       (const double2 *)in, (typename Cx<Tout>::type *)out, nk, n, p0, np, q0, nq);
    return hipGetLastError();
}

template <typename Tout>
__global__ void k_axis_slice(const double2 *in, typename Cx<Tout>::type *out, int nax, int nk, int n, int p0, int np,
                             int q0, int nq, int transpose) {
    const i64 N = (i64)nk * nax * np * nq;
    for (i64 t = blockIdx.x * (i64)blockDim.x + threadIdx.x; t < N; t += (i64)gridDim.x * blockDim.x) {
        i64 q = t;
        const int qq = take(q, nq);
        const int pp = take(q, np);
        const int x = (int)(q % nax);
        const int k = (int)(q / nax);
        const double2 v = transpose ? in[(((i64)x * nk + k) * n + q0 + qq) * n + p0 + pp]
                                    : in[(((i64)x * nk + k) * n + p0 + pp) * n + q0 + qq];
        out[t] = mk<Tout>((Tout)v.x, (Tout)v.y);
    }
}

template <typename Tout>
hipError_t axis_slice(const void *in, void *out, int nax, int nk, int n, int p0, int np, int q0, int nq, int transpose,
                      hipStream_t s) {
    hipLaunchKernelGGL(k_axis_slice<Tout>, dim3(grid_for((i64)nk * nax * np * nq)), dim3(256), 0, s,
                       (const double2 *)in, (typename Cx<Tout>::type *)out, nax, nk, n, p0, np, q0, nq, transpose);
    return hipGetLastError();
}

// Inverse of axis_slice: out[x][k][p0+p][q0+q] = in[k][x][p][q]
// (transpose: out[x][k][q0+q][p0+p] = in[k][x][p][q]); complex128.
__global__ void k_axis_scatter(const double2 *in, double2 *out, int nax, int nk, int n, int p0, int np, int q0,
                               int nq, int transpose) {
    const i64 N = (i64)nk * nax * np * nq;
    for (i64 t = blockIdx.x * (i64)blockDim.x + threadIdx.x; t < N; t += (i64)gridDim.x * blockDim.x) {
        i64 q = t;
        const int qq = take(q, nq);
        const int pp = take(q, np);
        const int x = (int)(q % nax);
        const int k = (int)(q / nax);
        const i64 dst = transpose ? (((i64)x * nk + k) * n + q0 + qq) * n + p0 + pp
                                  : (((i64)x * nk + k) * n + p0 + pp) * n + q0 + qq;
        out[dst] = in[t];
    }
}

hipError_t axis_scatter(const void *in, void *out, int nax, int nk, int n, int p0, int np, int q0, int nq,
                        int transpose, hipStream_t s) {
    hipLaunchKernelGGL(k_axis_scatter, dim3(grid_for((i64)nk * nax * np * nq)), dim3(256), 0, s,
                       (const double2 *)in, (double2 *)out, nax, nk, n, p0, np, q0, nq, transpose);
    return hipGetLastError();
}

// y = alpha * x (complex alpha, n elements, double2)
__global__ void k_scale_copy(double2 *y, const double2 *x, double ar, double ai, i64 n) {
    for (i64 t = blockIdx.x * (i64)blockDim.x + threadIdx.x; t < n; t += (i64)gridDim.x * blockDim.x) {
        const double2 v = x[t];
        y[t] = make_double2(ar * v.x - ai * v.y, ar * v.y + ai * v.x);
    }
}
hipError_t scale_copy(void *y, const void *x, double ar, double ai, i64 n, hipStream_t s) {
    hipLaunchKernelGGL(k_scale_copy, dim3(grid_for(n)), dim3(256), 0, s, (double2 *)y, (const double2 *)x, ar, ai, n);
    return hipGetLastError();
}

// out = scale * in with permuted indices: output dim d is input dim perm[d]; output blocks
// [k0][k1][k2] with k3 from the output momentum signs sg (both tensors conserve momentum).
__global__ void k_permute4(const double2 *in, double2 *out, KMesh km, int e0, int e1, int e2, int e3, int p0, int p1,
                           int p2, int p3, int s0, int s1, int s2, int s3, double scale) {
    const int ein[4] = {e0, e1, e2, e3}, perm[4] = {p0, p1, p2, p3}, sg[4] = {s0, s1, s2, s3};
    int eo[4];
    for (int d = 0; d < 4; ++d) eo[d] = ein[perm[d]];
    const int nk = km.size();
    const i64 inner = (i64)e0 * e1 * e2 * e3;
    const i64 n = (i64)nk * nk * nk * inner;
    for (i64 t = blockIdx.x * (i64)blockDim.x + threadIdx.x; t < n; t += (i64)gridDim.x * blockDim.x) {
        i64 q = t;
        int io[4], ko[4];
        for (int d = 3; d >= 0; --d) { io[d] = (int)(q % eo[d]); q /= eo[d]; }
        ko[2] = take(q, nk);
        ko[1] = take(q, nk);
        ko[0] = (int)q;
        ko[3] = km.sum3(-sg[3] * sg[0], ko[0], -sg[3] * sg[1], ko[1], -sg[3] * sg[2], ko[2]);
        int ii[4], ki[4];
        for (int d = 0; d < 4; ++d) { ii[perm[d]] = io[d]; ki[perm[d]] = ko[d]; }
        const i64 src = (((i64)(ki[0] * nk + ki[1]) * nk + ki[2]) * inner) +
                        (((i64)ii[0] * e1 + ii[1]) * e2 + ii[2]) * e3 + ii[3];
        const double2 x = in[src];
        out[t] = make_double2(scale * x.x, scale * x.y);
    }
}

hipError_t permute4(const void *in, void *out, KMesh km, const int *ext_in, const int *perm, const int *sg_out,
                    double scale, hipStream_t s) {
    const int nk = km.size();
    const i64 n = (i64)nk * nk * nk * ext_in[0] * ext_in[1] * ext_in[2] * ext_in[3];
    hipLaunchKernelGGL(k_permute4, dim3(grid_for(n)), dim3(256), 0, s, (const double2 *)in, (double2 *)out, km,
                       ext_in[0], ext_in[1], ext_in[2], ext_in[3], perm[0], perm[1], perm[2], perm[3], sg_out[0],
                       sg_out[1], sg_out[2], sg_out[3], scale);
    return hipGetLastError();
}

// One thread per output element; bound by the strided reads of `in`, once per set of amplitudes.
__global__ void k_ring_matrix(const double2 *in, const double2 *fbe, const double2 *fmj, double2 *out, KMesh km, int o,
                              int v, int transposed) {
    const int nk = km.size(), e2 = transposed ? o : v, e3 = transposed ? v : o;
    const i64 n = (i64)nk * nk * nk * o * v * v * o;
    for (i64 t = blockIdx.x * (i64)blockDim.x + threadIdx.x; t < n; t += (i64)gridDim.x * blockDim.x) {
        i64 q = t;
        const int i3 = take(q, e3);
        const int i2 = take(q, e2);
        const int e = take(q, v);
        const int m = take(q, o);
        const int k2 = take(q, nk);
        const int ke = (int)(q % nk);
        const int kmm = (int)(q / nk);
        // k_m + k_b = k_e + k_j
        const int k3 = transposed ? km.sum3(1, ke, 1, k2, -1, kmm) : km.sum3(1, kmm, -1, ke, 1, k2);
        const int b = transposed ? i3 : i2, j = transposed ? i2 : i3, kb = transposed ? k3 : k2;
        double2 x = in[((((((i64)kmm * nk + kb) * nk + ke) * o + m) * v + b) * v + e) * o + j];
        if (ke == kb) {                     // and k_m = k_j
            if (m == j && b != e) {
                const double2 f = fbe[((i64)kb * v + b) * v + e];
                x.x += 0.5 * f.x;
                x.y += 0.5 * f.y;
            }
            if (fmj && b == e && m != j) {
                const double2 f = fmj[((i64)kmm * o + m) * o + j];
                x.x -= 0.5 * f.x;
                x.y -= 0.5 * f.y;
            }
        }
        out[t] = x;
    }
}

// diag[k] = (fmj[k][m][m]; fbe[k][b][b])
__global__ void k_pair_diag(const double2 *fbe, const double2 *fmj, double2 *diag, int nk, int o, int v) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x, n = o + v;
    if (t >= nk * n) return;
    const int k = t / n, p = t % n;
    diag[t] = p < o ? fmj[(i64)k * o * o + (i64)p * (o + 1)] : fbe[(i64)k * v * v + (i64)(p - o) * (v + 1)];
}
hipError_t pair_diag(const void *fbe, const void *fmj, void *diag, int nk, int o, int v, hipStream_t s) {
    hipLaunchKernelGGL(k_pair_diag, dim3((nk * (o + v) + 255) / 256), dim3(256), 0, s, (const double2 *)fbe,
                       (const double2 *)fmj, (double2 *)diag, nk, o, v);
    return hipGetLastError();
}

hipError_t ring_matrix(const void *in, const void *fbe, const void *fmj, void *out, KMesh km, int o, int v,
                       int transposed, hipStream_t s) {
    const int nk = km.size();
    const i64 n = (i64)nk * nk * nk * o * v * v * o;
    hipLaunchKernelGGL(k_ring_matrix, dim3(grid_for(n)), dim3(256), 0, s, (const double2 *)in, (const double2 *)fbe,
                       (const double2 *)fmj, (double2 *)out, km, o, v, transposed);
    return hipGetLastError();
}

__global__ void k_off_diag(const double2 *in, double2 *out, int n, int m) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t < n) out[t] = t % m == t / m % m ? make_double2(0, 0) : in[t];
}
hipError_t off_diag(const void *in, void *out, int nk, int m, hipStream_t s) {
    const int n = nk * m * m;
    hipLaunchKernelGGL(k_off_diag, dim3((n + 255) / 256), dim3(256), 0, s, (const double2 *)in, (double2 *)out, n, m);
    return hipGetLastError();
}

// y = s * conj(x)
__global__ void k_conj_scale(double2 *y, const double2 *x, double s, i64 n) {
    for (i64 t = blockIdx.x * (i64)blockDim.x + threadIdx.x; t < n; t += (i64)gridDim.x * blockDim.x) {
        const double2 v = x[t];
        y[t] = make_double2(s * v.x, -s * v.y);
    }
}
hipError_t conj_scale(void *y, const void *x, double s, i64 n, hipStream_t st) {
    hipLaunchKernelGGL(k_conj_scale, dim3(grid_for(n)), dim3(256), 0, st, (double2 *)y, (const double2 *)x, s, n);
    return hipGetLastError();
}

// out = scale * c(y - y(ij swapped) - y(ab swapped) + y(both swapped)) on caller-layout doubles
// [R][ki][kj][ka][i][j][a][b] (kb implied), c = complex conjugation when conj != 0.  Out of place.
__global__ void k_antisym(const double2 *y, double2 *out, int R, KMesh km, int o, int v, double scale, int conj) {
    extern __shared__ __attribute__((aligned(16))) double2 lds[];
    const int nk = km.size(), vv = v * v;
    const i64 B = (i64)nk * nk * nk;
    const i64 rows = (i64)R * B * o * o;
    for (i64 row = blockIdx.x; row < rows; row += gridDim.x) {
        // row = [r][ki][kj][ka][i][j], elements (a, b)
        i64 q = row;
        const int j = take(q, o);
        const int i = take(q, o);
        const int ka = take(q, nk);
        const int kj = take(q, nk);
        const int ki = (int)(q % nk);
        const i64 r = q / nk;
        const int kb = km.comb(ki, kj, ka);
        const int pi = ki * o + i, pj = kj * o + j;
        if (pi > pj || ka > kb) continue;
        auto rowp = [&](int k0, int k1, int k2, int p, int q3) {
            return ((r * B + ((i64)k0 * nk + k1) * nk + k2) * o + p) * o * vv + (i64)q3 * vv;
        };
        const i64 yr[4] = {row * vv, rowp(kj, ki, ka, j, i), rowp(ki, kj, kb, i, j), rowp(kj, ki, kb, j, i)};
        orbit_rows(lds, v, pi != pj, ka != kb, [&](int rw, int e, int, int) { return y[yr[rw] + e]; },
                   [&](int rw, int e, int, int, double2 z) {
                       out[yr[rw] + e] = make_double2(scale * z.x, conj ? -scale * z.y : scale * z.y);
                   });
    }
}

hipError_t antisym(const void *y, void *out, int R, KMesh km, int o, int v, double scale, int conj, hipStream_t s) {
    const int nk = km.size();
    const i64 rows = (i64)R * nk * nk * nk * o * o;
    hipLaunchKernelGGL(k_antisym, dim3(rows_grid(rows)), dim3(256), orbit_lds(v), s, (const double2 *)y, (double2 *)out, R, km, o,
                       v, scale, conj);
    return hipGetLastError();
}

__global__ void k_convert(const double2 *in, float2 *out, i64 n) {
    for (i64 t = blockIdx.x * (i64)blockDim.x + threadIdx.x; t < n; t += (i64)gridDim.x * blockDim.x) {
        double2 v = in[t];
        out[t] = make_float2((float)v.x, (float)v.y);
    }
}

hipError_t convert_f64_f32(const void *in, void *out, i64 n, hipStream_t s) {
    hipLaunchKernelGGL(k_convert, dim3(grid_for(n)), dim3(256), 0, s, (const double2 *)in, (float2 *)out, n);
    return hipGetLastError();
}

// Z[ki,kj,ka][r][i][j][a][b] = scale * (P_ij P_ab y)[r][ki,kj,ka][i][j][a][b]  (caller layout in, block layout out)
template <typename T>
__global__ void k_pp_in(const double2 *y, typename Cx<T>::type *Z, KMesh km, int R, int o, int v, double scale) {
    extern __shared__ __attribute__((aligned(16))) double2 lds[];
    const int nk = km.size(), vv = v * v;
    const i64 B = (i64)nk * nk * nk;
    const i64 rows = B * R * o * o;
    for (i64 row = blockIdx.x; row < rows; row += gridDim.x) {
        // row indexes the block layout [blk][r][i][j], elements (a, b)
        i64 q = row;
        const int j = take(q, o);
        const int i = take(q, o);
        const int r = (int)(q % R);
        const i64 blk = q / R;
        const int ka = (int)(blk % nk), kj = (int)((blk / nk) % nk), ki = (int)(blk / (nk * nk));
        const int kb = km.comb(ki, kj, ka);
        const int pi = ki * o + i, pj = kj * o + j;
        if (pi > pj || ka > kb) continue;
        auto yrow = [&](int k0, int k1, int k2, int p, int q3) {
            return (((i64)r * B + ((i64)k0 * nk + k1) * nk + k2) * o + p) * o * vv + (i64)q3 * vv;
        };
        auto zrow = [&](int k0, int k1, int k2, int p, int q3) {
            return ((((i64)(k0 * nk + k1) * nk + k2) * R + r) * o + p) * o * vv + (i64)q3 * vv;
        };
        const i64 yr[4] = {yrow(ki, kj, ka, i, j), yrow(kj, ki, ka, j, i), yrow(ki, kj, kb, i, j), yrow(kj, ki, kb, j, i)};
        const i64 zr[4] = {row * vv, zrow(kj, ki, ka, j, i), zrow(ki, kj, kb, i, j), zrow(kj, ki, kb, j, i)};
        orbit_rows(lds, v, pi != pj, ka != kb, [&](int rw, int e, int, int) { return y[yr[rw] + e]; },
                   [&](int rw, int e, int, int, double2 z) { Z[zr[rw] + e] = mk<T>((T)(scale * z.x), (T)(scale * z.y)); });
    }
}

template <typename T>
hipError_t pp_in(const void *y, void *Z, KMesh km, int R, int o, int v, double scale, hipStream_t s) {
    const int nk = km.size();
    const i64 rows = (i64)nk * nk * nk * R * o * o;
    hipLaunchKernelGGL(k_pp_in<T>, dim3(rows_grid(rows)), dim3(wave_rows(rows, v) ? 64 : 256), orbit_lds(v), s, (const double2 *)y,
                       (typename Cx<T>::type *)Z, km, R, o, v, scale);
    return hipGetLastError();
}

// out[blk][r][i][j][a][b] (+)= scale * (in[blk][r][i][j][a][b] - in[blk'][r][i][j][b][a]), blk = (ki,kj,ka),
// blk' = (ki,kj,kb): the (a,b)-antisymmetric completion of a block-layout doubles array that holds
// only one block of each (ka, kb) pair
template <typename T>
__global__ void k_expand_ab(const typename Cx<T>::type *in, typename Cx<T>::type *out, KMesh km, int R, int o,
                            int v, T scale, int add) {
    const int nk = km.size(), vv = v * v;
    const i64 inblk = (i64)R * o * o;
    const i64 rows = (i64)nk * nk * nk * inblk;
    for (i64 row = blockIdx.x; row < rows; row += gridDim.x) {
        // row = [blk][r][i][j], elements (a, b)
        const i64 blk = row / inblk, rest = row - blk * inblk;
        const int ka = (int)(blk % nk), kj = (int)((blk / nk) % nk), ki = (int)(blk / (nk * nk));
        const int kb = km.comb(ki, kj, ka);
        const typename Cx<T>::type *X1 = in + row * vv;
        const typename Cx<T>::type *X2 = in + ((((i64)ki * nk + kj) * nk + kb) * inblk + rest) * vv;
        typename Cx<T>::type *dst = out + row * vv;
        for (int e = threadIdx.x; e < vv; e += blockDim.x) {
            const int a = e / v, b = e - a * v;
            const auto x1 = X1[e], x2 = X2[b * v + a];
            auto y = mk<T>(0, 0);
            if (add) y = dst[e];
            dst[e] = mk<T>(y.x + scale * (x1.x - x2.x), y.y + scale * (x1.y - x2.y));
        }
    }
}

template <typename T>
hipError_t expand_ab(const void *in, void *out, KMesh km, int R, int o, int v, double scale, int add, hipStream_t s) {
    const int nk = km.size();
    const i64 rows = (i64)nk * nk * nk * R * o * o;
    hipLaunchKernelGGL(k_expand_ab<T>, dim3(rows_grid(rows)), dim3(256), 0, s, (const typename Cx<T>::type *)in,
                       (typename Cx<T>::type *)out, km, R, o, v, (T)scale, add);
    return hipGetLastError();
}

// y += x (complex, n elements)
template <typename T>
__global__ void k_add(typename Cx<T>::type *y, const typename Cx<T>::type *x, i64 n) {
    for (i64 t = blockIdx.x * (i64)blockDim.x + threadIdx.x; t < n; t += (i64)gridDim.x * blockDim.x) {
        auto a = y[t], b = x[t];
        y[t] = mk<T>(a.x + b.x, a.y + b.y);
    }
}
template <typename T>
hipError_t add_inplace(void *y, const void *x, i64 n, hipStream_t s) {
    hipLaunchKernelGGL(k_add<T>, dim3(grid_for(n)), dim3(256), 0, s, (typename Cx<T>::type *)y,
                       (const typename Cx<T>::type *)x, n);
    return hipGetLastError();
}

// zero fill (a kernel rather than a memset so that programs stay capturable)
template <typename T>
__global__ void k_zero(typename Cx<T>::type *y, i64 n) {
    for (i64 t = blockIdx.x * (i64)blockDim.x + threadIdx.x; t < n; t += (i64)gridDim.x * blockDim.x) y[t] = mk<T>(0, 0);
}
template <typename T>
hipError_t zero_fill(void *y, i64 n, hipStream_t s) {
    hipLaunchKernelGGL(k_zero<T>, dim3(grid_for(n)), dim3(256), 0, s, (typename Cx<T>::type *)y, n);
    return hipGetLastError();
}

// out[k2][k1][Q][q][p] = in[k1][k2][Q][p][q]   ([nk][nk][naux][m][m] blocks)
template <typename T>
__global__ void k_pair_transpose(const typename Cx<T>::type *in, typename Cx<T>::type *out, int nk, int naux, int m) {
    const i64 n = (i64)nk * nk * naux * m * m;
    for (i64 t = blockIdx.x * (i64)blockDim.x + threadIdx.x; t < n; t += (i64)gridDim.x * blockDim.x) {
        i64 q = t;
        const int p = take(q, m);
        const int qq = take(q, m);
        const int Q = take(q, naux);
        const int k1 = (int)(q % nk);
        const int k2 = (int)(q / nk);
        // t = [k2][k1][Q][qq][p]
        out[t] = in[(((i64)(k1 * nk + k2) * naux + Q) * m + p) * m + qq];
    }
}
template <typename T>
hipError_t pair_transpose(const void *in, void *out, int nk, int naux, int m, hipStream_t s) {
    hipLaunchKernelGGL(k_pair_transpose<T>, dim3(grid_for((i64)nk * nk * naux * m * m)), dim3(256), 0, s,
                       (const typename Cx<T>::type *)in, (typename Cx<T>::type *)out, nk, naux, m);
    return hipGetLastError();
}

// Reverse of chol_slice (no conjugation, scale 1): out[k1][k2][Q][p0+p][q0+q] += in[k1][k2][Q][p][q]
// (complex128; out is a full [nk][nk][naux][n][n] array)
__global__ void k_slice_add(const double2 *in, double2 *out, int nk, int naux, int n, int p0, int np, int q0,
                            int nq) {
    const i64 N = (i64)nk * nk * naux * np * nq;
    for (i64 t = blockIdx.x * (i64)blockDim.x + threadIdx.x; t < N; t += (i64)gridDim.x * blockDim.x) {
        i64 q = t;
        const int qq = take(q, nq);
        const int pp = take(q, np);
        const i64 dst = (q * n + p0 + pp) * n + q0 + qq;   // q = (k1 * nk + k2) * naux + Q
        const double2 a = out[dst], b = in[t];
        out[dst] = make_double2(a.x + b.x, a.y + b.y);
    }
}

hipError_t slice_add(const void *in, void *out, int nk, int naux, int n, int p0, int np, int q0, int nq,
                     hipStream_t s) {
    hipLaunchKernelGGL(k_slice_add, dim3(grid_for((i64)nk * nk * naux * np * nq)), dim3(256), 0, s,
                       (const double2 *)in, (double2 *)out, nk, naux, n, p0, np, q0, nq);
    return hipGetLastError();
}

// g[ki][kj][ki][i][j][a][b] += c x[ki][i][a] y[kj][j][b]: the k-diagonal singles x, y put into the
// blocks (ki, kj, ka = ki, kb = kj) of an oovv-class array (complex128)
__global__ void k_outer_oovv(double2 *g, const double2 *x, const double2 *y, double c, int nk, int o, int v) {
    const i64 N = (i64)nk * nk * o * o * v * v;
    for (i64 t = blockIdx.x * (i64)blockDim.x + threadIdx.x; t < N; t += (i64)gridDim.x * blockDim.x) {
        i64 q = t;
        const int b = take(q, v);
        const int a = take(q, v);
        const int j = take(q, o);
        const int i = take(q, o);
        const int kj = (int)(q % nk);
        const int ki = (int)(q / nk);
        const double2 xv = x[((i64)ki * o + i) * v + a], yv = y[((i64)kj * o + j) * v + b];
        const i64 dst = (((((i64)ki * nk + kj) * nk + ki) * o + i) * o + j) * v * v + (i64)a * v + b;
        const double2 gv = g[dst];
        g[dst] = make_double2(gv.x + c * (xv.x * yv.x - xv.y * yv.y), gv.y + c * (xv.x * yv.y + xv.y * yv.x));
    }
}

hipError_t outer_oovv(void *g, const void *x, const void *y, double c, int nk, int o, int v, hipStream_t s) {
    hipLaunchKernelGGL(k_outer_oovv, dim3(grid_for((i64)nk * nk * o * o * v * v)), dim3(256), 0, s, (double2 *)g,
                       (const double2 *)x, (const double2 *)y, c, nk, o, v);
    return hipGetLastError();
}

#define INST(T)                                                                                              \
    template hipError_t pp_in<T>(const void *, void *, KMesh, int, int, int, double, hipStream_t);             \
    template hipError_t add_inplace<T>(void *, const void *, i64, hipStream_t);                              \
    template hipError_t expand_ab<T>(const void *, void *, KMesh, int, int, int, double, int, hipStream_t);        \
    template hipError_t zero_fill<T>(void *, i64, hipStream_t);                                              \
    template hipError_t pair_transpose<T>(const void *, void *, int, int, int, hipStream_t);                                                                                              \
    template hipError_t tau_like<T>(const void *, const void *, const void *, void *, KMesh, int, int, int,  \
                                    double, int, hipStream_t);                                               \
    template hipError_t inputs<T>(const void *, const void *, const void *, void *, void *, void *, KMesh, int, \
                                  int, int, double, hipStream_t);                                            \
    template hipError_t outputs<T>(const SlabList &, const SlabList &, const SlabList &, const void *,        \
                                   const void *, const void *, void *, void *, const double *, KMesh, int,    \
                                   int, int, double, hipStream_t);                                            \
    template hipError_t chol_slice<T>(const void *, void *, int, int, int, int, int, int, int, double, int,  \
                                      hipStream_t);                                                          \
    template hipError_t one_body_slice<T>(const void *, void *, int, int, int, int, int, int, hipStream_t);  \
    template hipError_t axis_slice<T>(const void *, void *, int, int, int, int, int, int, int, int, hipStream_t); \
    template hipError_t rhs_to_block<double, T>(const void *, void *, int, i64, i64, double, hipStream_t);
INST(double)
INST(float)

}  // namespace lrcc
