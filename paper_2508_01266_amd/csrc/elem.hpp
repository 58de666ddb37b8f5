// Launchers of the streaming kernels (definitions in elem.hip).
#pragma once
#include "common.hpp"
#include "group.hpp"

namespace lrcc {
template <typename Tin, typename Tout>
hipError_t rhs_to_block(const void *in, void *out, int R, i64 B, i64 E, double scale, hipStream_t s);
template <typename T>
hipError_t tau_like(const void *x1, const void *x2, const void *t1, void *out, KMesh km, int R, int o, int v,
                    double c, int x1_has_rhs, hipStream_t s);
// x1, x2 (caller layout) -> o1, o2 (blocks, doubles scaled) and dtau (tau_like of them with t1)
template <typename T>
hipError_t inputs(const void *x1, const void *x2, const void *t1, void *o1, void *o2, void *dtau, KMesh km, int R,
                  int o, int v, double scale, hipStream_t s);
// y1 = s1 - omega x1, y2 = scale P(ij)P(ab) (Z + D) - omega x2 (caller layout; omega may be null), D_ijab =
// diag_b x_ijab / 2 - diag_j x_ijab (the second for (ka, a) < (kb, b) alone), x = x2 / scale, or with X.n
// (diag_a + diag_b - diag_i - diag_j) / 4 X_ijab, X antisymmetric (diag: complex128 [nk][o + v], null for D = 0)
template <typename T>
hipError_t outputs(const SlabList &s1, const SlabList &Z, const SlabList &X, const void *diag, const void *x1,
                   const void *x2, void *y1, void *y2, const double *omega, KMesh km, int R, int o, int v,
                   double scale, hipStream_t s);
template <typename Tout>
hipError_t chol_slice(const void *L, void *out, int nk, int naux, int n, int p0, int np, int q0, int nq,
                      double scale, int conj_pair, hipStream_t s);
template <typename Tout>
hipError_t one_body_slice(const void *in, void *out, int nk, int n, int p0, int np, int q0, int nq, hipStream_t s);
hipError_t convert_f64_f32(const void *in, void *out, i64 n, hipStream_t s);
template <typename Tout>
hipError_t axis_slice(const void *in, void *out, int nax, int nk, int n, int p0, int np, int q0, int nq, int transpose,
                      hipStream_t s);
hipError_t scale_copy(void *y, const void *x, double ar, double ai, i64 n, hipStream_t s);
// inverse of axis_slice (complex128 in and out): out[x][k][p0+p][q0+q] = in[k][x][p][q]
hipError_t axis_scatter(const void *in, void *out, int nax, int nk, int n, int p0, int np, int q0, int nq,
                        int transpose, hipStream_t s);
hipError_t conj_scale(void *y, const void *x, double s, i64 n, hipStream_t st);
// caller-layout doubles: out = scale * c(P(ij) P(ab) y), c = conjugation when conj != 0 (out of place)
hipError_t antisym(const void *y, void *out, int R, KMesh km, int o, int v, double scale, int conj, hipStream_t s);
// four-index complex128 permutation, scaled: output dim d = input dim perm[d]; output momentum signs sg_out
hipError_t permute4(const void *in, void *out, KMesh km, const int *ext_in, const int *perm, const int *sg_out,
                    double scale, hipStream_t s);
// W-bar in the layouts of the ring products, with off-diagonal one-body terms of x2: out[m][e][b][j]
// (transposed: [m][e][j][b]) = in[m][b][e][j] + delta_mj fbe[b][e] / 2 (b != e) - delta_be fmj[m][j] / 2 (m != j)
// (complex128; fbe, fmj k-diagonal; fmj may be null)
hipError_t ring_matrix(const void *in, const void *fbe, const void *fmj, void *out, KMesh km, int o, int v,
                       int transposed, hipStream_t s);
// out[k] = in[k] (complex128 [nk][m][m]) with a zero diagonal
hipError_t off_diag(const void *in, void *out, int nk, int m, hipStream_t s);
// diag[k] = the diagonals of fmj and fbe (complex128 [nk][o + v])
hipError_t pair_diag(const void *fbe, const void *fmj, void *diag, int nk, int o, int v, hipStream_t s);
template <typename T>
hipError_t pp_in(const void *y, void *Z, KMesh km, int R, int o, int v, double scale, hipStream_t s);
// out (+)= scale * (in - in with (a,b) and ka/kb swapped), added where `add`: completes a doubles array that holds one
// block of each (ka, kb) pair
template <typename T>
hipError_t expand_ab(const void *in, void *out, KMesh km, int R, int o, int v, double scale, int add, hipStream_t s);
template <typename T>
hipError_t add_inplace(void *y, const void *x, i64 n, hipStream_t s);
template <typename T>
hipError_t zero_fill(void *y, i64 n, hipStream_t s);
template <typename T>
hipError_t pair_transpose(const void *in, void *out, int nk, int naux, int m, hipStream_t s);
// out[k1][k2][Q][p0+p][q0+q] += in[k1][k2][Q][p][q] (complex128; the reverse of chol_slice)
hipError_t slice_add(const void *in, void *out, int nk, int naux, int n, int p0, int np, int q0, int nq,
                     hipStream_t s);
// g[ki][kj][ki][i][j][a][b] += c x[ki][i][a] y[kj][j][b] (complex128, oovv-class blocks)
hipError_t outer_oovv(void *g, const void *x, const void *y, double c, int nk, int o, int v, hipStream_t s);
}  // namespace lrcc
