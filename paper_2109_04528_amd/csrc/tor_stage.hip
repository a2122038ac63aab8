// tor_stage.hip -- device staging of the input matrices, and sqrt(det(I - O)).
//
// One workgroup per matrix turns the caller's O (2n x 2n complex128,
// row-major, only its lower triangle read) into the layout a kernel reads:
//   * C = I - O as the Hermitian completion of its lower triangle;
//   * validation: every value read must be finite, and with
//     STAGE_CHECK_HERM the upper triangle must be the conjugate transpose of
//     the lower one (to 1e-12 relative);
//   * the Gaussian-state structure test.  The sampling matrix of a Gaussian
//     state in block order has the form [[P, Q], [conj Q, conj P]] with Q
//     symmetric (Sec. 1: A = I - Sigma^-1 from the Husimi covariance), and so
//     has C.  For such C the unitary w = [[1, 1], [-i, i]] / sqrt(2) applied
//     to every mode pair turns each 2x2 mode block [[p, q], [conj q, conj p]]
//     into the real block [[Re p + Re q, Im q - Im p], [Im p + Im q,
//     Re p - Re q]]; the result is real symmetric, and every principal
//     mode-submatrix keeps its determinant (w is unitary and acts inside
//     each mode), so the Torontonian is unchanged.  C is taken as structured
//     when both relations hold to 64 units of roundoff of max |C|; it is then
//     symmetrised exactly (P <- (P + conj P)/2 of the two diagonal blocks,
//     Q <- (Q + Q^T)/2) before the transform;
//   * packing: the node layout of tor_internal.hpp (real form in FP64, or in
//     double-double built from O itself for the double-double factor, or
//     the complex matrix), padded to the kernel's minimum size with
//     decoupled modes whose block of I - O is I/2 (such a mode multiplies the
//     Torontonian by 1/sqrt(1/4) - 1 = 1); or, for the removal-order kernel,
//     the complex matrix in the interleaved order a_0, a_0^dag, a_1, ... of
//     Sec. 2, lower triangle packed by rows.
// Positive definiteness is not tested here: every kernel tests the pivots
// of each subset it factorises, and the all-include subset is I - O itself.
//
// A pattern (sel) stages the principal submatrix of an M-mode O on the rows
// and columns {s, s + M : s in sel}, the matrix of a click pattern.
#include <cfloat>

#include "tor_stage.hpp"

namespace tor {

template <int NT>
__global__ void __launch_bounds__(NT) tor_stage(const StageDesc *descs)
{
    __shared__ c64 tri[STAGE_LDS_ENTRIES];
    stage_matrix<NT, STAGE_LDS_ENTRIES>(descs[blockIdx.x], tri);
}

// one matrix, its descriptor a kernel argument; clears the queue heads of the
// launches that follow
template <int NT>
__global__ void __launch_bounds__(NT) tor_stage_one(StageDesc D, unsigned long long *zero, int nzero)
{
    if ((int)threadIdx.x < nzero)
        zero[threadIdx.x] = 0ull;
    __shared__ c64 tri[STAGE_LDS_ENTRIES];
    stage_matrix<NT, STAGE_LDS_ENTRIES>(D, tri);
}

// A pivot whose determinant (or a square on the way to it) leaves the range of
// a double, entry by entry: an infinite one (of an input that is rejected only
// where a pattern holds it) divides its rows to nothing, as in a Cholesky
// factorisation.  root: of the determinant; false if the second pivot is not
// positive.
__device__ __forceinline__ bool wide_pivot(double a, c64 b, double g, Piv<c64> &pv, double &root)
{
    pv.inv_a = isinf(a) ? 0.0 : 1.0 / a;
    pv.ba = scale(b, pv.inv_a);
    const double g1 = g - (b.x * pv.ba.x + b.y * pv.ba.y);
    pv.inv_g = isinf(g1) ? 0.0 : 1.0 / g1;
    root = sqrt(a) * sqrt(g1);
    return g1 > 0.0;
}

// sqrt(det(I - O)) of an M-mode O (device, leading dimension ld, 0: packed
// lower triangle), M <= STAGE_LDS_MODES: the Hermitian completion of the lower
// triangle of C = I - O, its rows reordered to mode pairs, is eliminated in
// LDS one mode (2x2 pivot) at a time, from the last to the first.  A step
// rewrites only blocks of the modes that remain, each by the thread that
// reads it, so it needs one barrier; every thread forms the pivot itself.
// out[0] receives the root of the product of the pivots' determinants, out[1]
// = 1 when a pivot was not positive (or not a number).  What bounds it is the
// chain of M such steps, about 0.3 us each.
// A: entry e of block (a, b), a >= b, at [e][bidx(a, b)].
typedef c64 DetBlocks[NB(STAGE_LDS_MODES)];
template <int NT>
__device__ __forceinline__ void sqrt_det_lds(const double *O, long ld, int M, double *out, DetBlocks *A)
{
    const int t = threadIdx.x;
    const View v{O, ld, M, nullptr, M, nullptr};
    for (int q = t; q < 4 * NB(M); q += NT) {
        int a, b;
        block_ab(q >> 2, a, b);
        const int e = q & 3, ci = e >> 1, cj = e & 1;
        A[e][q >> 2] = v.c(a + ci * M, b + cj * M);
    }
    __syncthreads();
    double prod = 1.0;
    bool bad = false;
    for (int m = M - 1; m >= 0; --m) {
        const int d = bidx(m, m);
        const double al = A[0][d].x;
        Piv<c64> pv = pivot<c64>(al, A[2][d], A[3][d].x);
        double root = sqrt(pv.pdet);
        bool ok = pv.pdet > 0.0;
        // the same in every lane: a scalar branch
        if (__builtin_amdgcn_readfirstlane(!isfinite(pv.pdet) || fabs(pv.pdet) < DBL_MIN))
            ok = wide_pivot(al, A[2][d], A[3][d].x, pv, root);
        if (!(al > 0.0) || !ok)
            bad = true;
        prod *= root;
        for (int bi = t; bi < NB(m); bi += NT) {
            int a, b;
            block_ab(bi, a, b);
            c64 x[4], y[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                x[e] = A[e][bidx(m, a)];
                y[e] = A[e][bidx(m, b)];
            }
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                // rows of the LDL form of the pivot: r1, and r2 - r1 beta / alpha
                x[2 + c] = sub_mul(x[2 + c], x[c], pv.ba);
                y[2 + c] = sub_mul(y[2 + c], y[c], pv.ba);
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int c = e >> 1, f = e & 1;
                A[e][bi] = upd(A[e][bi], scale(x[c], pv.inv_a), y[f], scale(x[2 + c], pv.inv_g), y[2 + f]);
            }
        }
        __syncthreads();
    }
    if (t == 0) {
        out[0] = prod;
        out[1] = bad ? 1.0 : 0.0;
    }
}

template <int NT>
__global__ void __launch_bounds__(NT) tor_sqrt_det_lds(const double *O, long ld, int M, double *out)
{
    __shared__ DetBlocks A[4];
    sqrt_det_lds<NT>(O, ld, M, out, A);
}

// A state whose every pattern is wanted: staged by one workgroup while a
// second one forms sqrt(det(I - O)), which alone takes longer than the staging
// (at 15 modes one launch of 12 us in place of 6.5 + 11 and the gap between
// them); clears the queue head of the launch that follows.
template <int NT, int DET_NT>
__global__ void __launch_bounds__(NT) tor_stage_det(StageDesc D, unsigned long long *zero, double *det)
{
    static_assert(DET_NT <= NT, "");
    constexpr int SZ = STAGE_LDS_ENTRIES > 4 * NB(STAGE_LDS_MODES) ? STAGE_LDS_ENTRIES : 4 * NB(STAGE_LDS_MODES);
    __shared__ c64 buf[SZ];
    if (blockIdx.x == 0) {
        if (threadIdx.x == 0)
            *zero = 0ull;
        stage_matrix<NT, STAGE_LDS_ENTRIES>(D, buf);
    } else {
        if (__builtin_amdgcn_readfirstlane((int)threadIdx.x) >= DET_NT)
            return;  // whole waves: a barrier waits for the others alone
        sqrt_det_lds<DET_NT>(D.O, D.ld, D.M, det, reinterpret_cast<DetBlocks *>(buf));
    }
}

// the same for more modes, by a Cholesky factorisation in the caller's scratch
// (2M x 2M c64): the product of the diagonal of L.  One workgroup, two
// barriers per column.
template <int NT>
__global__ void __launch_bounds__(NT) tor_sqrt_det(const double *O, long ld, int M, c64 *A, double *out)
{
    const int t = threadIdx.x, m2 = 2 * M;
    const View v{O, ld, M, nullptr, M, nullptr};
    for (int q = t; q < m2 * m2; q += NT) {
        const int a = q / m2, b = q - a * m2;
        if (a >= b)
            A[(size_t)a * m2 + b] = v.c(a, b);
    }
    __syncthreads();
    double prod = 1.0;
    bool bad = false;
    for (int j = 0; j < m2; ++j) {
        const double d = A[(size_t)j * m2 + j].x;
        if (!(d > 0.0))
            bad = true;
        const double ljj = sqrt(d);
        prod *= ljj;
        const double inv = 1.0 / ljj;
        // column j of L, then the trailing update of the lower triangle
        for (int i = j + 1 + t; i < m2; i += NT) {
            c64 &x = A[(size_t)i * m2 + j];
            x = c64{x.x * inv, x.y * inv};
        }
        __syncthreads();
        const int r = m2 - j - 1;
        for (int q = t; q < r * (r + 1) / 2; q += NT) {
            int a, b;
            block_ab(q, a, b);
            a += j + 1;
            b += j + 1;
            const c64 la = A[(size_t)a * m2 + j], lb = A[(size_t)b * m2 + j];
            c64 &x = A[(size_t)a * m2 + b];
            // x -= la * conj(lb)
            x.x -= la.x * lb.x + la.y * lb.y;
            x.y -= la.y * lb.x - la.x * lb.y;
        }
        __syncthreads();
    }
    if (t == 0) {
        out[0] = prod;
        out[1] = bad ? 1.0 : 0.0;
    }
}

constexpr int STAGE_THREADS = 1024;
constexpr int DET_THREADS = 1024;
// 512 threads hold the blocks of 31 modes at one each
constexpr int DET_LDS_THREADS = 512;

hipError_t launch_stage(const StageDesc *descs, int count, hipStream_t s)
{
    if (count <= 0)
        return hipSuccess;
    hipLaunchKernelGGL((tor_stage<STAGE_THREADS>), dim3(count), dim3(STAGE_THREADS), 0, s, descs);
    return hipGetLastError();
}

hipError_t launch_stage_one(const StageDesc &d, unsigned long long *zero, int nzero, hipStream_t s)
{
    // a thread per entry of the lower triangle: fewer waves meet at fewer
    // barriers (n = 10: 5.7 us against 6.1)
    if (d.n <= 11)
        hipLaunchKernelGGL((tor_stage_one<256>), dim3(1), dim3(256), 0, s, d, zero, nzero);
    else
        hipLaunchKernelGGL((tor_stage_one<STAGE_THREADS>), dim3(1), dim3(STAGE_THREADS), 0, s, d, zero, nzero);
    return hipGetLastError();
}

hipError_t launch_stage_det(const StageDesc &d, unsigned long long *zero, double *det, hipStream_t s)
{
    if (d.M > STAGE_LDS_MODES || d.sel)
        return hipErrorInvalidValue;
    hipLaunchKernelGGL((tor_stage_det<STAGE_THREADS, DET_LDS_THREADS>), dim3(2), dim3(STAGE_THREADS), 0, s, d, zero, det);
    return hipGetLastError();
}

hipError_t launch_sqrt_det(const double *O, long ld, int M, c64 *scratch, double *out, hipStream_t s)
{
    if (M <= STAGE_LDS_MODES) {
        hipLaunchKernelGGL((tor_sqrt_det_lds<DET_LDS_THREADS>), dim3(1), dim3(DET_LDS_THREADS), 0, s, O, ld, M, out);
        return hipGetLastError();
    }
    hipLaunchKernelGGL((tor_sqrt_det<DET_THREADS>), dim3(1), dim3(DET_THREADS), 0, s, O, ld, M, scratch, out);
    return hipGetLastError();
}

}  // namespace tor
