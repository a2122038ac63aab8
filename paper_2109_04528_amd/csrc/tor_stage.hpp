// tor_stage.hpp -- the staging of one matrix by one workgroup (tor_stage.hip says
// what it does), for the staging kernels and for those that stage the matrix they
// work on.
#pragma once
#include "tor_device.hpp"
#include "tor_internal.hpp"

namespace tor {

namespace {

constexpr double kStageU = 1.1102230246251565e-16;  // FP64 unit roundoff

// the input seen as a 2n x 2n matrix (ld 0: its lower triangle packed by rows);
// with lds set, its lower triangle is read from there (packed by rows, pidx)
// instead of global memory
struct View {
    const double *O;
    long ld;
    int n;
    const int *sel;
    int M;
    const c64 *lds;
    __device__ int row(int a) const { return sel ? (a < n ? sel[a] : sel[a - n] + M) : a; }
    __device__ c64 og(int a, int b) const
    {
        // a host matrix is read across the bus, one 16-byte access per entry
        const size_t at = ld ? (size_t)row(a) * (size_t)ld + (size_t)row(b) : (size_t)pidx(row(a), row(b));
        typedef double dv2 __attribute__((ext_vector_type(2), aligned(8)));  // O is 8-byte aligned, no more
        const dv2 v = *(const dv2 *)(O + 2 * at);
        return c64{v.x, v.y};
    }
    // entry (a, b), a >= b, of O
    __device__ c64 o(int a, int b) const { return lds ? lds[pidx(a, b)] : og(a, b); }
    // C = I - O, Hermitian completion of the lower triangle
    __device__ c64 c(int a, int b) const
    {
        if (a >= b) {
            const c64 v = o(a, b);
            return a == b ? c64{1.0 - v.x, 0.0} : c64{-v.x, -v.y};
        }
        const c64 v = o(b, a);
        return c64{-v.x, v.y};
    }
};

// host-order double-double helpers for the double-double form
struct hd {
    double hi, lo;
};
__device__ inline hd two_sum(double a, double b)
{
#pragma clang fp contract(off)
    const double s = a + b, bb = s - a;
    return hd{s, (a - (s - bb)) + (b - bb)};
}
__device__ inline hd hd_add(hd a, hd b)
{
#pragma clang fp contract(off)
    hd s = two_sum(a.hi, b.hi);
    const hd t = two_sum(a.lo, b.lo);
    s.lo += t.hi;
    s = two_sum(s.hi, s.lo);
    s.lo += t.lo;
    return two_sum(s.hi, s.lo);
}
__device__ inline hd hd_neg(hd a) { return hd{-a.hi, -a.lo}; }
__device__ inline hd hd_half(hd a) { return hd{0.5 * a.hi, 0.5 * a.lo}; }

// entry (a, b) of I - O in double-double
__device__ inline void c_dd(const View &v, int a, int b, hd &re_, hd &im_)
{
    const bool up = a < b;
    const int i = up ? b : a, j = up ? a : b;
    const c64 x = v.o(i, j);
    re_ = two_sum(i == j ? 1.0 : 0.0, -x.x);
    im_ = hd{i == j ? 0.0 : (up ? x.y : -x.y), 0.0};
}

// real form entry: modes (mi, mj), components (ci, cj), of the symmetrised C
__device__ inline double real_entry(const View &v, int mi, int mj, int ci, int cj)
{
    const int n = v.n;
    const c64 p1 = v.c(mi, mj), p2 = v.c(mi + n, mj + n);
    const c64 q1 = v.c(mi, mj + n), q2 = v.c(mj, mi + n);
    const double pr = 0.5 * (p1.x + p2.x);
    const double pi = 0.5 * (p1.y - p2.y);
    const double qr = 0.5 * (q1.x + q2.x);
    const double qi = 0.5 * (q1.y + q2.y);
    if (ci == 0 && cj == 0)
        return pr + qr;
    if (ci == 0 && cj == 1)
        return qi - pi;
    if (ci == 1 && cj == 0)
        return pi + qi;
    return pr - qr;
}

__device__ inline hd quad_entry(const View &v, int mi, int mj, int ci, int cj)
{
    const int n = v.n;
    hd p1r, p1i, p2r, p2i, q1r, q1i, q2r, q2i;
    c_dd(v, mi, mj, p1r, p1i);
    c_dd(v, mi + n, mj + n, p2r, p2i);
    c_dd(v, mi, mj + n, q1r, q1i);
    c_dd(v, mj, mi + n, q2r, q2i);
    const hd pr = hd_half(hd_add(p1r, p2r)), pi = hd_half(hd_add(p1i, hd_neg(p2i)));
    const hd qr = hd_half(hd_add(q1r, q2r)), qi = hd_half(hd_add(q1i, q2i));
    if (ci == 0 && cj == 0)
        return hd_add(pr, qr);
    if (ci == 0 && cj == 1)
        return hd_add(qi, hd_neg(pi));
    if (ci == 1 && cj == 0)
        return hd_add(pi, qi);
    return hd_add(pr, hd_neg(qr));
}

__device__ inline double sq(double x, double y) { return x * x + y * y; }

// v with the lane's neighbour under a DPP pattern (lanes without one get 0)
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_or_zero(double v)
{
    const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)u, CTRL, ROWS, 0xf, false);
    const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(u >> 32), CTRL, ROWS, 0xf, false);
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// Block-wide maxima of the K non-negative values v (infinity included; no
// NaN): every thread receives them.  best[K] is zero, and a barrier has passed
// since.  Within a wave by DPP moves on the vector unit, then one LDS atomic
// per wave on the bit patterns, whose order is that of non-negative doubles:
// lane shuffles and a read of every wave's maximum went through LDS 960 times
// per workgroup, which took longer than all else the kernel does.
template <int K>
__device__ __forceinline__ void block_max(double (&v)[K], unsigned long long *best)
{
#pragma unroll
    for (int k = 0; k < K; ++k) {
        v[k] = fmax(v[k], dpp_or_zero<0x111, 0xf>(v[k]));  // row_shr:1
        v[k] = fmax(v[k], dpp_or_zero<0x112, 0xf>(v[k]));  // row_shr:2
        v[k] = fmax(v[k], dpp_or_zero<0x114, 0xf>(v[k]));  // row_shr:4
        v[k] = fmax(v[k], dpp_or_zero<0x118, 0xf>(v[k]));  // row_shr:8
        v[k] = fmax(v[k], dpp_or_zero<0x142, 0xa>(v[k]));  // row_bcast:15
        v[k] = fmax(v[k], dpp_or_zero<0x143, 0xc>(v[k]));  // row_bcast:31
    }
    if ((threadIdx.x & 63) == 63)
#pragma unroll
        for (int k = 0; k < K; ++k)
            atomicMax(&best[k], __builtin_bit_cast(unsigned long long, v[k]));
    __syncthreads();
#pragma unroll
    for (int k = 0; k < K; ++k)
        v[k] = __builtin_bit_cast(double, best[k]);
}

}  // namespace

// lower-triangle entries staged in LDS (51.8 KB); larger inputs are read from
// global memory throughout
constexpr int STAGE_LDS_ENTRIES = NB(2 * STAGE_LDS_MODES);

// One matrix, staged by the NT threads of a workgroup with CAP entries of LDS
// (tri).  What bounds it is latency: one pass
// over the input (across the bus for a host matrix), one block-wide maximum,
// one pass over the output.
template <int NT, int CAP>
__device__ __forceinline__ void stage_matrix(const StageDesc &D, c64 *tri)
{
    __shared__ unsigned long long best[5];
    const int t = threadIdx.x;
    if (t < 5)
        best[t] = 0ull;
    const int n = D.n, n2 = 2 * n;
    const bool in_lds = NB(n2) <= CAP;
    View v{D.O, D.ld, n, D.sel, D.M, nullptr};
    const unsigned fl = D.flags;

    // one pass over global memory: validation, max |C|, the Hermitian check,
    // and the lower triangle of O into LDS (a NaN fails every comparison
    // below, so it is caught by the finite test alone)
    double nonfin = 0.0, cmax2 = 0.0, dev2 = 0.0, hs2 = 0.0, hd2 = 0.0;
    const bool herm = (fl & STAGE_CHECK_HERM) != 0;
    auto lower = [&](int q, int a, int b) {
        const c64 x = v.og(a, b);
        if (!isfinite(x.x) || !isfinite(x.y))
            nonfin = 1.0;
        const c64 y = a == b ? c64{1.0 - x.x, 0.0} : c64{-x.x, -x.y};
        cmax2 = fmax(cmax2, sq(y.x, y.y));
        if (in_lds)
            tri[q] = x;
    };
    if (!herm) {
        // the lower triangle only, entry q = pidx(a, b)
        for (int q = t; q < NB(n2); q += NT) {
            int a, b;
            block_ab(q, a, b);
            lower(q, a, b);
        }
    } else {
        for (int q = t; q < n2 * n2; q += NT) {
            const int a = q / n2, b = q - a * n2;
            if (a >= b)
                lower(pidx(a, b), a, b);
            const c64 x = v.og(a, b), y = v.og(b, a);
            if (!isfinite(x.x) || !isfinite(x.y))
                nonfin = 1.0;
            hs2 = fmax(hs2, sq(x.x, x.y));
            hd2 = fmax(hd2, sq(x.x - y.x, x.y + y.y));
        }
    }
    __syncthreads();
    if (in_lds)
        v.lds = tri;
    const bool interleaved = (fl & STAGE_INTERLEAVED) != 0;
    const bool dd = (fl & STAGE_DD) != 0;
    const bool want_real = !interleaved && (dd || (n > 0 && !(fl & STAGE_FORCE_CPLX)));
    if (want_real) {
        for (int q = t; q < n * n; q += NT) {
            const int i = q / n, j = q - i * n;
            // lower-right block = conj(upper-left); lower-left block symmetric
            const c64 d1a = v.c(i + n, j + n), d1b = v.c(i, j);
            const c64 d2a = v.c(i + n, j), d2b = v.c(j + n, i);
            dev2 = fmax(dev2, sq(d1a.x - d1b.x, d1a.y + d1b.y));
            dev2 = fmax(dev2, sq(d2a.x - d2b.x, d2a.y - d2b.y));
        }
    }
    double mx[3] = {nonfin, cmax2, dev2}, mh[2] = {hs2, hd2};
    block_max(mx, best);
    nonfin = mx[0];
    cmax2 = mx[1];
    dev2 = mx[2];
    if (herm) {
        block_max(mh, best + 3);
        hs2 = mh[0];
        hd2 = mh[1];
    }
    const double tol = 64.0 * kStageU * fmax(sqrt(cmax2), 1.0);
    const bool structured = want_real && dev2 <= tol * tol;
    int status = 0;
    if (nonfin != 0.0 || (herm && hd2 > 1e-24 * fmax(hs2, 1.0)) || (dd && !structured))
        status = STAGE_BAD_INPUT;
    const int path = structured ? (dd ? PATH_QUAD : PATH_REAL) : PATH_CPLX;
    const int N = interleaved ? n
                  : path == PATH_REAL ? max(n, REAL_R)
                  : path == PATH_QUAD ? max(n, QUAD_R)
                                      : max(n, D.min_cplx);
    if (t == 0)
        *D.info = StageInfo{status, status ? -1 : path, N, 0, sqrt(cmax2)};
    if (status != 0)
        return;

    if (interleaved) {
        // the removal-order layout: row x = 2 q + c is a_q (c = 0) or a_q^dag
        c64 *out = (c64 *)D.out;
        for (int q = t; q < NB(n2); q += NT) {
            int x, y;
            block_ab(q, x, y);
            out[pidx(x, y)] = v.c((x >> 1) + (x & 1) * n, (y >> 1) + (y & 1) * n);
        }
        return;
    }
    // node layout: block bi = (a, b) of the reversed interleaved rows
    const int nb = NB(N);
    for (int q = t; q < 4 * nb; q += NT) {
        const int bi = q >> 2, e = q & 3;
        int a, b;
        block_ab(bi, a, b);
        const int x = 2 * a + (e >> 1), y = 2 * b + (e & 1);
        const int qi = 2 * N - 1 - x, qj = 2 * N - 1 - y;
        const int mi = qi >> 1, ci = qi & 1, mj = qj >> 1, cj = qj & 1;
        const bool padm = mi >= n || mj >= n;
        if (path == PATH_REAL) {
            const double val = padm ? (qi == qj ? 0.5 : 0.0) : real_entry(v, mi, mj, ci, cj);
            ((double *)D.out)[gpos((int)sizeof(double), nb, bi, e)] = val;
        } else if (path == PATH_QUAD) {
            const hd val = padm ? hd{qi == qj ? 0.5 : 0.0, 0.0} : quad_entry(v, mi, mj, ci, cj);
            ((ddr *)D.out)[gpos((int)sizeof(ddr), nb, bi, e)] = ddr{val.hi, val.lo};
        } else {
            c64 val = padm ? c64{qi == qj ? 0.5 : 0.0, 0.0} : v.c(mi + ci * n, mj + cj * n);
            if (x == y)
                val.y = 0.0;
            ((c64 *)D.out)[gpos((int)sizeof(c64), nb, bi, e)] = val;
        }
    }
}

}  // namespace tor
