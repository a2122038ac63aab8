// tor_zeta.hip -- click probabilities of every pattern of one state at once.
//
// The probability that threshold detectors click exactly on the modes S of a
// Gaussian state is p(S) = Tor(O_S) sqrt(det(I - O)) (Sec. 1), and Tor(O_S)
// is Eq. 2 for the principal submatrix O_S: a signed sum of
// 1/sqrt(det (I - O)_Z) over the subsets Z of S.  Every pattern therefore
// draws its terms from the same 2^M subset determinants of I - O.  One launch
// of the recursive kernel over the whole state stores each signed term
//     t[Z] = (-1)^(N-|Z|) / sqrt(det (I - O)_Z)
// (N the modes of the staged form, index bit N-1-l = the decision at level l,
// which is mode l), so every prefix factor of the state is formed once for all
// patterns.  The subset sums
//     g[S] = sum over Z subset of S of t[Z]
// (the zeta transform over the subset lattice) then give every pattern at
// once: Tor(O_S) = (-1)^(N-|S|) g[S].  That is 2^M determinants and M passes
// of additions over 2^M entries, against 3^M determinants for the patterns
// one by one.
//
// The transform adds along one index bit at a time (g[S] += g[S without bit b]
// for every S with bit b set).  What bounds it is memory: every pass reads and
// writes all 2^M sums, so a call takes as few as it can:
//   * the low 10 or 12 bits in one workgroup per block of 1024 or 4096 entries,
//     its threads adding along a few bits in registers and exchanging the
//     block through LDS between those rounds (tor_zeta_lds_r);
//   * the highest 3 to 8 bits together with the output (tor_zeta_tile): a
//     workgroup takes 2^HB x 2^CB entries, HB + CB = 12, that differ in the HB
//     highest and the CB lowest bits, adds along the high ones, and writes the
//     patterns: reversed, the high bits are a pattern's lowest, so what was
//     read in runs of 2^CB entries (256 B at least) is written in runs of 2^HB
//     patterns, and the sums are not stored once more to be permuted;
//   * the bits between, if any, up to 5 in registers alone (tor_zeta_bits) or
//     6 to 8 by tiles.
// At M = 25 that is 12 + 5 + 8 bits in three passes against 10 + 5 + 5 + 5 and
// a permutation, 2.9 GB against 5.1 with the terms, 569 us against 980 (5.0, 5.2 and
// 4.0 TB/s; a 1 GiB copy moves 4.8); at M = 32 12 + 4 +
// 8 + 8 in four against six passes.
//
// Exactness: for a Gaussian state every subset determinant is at most 1
// (sqrt(det(I - O)) / sqrt(det (I - O)_Z) is the probability that no mode
// outside Z clicks, at least the probability sqrt(det(I - O)) that none
// does), so every term is a double of magnitude at least 1, a multiple of
// 2^-52, and the additions are double-double sums built from error-free ones
// (Knuth's TwoSum, Dekker's Fast2Sum) alone.  While a partial sum stays below
// 2^53 in magnitude, every intermediate quantity is a multiple of 2^-52 that fits
// its double, so every g[S] is the exact sum of its terms, whatever the order.
// Beyond that (brighter states: 24 modes at r = 2 have a sum of |t| of 2^54) the
// additions still keep both low parts; a shorter one that rounds their sum, 14
// operations, is 0.5 % of a call faster (25 modes 746 us, 749) and loses a bit
// of the sums there.
#include "tor_internal.hpp"

namespace tor {

namespace {

constexpr int ZB_MAX = 12;  // most index bits of the first stage, and of a tile (4096 entries)
constexpr int ZG = 5;       // index bits per global pass
__device__ __forceinline__ void two_sum(double a, double b, double &s, double &e)
{
    s = a + b;
    const double bb = s - a;
    e = (a - (s - bb)) + (b - bb);
}

// a + b exactly, |a| >= |b| or a = 0 (Dekker)
__device__ __forceinline__ void fast_two_sum(double a, double b, double &s, double &e)
{
    s = a + b;
    e = b - (s - a);
}

// a + b in double-double to 3 * 2^-106 of the result, from error-free sums
// (AccurateDWPlusDW of Joldes, Muller and Popescu, 2017: 20 operations)
__device__ __forceinline__ void dd_acc(double &ah, double &al, double bh, double bl)
{
    double s, e, t, f;
    two_sum(ah, bh, s, e);
    two_sum(al, bl, t, f);
    e += t;
    fast_two_sum(s, e, s, e);
    e += f;
    fast_two_sum(s, e, ah, al);
}

// Where a click call's outputs go (null: not wanted).  full: the sum of the
// pattern of every mode.  go: 0 where an earlier step of the call failed (null:
// there is none); the kernels then leave everything as it is, so that the whole
// call is enqueued at once (a wait for the verdict between the recursive kernel
// and the transform left the device idle for 10 us).
struct ClickOut {
    const double *sqrt_det;
    double *probs, *tor_hi, *tor_lo;
    ddr *full;
    const double *go;
};
__device__ __forceinline__ bool stopped(const double *go) { return go && *go == 0.0; }

// bits 0 .. nb-1 of a block of 2^nb entries (nb <= ZB), one bit at a time in
// LDS, terms in, double-double out; ZT threads
template <int ZB, int ZT>
__global__ void __launch_bounds__(ZT) tor_zeta_lds(const double *t, ddr *g, int nb, const double *go)
{
    if (stopped(go))
        return;
    __shared__ double hs[1 << ZB], ls[1 << ZB];
    const int size = 1 << nb;
    const long long base = (long long)blockIdx.x << nb;
    for (int i = threadIdx.x; i < size; i += ZT) {
        hs[i] = t[base + i];
        ls[i] = 0.0;
    }
    __syncthreads();
    for (int b = 0; b < nb; ++b) {
        const int low = (1 << b) - 1;
        for (int p = threadIdx.x; p < size / 2; p += ZT) {
            const int i1 = ((p & ~low) << 1) | (1 << b) | (p & low);  // the p-th index with bit b set
            const int i0 = i1 ^ (1 << b);
            double h = hs[i1], l = ls[i1];
            dd_acc(h, l, hs[i0], ls[i0]);
            hs[i1] = h;
            ls[i1] = l;
        }
        __syncthreads();
    }
    for (int i = threadIdx.x; i < size; i += ZT)
        g[base + i] = ddr{hs[i], ls[i]};
}

// All ZB bits of a block of 2^ZB entries, with the additions in registers:
// each of the ZT threads holds E = 2^RB entries that differ only in RB index
// bits and adds along those bits; between rounds (bits from the highest down)
// the block moves through LDS so that each thread holds the entries of the
// next RB bits.  Per entry that is 4 doubles of LDS traffic per round and
// two barriers, against 3 doubles and one barrier per bit.  The LDS index is
// XOR-swizzled within each run of 16 entries, i ^ ((i >> RB) & 15), which
// leaves no two of the 16 lanes that one cycle of a 64-bit access serves on
// the same bank in any round or in the final copy.  The first round reads
// the terms straight from global memory (consecutive lanes, consecutive
// entries); the last one goes out through LDS so that the double-double
// sums are written in consecutive runs.  Terms in, double-double out.  At
// M = 32, 256 threads of 16 entries gave 159.8 ms per call, 512 of 8 161.0, 1024
// of 4 164.8, one bit at a time 167.5 to 168.8 (M = 24: 0.56 against 0.58 ms).
template <int ZB, int ZT, int RB>
__global__ void __launch_bounds__(ZT) tor_zeta_lds_r(const double *t, ddr *g, const double *go)
{
    if (stopped(go))
        return;
    static_assert((ZT << RB) == (1 << ZB) && ZB % RB == 0, "a block is ZT threads of 2^RB entries");
    constexpr int E = 1 << RB;
    __shared__ double hs[1 << ZB], ls[1 << ZB];
    const long long base = (long long)blockIdx.x << ZB;
    const int q = threadIdx.x;
    auto sw = [](int i) { return i ^ ((i >> RB) & 15); };
    // entry j of thread q in the round of bits s .. s+RB-1
    auto idx = [&](int s, int j) { return (q & ((1 << s) - 1)) | (j << s) | ((q >> s) << (s + RB)); };
    double h[E], l[E];
#pragma unroll
    for (int j = 0; j < E; ++j) {
        h[j] = t[base + idx(ZB - RB, j)];
        l[j] = 0.0;
    }
#pragma unroll
    for (int s = ZB - RB; s >= 0; s -= RB) {
#pragma unroll
        for (int b = 0; b < RB; ++b)
#pragma unroll
            for (int j = 0; j < E; ++j)
                if ((j >> b) & 1)
                    dd_acc(h[j], l[j], h[j ^ (1 << b)], l[j ^ (1 << b)]);
#pragma unroll
        for (int j = 0; j < E; ++j) {
            const int i = sw(idx(s, j));
            hs[i] = h[j];
            ls[i] = l[j];
        }
        __syncthreads();
        if (s == 0)
            break;
#pragma unroll
        for (int j = 0; j < E; ++j) {
            const int i = sw(idx(s - RB, j));
            h[j] = hs[i];
            l[j] = ls[i];
        }
        __syncthreads();  // every entry is read before the next round writes
    }
#pragma unroll
    for (int k = 0; k < E; ++k) {
        const int i = q + k * ZT;
        g[base + i] = ddr{hs[sw(i)], ls[sw(i)]};
    }
}

// bits b0 .. b0+nb-1 (nb <= ZG) over all 2^nbits entries: thread q holds the
// 2^nb entries whose index has q's bits below b0 and above b0+nb-1
// NT: streaming (non-temporal) loads and stores, for sums too large to stay
// in the caches between passes
template <bool NT>
__global__ void __launch_bounds__(256) tor_zeta_bits(ddr *g, int nbits, int b0, int nb, const double *go)
{
    if (stopped(go))
        return;
    const long long q = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= (1ll << (nbits - nb)))
        return;
    const long long lowm = (1ll << b0) - 1;
    const long long base = (q & lowm) | ((q & ~lowm) << nb);
    double h[1 << ZG], l[1 << ZG];
#pragma unroll
    for (int j = 0; j < (1 << ZG); ++j)
        if (j < (1 << nb)) {
            const double *pv = reinterpret_cast<const double *>(g + base + ((long long)j << b0));
            if constexpr (NT) {
                h[j] = __builtin_nontemporal_load(pv);
                l[j] = __builtin_nontemporal_load(pv + 1);
            } else {
                h[j] = pv[0];
                l[j] = pv[1];
            }
        }
#pragma unroll
    for (int b = 0; b < ZG; ++b)
        if (b < nb) {
#pragma unroll
            for (int j = 0; j < (1 << ZG); ++j)
                if (j < (1 << nb) && ((j >> b) & 1))
                    dd_acc(h[j], l[j], h[j ^ (1 << b)], l[j ^ (1 << b)]);
        }
#pragma unroll
    for (int j = 0; j < (1 << ZG); ++j)
        if (j < (1 << nb)) {
            if constexpr (NT) {
                double *pv = reinterpret_cast<double *>(g + base + ((long long)j << b0));
                __builtin_nontemporal_store(h[j], pv);
                __builtin_nontemporal_store(l[j], pv + 1);
            } else {
                g[base + ((long long)j << b0)] = ddr{h[j], l[j]};
            }
        }
}


// one pattern's outputs from its subset sum v
__device__ __forceinline__ void put_pattern(long long S, int N, int M, ddr v, double sq, const ClickOut &o)
{
    const double sg = ((N - __popcll((unsigned long long)S)) & 1) ? -1.0 : 1.0;
    if (o.tor_hi)
        o.tor_hi[S] = sg * v.hi;
    if (o.tor_lo)
        o.tor_lo[S] = sg * v.lo;
    if (o.probs)
        o.probs[S] = sg * (v.hi + v.lo) * sq;
    if (o.full && S == (1ll << M) - 1)
        *o.full = v;
}

// HB index bits from b0 up, over tiles of 2^HB x 2^CB entries that differ in
// those bits and in the CB = 12 - HB lowest: 256 threads of 16 entries, which
// add along the tile index's bits 8..11, exchange the tile through LDS, and
// add along what is left of bits 4..7.  OUT: these are the highest bits of the
// N; the tile goes through LDS once more and out as patterns, in runs of 2^HB
// (no padding modes: M = N).  Otherwise it goes back from the registers, in
// the runs of 2^CB it came in.  The LDS index is swizzled within each run of
// 16 by both nibbles above it, which keeps the 16 lanes that one cycle of a
// 64-bit access serves on different banks in the exchange (lanes differ in the
// lowest nibble) and in the output (consecutive patterns differ in the tile
// index's highest bits).
template <int HB, bool OUT, bool NT>
__global__ void __launch_bounds__(256) tor_zeta_tile(ddr *g, int N, int b0, ClickOut out)
{
    if (stopped(out.go))
        return;
    static_assert(HB >= 3 && HB <= 8, "two rounds of up to 4 bits, runs of 16 entries at least");
    constexpr int CB = ZB_MAX - HB, E = 16, RB = 4;
    __shared__ double hs[1 << ZB_MAX], ls[1 << ZB_MAX];
    const int q = threadIdx.x;
    const long long blk = blockIdx.x;
    const int mb = b0 - CB;  // bits between the tile's low and high ones
    const long long mid = blk & ((1ll << mb) - 1), up = blk >> mb;
    const long long base = (up << (b0 + HB)) | (mid << CB);
    auto sw = [](int i) { return i ^ (((i >> 4) ^ (i >> 8)) & 15); };
    auto idx = [&](int s, int j) { return (q & ((1 << s) - 1)) | (j << s) | ((q >> s) << (s + RB)); };
    auto at = [&](int i) { return base + ((long long)(i >> CB) << b0) + (i & ((1 << CB) - 1)); };
    double h[E], l[E];
#pragma unroll
    for (int j = 0; j < E; ++j) {
        const double *pv = reinterpret_cast<const double *>(g + at(idx(8, j)));
        if constexpr (NT) {
            h[j] = __builtin_nontemporal_load(pv);
            l[j] = __builtin_nontemporal_load(pv + 1);
        } else {
            h[j] = pv[0];
            l[j] = pv[1];
        }
    }
    constexpr bool TWO = CB < 8;
#pragma unroll
    for (int s = 8; s >= (TWO ? 4 : 8); s -= RB) {
#pragma unroll
        for (int b = 0; b < RB; ++b)
            if (s + b >= CB)
#pragma unroll
                for (int j = 0; j < E; ++j)
                    if ((j >> b) & 1)
                        dd_acc(h[j], l[j], h[j ^ (1 << b)], l[j ^ (1 << b)]);
        if (s == 8 && TWO) {
#pragma unroll
            for (int j = 0; j < E; ++j) {
                const int i = sw(idx(8, j));
                hs[i] = h[j];
                ls[i] = l[j];
            }
            __syncthreads();
#pragma unroll
            for (int j = 0; j < E; ++j) {
                const int i = sw(idx(4, j));
                h[j] = hs[i];
                l[j] = ls[i];
            }
        }
    }
    constexpr int SL = TWO ? 4 : 8;  // the layout the entries are in now
    if constexpr (!OUT) {
#pragma unroll
        for (int j = 0; j < E; ++j) {
            double *pv = reinterpret_cast<double *>(g + at(idx(SL, j)));
            if constexpr (NT) {
                __builtin_nontemporal_store(h[j], pv);
                __builtin_nontemporal_store(l[j], pv + 1);
            } else {
                pv[0] = h[j];
                pv[1] = l[j];
            }
        }
    } else {
        // every thread wrote and read the same entries in the exchange above
        // only in the second layout, so the tile can be overwritten in it
#pragma unroll
        for (int j = 0; j < E; ++j) {
            const int i = sw(idx(SL, j));
            hs[i] = h[j];
            ls[i] = l[j];
        }
        __syncthreads();
        const double sq = out.sqrt_det[0];
        const long long rmid = mb > 0 ? (long long)(__builtin_bitreverse64((unsigned long long)mid) >> (64 - mb)) : 0;
#pragma unroll
        for (int k = 0; k < E; ++k) {
            const int f = q + 256 * k;
            const int rh = f & ((1 << HB) - 1), rc = f >> HB;
            const int hh = (int)(__builtin_bitreverse32((unsigned)rh) >> (32 - HB));
            const int cc = (int)(__builtin_bitreverse32((unsigned)rc) >> (32 - CB));
            const int i = sw((hh << CB) | cc);
            const long long S = ((long long)rc << (N - CB)) | (rmid << HB) | rh;
            put_pattern(S, N, N, ddr{hs[i], ls[i]}, sq, out);
        }
    }
}

// Pattern S's sum sits at index bitreverse_N(S) (S's bit i is mode i, the
// decision at level i, index bit N-1-i).  Without padding modes (M = N) the
// permutation of a transform of one stage runs in tiles: a workgroup fixes the middle N-2A index bits,
// reads the 2^A x 2^A entries of its top and bottom A bits in runs of 2^A
// neighbours, and writes them out again in runs of 2^A neighbours of S
// through LDS (the top A bits of S are the bottom A bits of the index
// reversed, and the other way round).
constexpr int TA = 5;
__global__ void __launch_bounds__(256) tor_click_out_tiled(const ddr *g, int N, ClickOut out)
{
    if (stopped(out.go))
        return;
    __shared__ double th[1 << TA][(1 << TA) + 1], tl[1 << TA][(1 << TA) + 1];
    const long long mid = blockIdx.x;
    const int nm = N - 2 * TA;
    for (int q = threadIdx.x; q < (1 << (2 * TA)); q += 256) {
        const int h = q >> TA, l = q & ((1 << TA) - 1);
        const ddr v = g[((long long)h << (N - TA)) | (mid << TA) | l];
        th[h][l] = v.hi;
        tl[h][l] = v.lo;
    }
    __syncthreads();
    const long long rmid = nm > 0 ? (long long)(__builtin_bitreverse64((unsigned long long)mid) >> (64 - nm)) : 0;
    const double sq = out.sqrt_det[0];
    for (int q = threadIdx.x; q < (1 << (2 * TA)); q += 256) {
        const int rl = q >> TA, rh = q & ((1 << TA) - 1);
        const int h = (int)(__builtin_bitreverse32((unsigned)rh) >> (32 - TA));
        const int l = (int)(__builtin_bitreverse32((unsigned)rl) >> (32 - TA));
        const long long S = ((long long)rl << (N - TA)) | (rmid << TA) | rh;
        put_pattern(S, N, N, ddr{th[h][l], tl[h][l]}, sq, out);
    }
}

// one thread per pattern S < 2^M (any M <= N): a gather, for the padded forms
__global__ void __launch_bounds__(256) tor_click_out(const ddr *g, int N, int M, ClickOut out)
{
    if (stopped(out.go))
        return;
    const long long S = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (S >= (1ll << M))
        return;
    const unsigned long long idx = __builtin_bitreverse64((unsigned long long)S) >> (64 - N);
    put_pattern(S, N, M, g[idx], out.sqrt_det[0], out);
}

}  // namespace

namespace {

// the first nb bits (10 and 12 in registers and LDS, others bit by bit in LDS)
hipError_t first_stage(const double *t, ddr *g, int nbits, int nb, const double *go, hipStream_t s)
{
    const dim3 grid((unsigned)(1ll << (nbits - nb)));
    if (nb == 12)
        hipLaunchKernelGGL((tor_zeta_lds_r<12, 256, 4>), grid, dim3(256), 0, s, t, g, go);
    else if (nb == 10)
        hipLaunchKernelGGL((tor_zeta_lds_r<10, 256, 2>), grid, dim3(256), 0, s, t, g, go);
    else if (nb == 11)
        hipLaunchKernelGGL((tor_zeta_lds<11, 512>), grid, dim3(512), 0, s, t, g, nb, go);
    else
        hipLaunchKernelGGL((tor_zeta_lds<10, 256>), grid, dim3(256), 0, s, t, g, nb, go);
    return hipGetLastError();
}

// streaming accesses once the sums (16 B each) pass 1 GiB: at M = 28 and 32
// they took the register passes' call from 10.6 to 10.3 ms and from 159.6 to
// 156.0 ms, at M = 24 (268 MB, mostly held by the caches) from 0.56 to 0.59 ms
// the other way
bool streaming(int nbits) { return nbits >= 26; }

// bits b0 .. b0+w-1, w <= ZG, in registers
hipError_t bits_pass(ddr *g, int nbits, int b0, int w, const double *go, hipStream_t s)
{
    const long long threads = 1ll << (nbits - w);
    const dim3 grid((unsigned)((threads + 255) / 256));
    if (streaming(nbits))
        hipLaunchKernelGGL((tor_zeta_bits<true>), grid, dim3(256), 0, s, g, nbits, b0, w, go);
    else
        hipLaunchKernelGGL((tor_zeta_bits<false>), grid, dim3(256), 0, s, g, nbits, b0, w, go);
    return hipGetLastError();
}

template <int HB, bool OUT>
hipError_t tile_pass_hb(ddr *g, int nbits, int b0, const ClickOut &o, hipStream_t s)
{
    const dim3 grid((unsigned)(1ll << (nbits - ZB_MAX)));
    if (streaming(nbits))
        hipLaunchKernelGGL((tor_zeta_tile<HB, OUT, true>), grid, dim3(256), 0, s, g, nbits, b0, o);
    else
        hipLaunchKernelGGL((tor_zeta_tile<HB, OUT, false>), grid, dim3(256), 0, s, g, nbits, b0, o);
    return hipGetLastError();
}

// bits b0 .. b0+w-1, 3 <= w <= 8, by tiles (b0 >= 12 - w)
template <bool OUT>
hipError_t tile_pass(ddr *g, int nbits, int b0, int w, const ClickOut &o, hipStream_t s)
{
    switch (w) {
    case 3: return tile_pass_hb<3, OUT>(g, nbits, b0, o, s);
    case 4: return tile_pass_hb<4, OUT>(g, nbits, b0, o, s);
    case 5: return tile_pass_hb<5, OUT>(g, nbits, b0, o, s);
    case 6: return tile_pass_hb<6, OUT>(g, nbits, b0, o, s);
    case 7: return tile_pass_hb<7, OUT>(g, nbits, b0, o, s);
    case 8: return tile_pass_hb<8, OUT>(g, nbits, b0, o, s);
    default: return hipErrorInvalidValue;
    }
}

// bits b0 .. b1-1 in as few passes as there are: 8 by tiles, up to 5 in
// registers (which read and write nothing but their own entries, in longer
// runs), 6 and 7 by tiles
hipError_t middle(ddr *g, int nbits, int b0, int b1, const double *go, hipStream_t s)
{
    hipError_t e = hipSuccess;
    ClickOut o{};
    o.go = go;
    while (e == hipSuccess && b0 < b1) {
        const int left = b1 - b0, w = left <= ZG ? left : left <= 8 ? left : left <= 8 + ZG ? left - 8 : 8;
        e = w <= ZG ? bits_pass(g, nbits, b0, w, go, s) : tile_pass<false>(g, nbits, b0, w, o, s);
        b0 += w;
    }
    return e;
}

}  // namespace

static hipError_t subset_sums(const double *t, ddr *g, int nbits, const double *go, hipStream_t s)
{
    const int nb = nbits < ZB_MAX ? nbits : ZB_MAX;
    const hipError_t e = first_stage(t, g, nbits, nb, go, s);
    return e == hipSuccess ? middle(g, nbits, nb, nbits, go, s) : e;
}

hipError_t launch_zeta(const double *t, ddr *g, int nbits, hipStream_t s) { return subset_sums(t, g, nbits, nullptr, s); }

hipError_t launch_click_transform(const double *t, ddr *g, int N, int M, const double *det, double *probs,
                                  double *tor_hi, double *tor_lo, ddr *full, hipStream_t s)
{
    const ClickOut o{det, probs, tor_hi, tor_lo, full, det + 2};
    if (M == N && N >= 13) {
        // the last pass takes 8 bits, or what a first stage of 10 leaves (its
        // 1024-entry blocks keep more loads in flight than 4096-entry ones)
        const int last = N - 10 < 8 ? N - 10 : 8;
        const int first = N - last <= 10 ? 10 : ZB_MAX < N - last ? ZB_MAX : N - last;
        hipError_t e = first_stage(t, g, N, first, o.go, s);
        if (e == hipSuccess)
            e = middle(g, N, first, N - last, o.go, s);
        return e == hipSuccess ? tile_pass<true>(g, N, N - last, last, o, s) : e;
    }
    hipError_t e = subset_sums(t, g, N, o.go, s);
    if (e != hipSuccess)
        return e;
    if (M == N && N >= 2 * TA) {
        hipLaunchKernelGGL(tor_click_out_tiled, dim3((unsigned)(1ll << (N - 2 * TA))), dim3(256), 0, s, g, N, o);
        return hipGetLastError();
    }
    const long long n = 1ll << M;
    hipLaunchKernelGGL(tor_click_out, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, g, N, M, o);
    return hipGetLastError();
}

}  // namespace tor
