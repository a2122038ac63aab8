// tor_kernels.hip -- gfx950 kernels of the recursive Torontonian.
//
// Tor(O) = sum_Z (-1)^(n-|Z|) / sqrt(det (I-O)_Z)   (Eq. 2)
//
// The include/exclude tree over the modes (in order 0..N-1) enumerates every
// subset Z once; a node at level l has decided modes 0..l-1 and carries the
// Schur complement of its included modes over the undecided ones (packed
// layout described in tor_device.hpp).  Excluding the next mode is free (a
// prefix), including it is one rank-2 update whose pivot determinant
// multiplies the running determinant (the product of the new squared diagonal
// entries of the Cholesky factor).  A leaf is one subset: its term is
// (-1)^(#excluded) / sqrt(det).  This is the reuse of Sec. 2 / Algorithm 2 --
// a child only appends the two rows of its new mode to the parent's factor --
// in right-looking form, so each child costs O(remaining modes^2) instead of
// a fresh factorisation.
//
// Work split (one persistent launch, one wavefront per workgroup):
//  * queue items are subtree roots: the include/exclude decisions on modes
//    0..k-1 (the paper's MPI layer hands over only the list of modes and lets
//    the receiver recompute the factor, Sec. 4; here a wave pops a root id
//    from an atomic counter and recomputes the root's Schur complement);
//  * tier A: the wave walks the levels k..N-R-1 depth first; each step that
//    changes the path is one wave-parallel rank-2 update, stacked per level
//    in a private global scratch area (L2-resident).  On the real path the
//    node one level above the tier-A leaf (R+1 modes) is kept whole in LDS,
//    so the last tier-A level is included in place in LDS and has no stack
//    slot;
//  * tier B: from each tier-A leaf (R = T + B modes left) the wave expands
//    B-L levels breadth first in LDS, every include node of a level updated
//    together (all lanes busy);
//  * tier C: lane l takes node l of level B.  Its ancestor of level B-L is
//    an LDS node; the lane makes the last L decisions itself (an exclude is
//    a zero update, so all lanes run the same code), fused into one pass over
//    that node, and finishes the last T modes alone in registers: 2^T
//    subsets per lane.
// Terms are summed per lane in double-double, reduced over the wave, and
// written to the root's partial slot; a second kernel sums the slots of each
// matrix in a fixed order (the last wave of a lone evaluation of few roots does).
// The double-double factor's instantiation of the main kernel is built in
// tor_kernels_quad.hip, and the one-launch form of the smallest evaluations in
// tor_small.hip; both include this file with TOR_KERNELS_TEMPLATES_ONLY defined
// (templates only, no launchers).
#include <type_traits>

#include "tor_device.hpp"
#include "tor_internal.hpp"

namespace tor {

// ---------------------------------------------------------------------------
// LDS placement of the nodes tier B stores: node 0 is the tier-A leaf (R
// modes), node 2^(j-1) + i the include node i of level j (R - j modes), for
// j = 1..BL.  Nodes follow one another in that order, each on a 16-byte
// boundary.  Tier C reads the same entry of all 2^BL nodes in one
// instruction, 2^L lanes per node (lane l reads the node that level-BL view
// l >> L stands for).  LDS serves such an access in groups of lanes that move
// 128 bytes per cycle (256 with 64 banks), and two lanes of one group that
// touch different words of one bank wait for each other.  Each node is
// therefore moved forward (by at most 15 granules) to the first place where
// the start of each of its granule arrays, as a 16-byte slot modulo 8 (and
// modulo 16), differs from that of the other nodes read by the same group of
// lanes; failing that, to the place with the fewest such clashes.
// 16-byte scalars (X0 = 0): when level BL is formed, only the first NB(R-BL+1)
// blocks of a stored node are still read, so the last two nodes of that level lie
// in the granule arrays of nodes 0 and 1, behind those blocks, with the host
// node's array stride (these two of the eight, for no lane group meets on a bank
// then).  What node 0 has left behind that holds the pivots of levels 2 on.
// Together that is 22624 -> 20448 B a wave (double-double 22880 -> 20432) and
// an eighth wave per CU, two on each SIMD, with the split depths that suit 2048
// waves: complex n = 27 1331 -> 1185 us a call, n = 30 9.5 -> 8.57 ms,
// double-double n = 23 265 -> 243 us, n = 30 22.6 -> 20.9 ms.
template <int R, int BL, int ESZ, int L, int X0 = 0>
struct NodePlacement {
    static constexpr int NN = 1 << BL;
    static constexpr int LIVE = NB(R - BL + 1);  // blocks the parents of level BL have
    static constexpr bool TUCK = X0 == 0;
    static_assert(!TUCK || (BL >= 3 && LIVE + NB(R - BL) <= NB(R - 1)), "room behind the live blocks of nodes 0 and 1");
    int off[NN + 1];
    int nb[NN];  // blocks per granule array
    // the level-BL view whose stored node is t: the include node i of
    // level j is followed by excludes only
    static constexpr int reader(int t)
    {
        if (t == 0)
            return 0;
        int lev = 0;
        while ((1 << lev) <= t)
            ++lev;
        const int idx = t - (1 << (lev - 1));
        return ((idx << 1) | 1) << (BL - lev);
    }
    static constexpr int level(int t)
    {
        int lev = 0;
        while ((1 << lev) <= t)
            ++lev;
        return lev;
    }
    constexpr NodePlacement() : off{}, nb{}
    {
        constexpr int gpb = 4 / EPG(ESZ);          // granule arrays per node
        constexpr int acc = ESZ == 8 ? 8 : 16;     // bytes per lane per access
        // nodes per lane group and slot modulus: 32 banks, then 64 banks
        constexpr int grp[2] = {(128 / acc) >> L, (256 / acc) >> L};
        constexpr int mods[2] = {8, 16};
        int slot[NN] = {};
        int pos = 0;
        for (int t = 0; t < NN; ++t) {
            nb[t] = t == 0 ? NB(R + X0) : NB(R - level(t));
            if (TUCK && t >= NN - 2) {
                const int host = NN - 1 - t;
                nb[t] = nb[host];
                off[t] = off[host] + 16 * LIVE;
                continue;
            }
            const int b0 = (pos + 15) & ~15;
            int best = b0, bestc = 1 << 30;
            for (int k = 0; k < 16 && bestc > 0; ++k) {
                const int st = (b0 >> 4) + k;
                int c = 0;
                for (int u = 0; u < t; ++u) {
                    for (int mdl = 0; mdl < 2; ++mdl) {
                        const int G = grp[mdl] > 1 ? grp[mdl] : 1;
                        if (reader(u) / G != reader(t) / G)
                            continue;
                        for (int g = 0; g < gpb; ++g)
                            if ((st + g * nb[t]) % mods[mdl] == (slot[u] + g * nb[u]) % mods[mdl])
                                ++c;
                    }
                }
                if (c < bestc) {
                    bestc = c;
                    best = b0 + 16 * k;
                }
            }
            off[t] = best;
            slot[t] = best >> 4;
            pos = best + ESZ * (t == 0 ? NSZ(R + X0) : NSZ(R - level(t)));
        }
        off[NN] = pos;
    }
};

// 2x2 pivot of the highest mode m of a node, and the update of one output
// block (a, b), a >= b, m > a:
//   H'[x][y] = H[x][y] - conj(r1[x]) r1[y] / alpha - conj(r2'[x]) r2'[y] / gamma1
// with r1 = row 2m, r2' = row 2m+1 - r1 beta/alpha (the LDL form of the 2x2
// pivot); rows 2a, 2a+1 read r1, r2 from block (m, a), columns from (m, b).
//
// A whole block moves as 16-byte granules (node bases and granule arrays
// are 16-byte aligned), one 128-bit access each: lanes on neighbouring
// blocks then touch neighbouring 16-byte words, which LDS serves without
// bank conflicts (two 64-bit halves of a 16-byte stride would conflict)
template <class S>
struct __align__(16) Gran {
    S e[EPG((int)sizeof(S))];
};
template <class S>
__device__ __forceinline__ void get_block(const S *node, int nb, int bi, S *v)
{
    constexpr int G = EPG((int)sizeof(S));
#pragma unroll
    for (int g = 0; g < 4 / G; ++g) {
        const Gran<S> q = *reinterpret_cast<const Gran<S> *>(node + gpos((int)sizeof(S), nb, bi, g * G));
#pragma unroll
        for (int j = 0; j < G; ++j)
            v[g * G + j] = q.e[j];
    }
}
template <class S>
__device__ __forceinline__ void put_block(S *node, int nb, int bi, const S *o)
{
    constexpr int G = EPG((int)sizeof(S));
#pragma unroll
    for (int g = 0; g < 4 / G; ++g) {
        Gran<S> q;
#pragma unroll
        for (int j = 0; j < G; ++j)
            q.e[j] = o[g * G + j];
        *reinterpret_cast<Gran<S> *>(node + gpos((int)sizeof(S), nb, bi, g * G)) = q;
    }
}

// the same accesses through global-address-space pointers (tier A and the
// root path read and write the wave's stack and the matrix in global memory;
// a generic pointer would make them flat accesses)
typedef double dv2 __attribute__((ext_vector_type(2)));
template <class S>
__device__ __forceinline__ void get_block_g(const S *node, int nb, int bi, S *v)
{
    typedef const __attribute__((address_space(1))) dv2 GG;
    constexpr int G = EPG((int)sizeof(S));
#pragma unroll
    for (int g = 0; g < 4 / G; ++g) {
        const dv2 raw = *(GG *)(node + gpos((int)sizeof(S), nb, bi, g * G));
        Gran<S> q;
        __builtin_memcpy(&q, &raw, 16);
#pragma unroll
        for (int j = 0; j < G; ++j)
            v[g * G + j] = q.e[j];
    }
}
template <class S>
__device__ __forceinline__ void put_block_g(S *node, int nb, int bi, const S *o)
{
    typedef __attribute__((address_space(1))) dv2 GG;
    constexpr int G = EPG((int)sizeof(S));
#pragma unroll
    for (int g = 0; g < 4 / G; ++g) {
        Gran<S> q;
#pragma unroll
        for (int j = 0; j < G; ++j)
            q.e[j] = o[g * G + j];
        dv2 raw;
        __builtin_memcpy(&raw, &q, 16);
        *(GG *)(node + gpos((int)sizeof(S), nb, bi, g * G)) = raw;
    }
}
__device__ __forceinline__ double ld_g(const double *p) { return *(const __attribute__((address_space(1))) double *)p; }
template <class S>
__device__ __forceinline__ S ld_g(const S *p)
{
    const dv2 raw = *(const __attribute__((address_space(1))) dv2 *)p;
    S v;
    __builtin_memcpy(&v, &raw, 16);
    return v;
}
template <class S>
__device__ __forceinline__ Piv<S> node_pivot_g(const S *node, int nb, int m)
{
    const int bi = bidx(m, m);
    return pivot(re(ld_g(&blk(node, nb, bi, 0))), ld_g(&blk(node, nb, bi, 2)), re(ld_g(&blk(node, nb, bi, 3))));
}

template <class S>
__device__ __forceinline__ Piv<S> node_pivot(const S *node, int nb, int m)
{
    const int bi = bidx(m, m);
    return pivot(re(blk(node, nb, bi, 0)), blk(node, nb, bi, 2), re(blk(node, nb, bi, 3)));
}

// the update of block (a, b) from its row blocks A = (m, a), Bk = (m, b)
template <class S>
__device__ __forceinline__ void elim_math(const S *A, const S *Bk, const S *H, bool diag, const Piv<S> &pv, S *o)
{
    const S ra0 = A[0], ra1 = A[1];
    const S qa0 = sub_mul(A[2], ra0, pv.ba), qa1 = sub_mul(A[3], ra1, pv.ba);
    const S rb0 = Bk[0], rb1 = Bk[1];
    const S qb0 = sub_mul(Bk[2], rb0, pv.ba), qb1 = sub_mul(Bk[3], rb1, pv.ba);
    const S ua0 = scale(ra0, pv.inv_a), ua1 = scale(ra1, pv.inv_a);
    const S va0 = scale(qa0, pv.inv_g), va1 = scale(qa1, pv.inv_g);
    o[0] = upd(H[0], ua0, rb0, va0, qb0);
    o[1] = upd(H[1], ua0, rb1, va0, qb1);
    o[2] = upd(H[2], ua1, rb0, va1, qb0);
    o[3] = upd(H[3], ua1, rb1, va1, qb1);
    // diagonal block: real diagonal, conjugate upper entry.  Nothing reads
    // the upper entry of a diagonal block (pivots read entries 0, 2, 3, the
    // lanes read the lower triangle), so real scalars leave it as computed.
    if constexpr (std::is_same<S, c64>::value) {
        if (diag) {
            o[0] = fix_diag(o[0]);
            o[3] = fix_diag(o[3]);
            o[1] = conj_of(o[2]);
        }
    }
}

template <class S, bool GLOBAL = false>
__device__ __forceinline__ void elim_block(const S *node, int nb, int m, int a, int b, int ih, const Piv<S> &pv,
                                           S *o)
{
    S A[4], Bk[4], H[4];
    if constexpr (GLOBAL) {
        get_block_g(node, nb, bidx(m, a), A);
        get_block_g(node, nb, bidx(m, b), Bk);
        get_block_g(node, nb, ih, H);
    } else {
        get_block(node, nb, bidx(m, a), A);
        get_block(node, nb, bidx(m, b), Bk);
        get_block(node, nb, ih, H);
    }
    elim_math(A, Bk, H, a == b, pv, o);
}


// ---------------------------------------------------------------------------
// one include step on global memory (tier A and the root path): src is a view
// of s modes of a node with snb blocks per granule array, dst receives the
// Schur complement of s-1 modes as a node with dnb blocks per granule array.
// Every lane forms the pivot itself; lane l updates blocks l, l+64, ...  dst
// (global, may be null) receives the whole child; lds (may be null) receives
// its first nlds blocks (the tier-A leaf) as a node of nlds blocks.
//
// dst may be src itself (the root path eliminates in place, with dnb = snb):
// block (a, b) of the child is read and rewritten by the same lane, and the
// pivot rows (blocks of mode s-1) are never written, so no lane reads a
// block another lane has already replaced.  Block indices do not depend on
// the node's size, so the same lane owns the same block at every step.
template <class S>
__device__ __forceinline__ void elim_global_body(const S *src, int snb, S *dst, int dnb, S *lds, int nlds, int s,
                                                 int lane, RT<S> &pdet, int &bad)
{
    __asm__ volatile("" : "+v"(lane));  // as in copy_node
    const int m = s - 1;
    const Piv<S> pv = node_pivot_g(src, snb, m);
    pdet = pv.pdet;
    if (!is_pos(pv.pdet) || !is_pos(pv.inv_a))
        bad = 1;
    const int nbo = dst ? NB(m) : nlds;
    for (int bi = lane; bi < nbo; bi += 64) {
        int a, b;
        block_ab(bi, a, b);
        S o[4];
        elim_block<S, true>(src, snb, m, a, b, bidx(a, b), pv, o);
        if (dst)
            put_block_g(dst, dnb, bi, o);
        if (lds && bi < nlds)
            put_block(lds, nlds, bi, o);
    }
    __syncthreads();
}

// the same with src and dst distinct (tier A).  A step of at most 128
// blocks (every step that makes a tier-A leaf, and the deeper stack levels)
// issues the loads of the pivot and of both of each lane's blocks before any
// arithmetic, so it waits for L2 once instead of once for the pivot and once
// per pass; larger steps take the loop above.
template <class S>
__device__ void elim_global(const S *__restrict__ src, int snb, S *__restrict__ dst, int dnb, S *lds, int nlds, int s,
                            int lane, RT<S> &pdet, int &bad)
{
    const int m = s - 1;
    const int nbo = dst ? NB(m) : nlds;
    if (nbo > 128) {
        elim_global_body(src, snb, dst, dnb, lds, nlds, s, lane, pdet, bad);
        return;
    }
    // real path: the second block's coordinates are found again at every step
    // (a step that makes a leaf has two lanes with one), which frees the
    // registers that its accumulators take
    int lane1 = lane;
    if constexpr (std::is_same<S, double>::value)
        __asm__ volatile("" : "+v"(lane1));
    const int bi0 = lane, bi1 = lane1 + 64;
    const bool h0 = bi0 < nbo, h1 = bi1 < nbo;
    int a0 = 0, b0 = 0, a1 = 0, b1 = 0;
    block_ab(bi0, a0, b0);
    block_ab(bi1, a1, b1);
    S A0[4], B0[4], H0[4], A1[4], B1[4], H1[4];
    const int dbi = bidx(m, m);
    const RT<S> al = re(ld_g(&blk(src, snb, dbi, 0)));
    const S be = ld_g(&blk(src, snb, dbi, 2));
    const RT<S> ga = re(ld_g(&blk(src, snb, dbi, 3)));
    if (h0) {
        get_block_g(src, snb, bidx(m, a0), A0);
        get_block_g(src, snb, bidx(m, b0), B0);
        get_block_g(src, snb, bidx(a0, b0), H0);
    }
    if (h1) {
        get_block_g(src, snb, bidx(m, a1), A1);
        get_block_g(src, snb, bidx(m, b1), B1);
        get_block_g(src, snb, bidx(a1, b1), H1);
    }
    const Piv<S> pv = pivot(al, be, ga);
    pdet = pv.pdet;
    if (!is_pos(pv.pdet) || !is_pos(pv.inv_a))
        bad = 1;
    if (h0) {
        S o[4];
        elim_math(A0, B0, H0, a0 == b0, pv, o);
        if (dst)
            put_block_g(dst, dnb, bi0, o);
        if (lds && bi0 < nlds)
            put_block(lds, nlds, bi0, o);
    }
    if (h1) {
        S o[4];
        elim_math(A1, B1, H1, a1 == b1, pv, o);
        if (dst)
            put_block_g(dst, dnb, bi1, o);
        if (lds && bi1 < nlds)
            put_block(lds, nlds, bi1, o);
    }
    __syncthreads();
}

// in place (dst == src, or src the read-only matrix): the root path
template <class S>
__device__ void elim_inplace(const S *src, int snb, S *dst, int dnb, int s, int lane, RT<S> &pdet, int &bad)
{
    elim_global_body(src, snb, dst, dnb, (S *)nullptr, 0, s, lane, pdet, bad);
}

// one include step in place in LDS on a node of s modes with nb blocks per
// granule array (each lane rewrites only blocks it reads, and never a pivot
// row, as in elim_inplace)
template <class S>
__device__ __forceinline__ void elim_lds(S *node, int nb, int s, int lane, RT<S> &pdet, int &bad)
{
    const int m = s - 1;
    const Piv<S> pv = node_pivot(node, nb, m);
    pdet = pv.pdet;
    if (!is_pos(pv.pdet) || !is_pos(pv.inv_a))
        bad = 1;
    for (int bi = lane; bi < NB(m); bi += 64) {
        int a, b;
        block_ab(bi, a, b);
        S o[4];
        elim_block<S, false>(node, nb, m, a, b, bidx(a, b), pv, o);
        put_block(node, nb, bi, o);
    }
    __syncthreads();
}

// 16-byte granule gi of a node, from LDS or (GLOBAL) global memory
template <bool GLOBAL, class S>
__device__ __forceinline__ dv2 ld_gran(const S *node, int gi)
{
    const S *p = node + EPG((int)sizeof(S)) * gi;
    if constexpr (GLOBAL)
        return *(const __attribute__((address_space(1))) dv2 *)p;
    return *reinterpret_cast<const dv2 *>(p);
}
template <bool GLOBAL, class S>
__device__ __forceinline__ void st_gran(S *node, int gi, dv2 v)
{
    S *p = node + EPG((int)sizeof(S)) * gi;
    if constexpr (GLOBAL)
        *(__attribute__((address_space(1))) dv2 *)p = v;
    else
        *reinterpret_cast<dv2 *>(p) = v;
}

// the first s modes of a node with snb blocks per granule array, copied into
// a node with dnb (global source or destination as flagged), in 16-byte
// granules.  What bounds it is the latency of its loads (a root starts with
// one such copy of its matrix): each lane issues 8 loads (4 on the 16-byte
// paths, whose registers allow no more) before it stores any.
template <class S, bool SRC_G, bool DST_G>
__device__ __forceinline__ void copy_node(const S *src, int snb, S *dst, int dnb, int s, int lane)
{
    constexpr int GPB = 4 / EPG((int)sizeof(S));  // granule arrays
    constexpr int U = GPB == 2 ? 4 : 1;
    // the empty asm keeps what a lane derives from its index alone, the same in
    // every call, from being held in registers through the whole kernel
    __asm__ volatile("" : "+v"(lane));
    const int nb = NB(s);
    for (int b0 = lane; b0 < nb; b0 += 64 * U) {
        dv2 v[U][GPB];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (b0 + 64 * u < nb)
#pragma unroll
                for (int g = 0; g < GPB; ++g)
                    v[u][g] = ld_gran<SRC_G>(src, g * snb + b0 + 64 * u);
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (b0 + 64 * u < nb)
#pragma unroll
                for (int g = 0; g < GPB; ++g)
                    st_gran<DST_G>(dst, g * dnb + b0 + 64 * u, v[u][g]);
    }
}

// the first SM modes of a node in LDS, moved to the front of its buffer with
// the stride NB(SM) (the source's granule arrays start at node and are nb
// blocks apart, nb >= NB(SM)): the two overlap, so every granule is read
// before any is written
template <class S, int SM>
__device__ __forceinline__ void restride_node(S *node, int nb, int s, int lane)
{
    constexpr int GPB = 4 / EPG((int)sizeof(S)), IT = (NB(SM) + 63) / 64;
    __asm__ volatile("" : "+v"(lane));  // as in copy_node
    const int n = NB(s);
    dv2 v[IT][GPB];
#pragma unroll
    for (int i = 0; i < IT; ++i)
        if (lane + 64 * i < n)
#pragma unroll
            for (int g = 0; g < GPB; ++g)
                v[i][g] = ld_gran<false>(node, g * nb + lane + 64 * i);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < IT; ++i)
        if (lane + 64 * i < n)
#pragma unroll
            for (int g = 0; g < GPB; ++g)
                st_gran<false>(node, g * NB(SM) + lane + 64 * i, v[i][g]);
}

// ---------------------------------------------------------------------------
// The tier-B tables, made at compile time and copied to LDS once per wave.
// View t: for the node of level jl with id i (bit jl-1-m of i = decision on the
// m-th mode below the tier-A leaf, 1 = include; t = (2^jl - 1) + i) the LDS
// offset of the stored node it is a view of, that node's blocks per granule
// array, and the slot of its determinant (0xff: the tier-A leaf).  The include
// node (lev, idx) keeps its determinant at (2^(lev-1) - 1) + idx.  Per include
// node i of level J (record (2^(J-1) - 1) + i, J = 1..B-1) its parent's stored
// offset and blocks per array and its own stored offset, packed in 64 bits (its
// own blocks per array too where they differ within the level, NodePlacement);
// per block bi of a child (a, b) and its block index bidx(a, b) packed (real
// path: of the leaf's own include step too, elim_leaf).
template <int R, int B, int ESZ, int L, int X0>
struct TierBTables {
    static constexpr int NV = (1 << B) - 1, NR = (1 << (B - 1)) - 1, NK = NB(R - 1 + X0);
    unsigned long long nodeRec[NR];
    uint32_t blkRec[NK];
    uint16_t srcOff[NV];
    uint8_t srcNB[NV], srcDet[NV];
    constexpr TierBTables() : nodeRec{}, blkRec{}, srcOff{}, srcNB{}, srcDet{}
    {
        constexpr NodePlacement<R, B - 1, ESZ, L, X0> place{};
        for (int t = 0; t < NV; ++t) {
            int jl = 0;
            while ((2 << jl) <= t + 1)
                ++jl;
            const int i = t + 1 - (1 << jl);
            int off = 0, nb = NB(R + X0), det = 0xff;
            if (i != 0) {
                int tz = 0;
                while (((i >> tz) & 1) == 0)
                    ++tz;
                const int lev = jl - tz, idx = (i >> tz) >> 1;
                off = place.off[(1 << (lev - 1)) + idx] / ESZ;
                nb = place.nb[(1 << (lev - 1)) + idx];
                det = (1 << (lev - 1)) - 1 + idx;
            }
            srcOff[t] = (uint16_t)off;
            srcNB[t] = (uint8_t)nb;
            srcDet[t] = (uint8_t)det;
        }
        for (int J = 1; J < B; ++J)
            for (int i = 0; i < 1 << (J - 1); ++i) {
                const int t = (1 << (J - 1)) - 1 + i, c = (1 << J) - 1 + 2 * i + 1;
                nodeRec[t] = (unsigned long long)(srcOff[t] * ESZ) | ((unsigned long long)(16 * srcNB[t]) << 16) |
                             ((unsigned long long)(srcOff[c] * ESZ) << 32) |
                             (X0 == 0 && J == B - 1 ? (unsigned long long)(16 * srcNB[c]) << 48 : 0ull);
            }
        for (int a = 0, bi = 0; a < R - 1 + X0; ++a)
            for (int b = 0; b <= a; ++b, ++bi)
                blkRec[bi] = (uint32_t)(16 * bidx(a, b) | (16 * a) << 16 | (16 * b) << 24);
    }
};
template <class S, int R, int B, int L>
__device__ __forceinline__ void build_tables(uint16_t *srcOff, uint8_t *srcNB, uint8_t *srcDet,
                                             unsigned long long *nodeRec, uint32_t *blkRec, int lane)
{
    constexpr int X0 = std::is_same<S, double>::value ? 1 : 0;
    using Tab = TierBTables<R, B, (int)sizeof(S), L, X0>;
    static constexpr Tab tab{};
    static_assert(Tab::NV <= 64, "one entry per lane");
    if (lane < Tab::NV) {
        srcOff[lane] = tab.srcOff[lane];
        srcNB[lane] = tab.srcNB[lane];
        srcDet[lane] = tab.srcDet[lane];
    }
    if (lane < Tab::NR)
        nodeRec[lane] = tab.nodeRec[lane];
    for (int t = lane; t < Tab::NK; t += 64)
        blkRec[t] = tab.blkRec[t];
}

// LDS tables of tier B (see build_tables) and its per-node pivot scalars
template <class S>
struct TierB {
    S *buf;                 // stored nodes (NodePlacement)
    const uint16_t *srcOff; // per view: offset of its stored node
    const uint8_t *srcNB;   // per view: blocks per granule array of that node
    const uint8_t *srcDet;  // per view: determinant slot (0xff: tier-A leaf)
    const unsigned long long *nodeRec;  // per include node, bytes: parent | its granule array stride << 16 | own << 32, 48
    const uint32_t *blkRec;             // block index, bytes: 16 bidx(a, b) | 16 a << 16 | 16 b << 24
    RT<S> *ndet;            // per include node: running determinant (det_at)
    RT<S> *nInvS;           // per include node of a level: 1/alpha, 1/gamma1 (real path; pivot_slots)
    S *nBaS;                // per include node of a level: beta/alpha (the same)
};

// Where the pivots of a level are kept between its two phases: arrays of their
// own on the real path; on the 16-byte paths behind the blocks of node 0 that
// level 1 was the last to read, 1/alpha, 1/gamma1 and beta/alpha in one granule
// array each, and level 1's own in the last node of level BL but the two tucked
// away, which is not there yet.  The double-double factor's determinants of level
// BL lie in the fourth array.
template <class S, int R, int BL, int L>
struct TuckedPivots {
    using Place = NodePlacement<R, BL, (int)sizeof(S), L, 0>;
    static constexpr Place place{};
    static constexpr int AT = 16 * (Place::LIVE + NB(R - BL)), ROOM = 16 * NB(R) - AT;
    // the pass that forms level 2 reads pivots there and node 0's first NB(R - 1) blocks
    static_assert(Place::LIVE + NB(R - BL) >= NB(R - 1), "pivots behind the blocks that are still read");
    static_assert((int)sizeof(S) << (BL - 1) <= ROOM && (int)sizeof(RT<S>) << (BL - 1) <= ROOM, "one entry per include node");
    // array a of level J, from the start of the buffer
    static constexpr int at(int J, int a)
    {
        return J == 1 ? place.off[Place::NN] - 64 * NB(R - BL) + 16 * a : place.off[0] + 16 * NB(R) * a + AT;
    }
};
// 1/alpha, 1/gamma1 and beta/alpha of include node i of level J
template <class S, int R, int J, int BL, int L>
__device__ __forceinline__ void pivot_slots(const TierB<S> &tb, int i, RT<S> *&inv_a, RT<S> *&inv_g, S *&ba)
{
    if constexpr (std::is_same<S, double>::value) {
        inv_a = tb.nInvS + 2 * i;
        inv_g = tb.nInvS + 2 * i + 1;
        ba = tb.nBaS + i;
    } else {
        using P = TuckedPivots<S, R, BL, L>;
        char *const lb = reinterpret_cast<char *>(tb.buf);
        inv_a = reinterpret_cast<RT<S> *>(lb + P::at(J, 0)) + i;
        inv_g = reinterpret_cast<RT<S> *>(lb + P::at(J, 1)) + i;
        ba = reinterpret_cast<S *>(lb + P::at(J, 2)) + i;
    }
}
// the running determinant of include node d (levels in order)
template <class S, int R, int BL, int L>
__device__ __forceinline__ RT<S> *det_at(const TierB<S> &tb, int d)
{
    if constexpr (std::is_same<S, ddr>::value) {
        constexpr int LAST = (1 << (BL - 1)) - 1;  // the first one of level BL
        if (d >= LAST)
            return reinterpret_cast<RT<S> *>(reinterpret_cast<char *>(tb.buf) + TuckedPivots<S, R, BL, L>::at(2, 3)) + (d - LAST);
    }
    return tb.ndet + d;
}

// tier B, level J: every include node of level J from its parent of level J-1
template <class S, int R, int J, int BL, int L>
__device__ __forceinline__ void tierB_level(const TierB<S> &tb, RT<S> leafDet, int lane, int &bad)
{
    constexpr int m = R - J;          // pivot mode of the parent (it has m+1 modes)
    constexpr int NN = 1 << (J - 1);  // include nodes at level J
    constexpr int NBO = NB(m);        // blocks of a child
    if (lane < NN) {
        const S *par = tb.buf + tb.srcOff[NN - 1 + lane];
        const int di = tb.srcDet[NN - 1 + lane];
        const RT<S> pdp = di == 0xff ? leafDet : *det_at<S, R, BL, L>(tb, di);
        const Piv<S> pq = node_pivot(par, (int)tb.srcNB[NN - 1 + lane], m);
        RT<S> *pa, *pg;
        S *pb;
        pivot_slots<S, R, J, BL, L>(tb, lane, pa, pg, pb);
        *pa = pq.inv_a;
        *pg = pq.inv_g;
        *pb = pq.ba;
        *det_at<S, R, BL, L>(tb, NN - 1 + lane) = rmul(pdp, pq.pdet);
        if (!is_pos(pq.pdet) || !is_pos(pq.inv_a))
            bad = 1;
    }
    __syncthreads();
    // granule g of the block at byte offset o of a node at byte offset p
    // with arrays st bytes apart: buf + p + g st + o
    char *const lb = reinterpret_cast<char *>(tb.buf);
    constexpr int GPB = 4 / EPG((int)sizeof(S));  // granules per block
    // 16-byte scalars: each node's blocks start on a 16-lane boundary (NS
    // lanes per node), so the 16 lanes one LDS cycle serves of a 128-bit
    // access never span two nodes, whose neighbouring 16-byte words would
    // meet in the same banks.  This costs no pass at the levels of the
    // complex and double-double kernels and halves their LDS bank-conflict
    // cycles; the 8-byte path keeps packed nodes (its passes hold two
    // granules per block, and the extra index registers cost it waves).
    constexpr bool AL = !std::is_same<S, double>::value;
    constexpr bool TUCK = AL && J == BL;  // nodes of several array strides
    constexpr int NS = AL ? (NBO + 15) / 16 * 16 : NBO;  // lanes per node in a pass
    auto pass = [&](int it) {
        const int i = (int)((unsigned)it / NS), bi = it - i * NS;
        if (AL && bi >= NBO)
            return;
        const unsigned long long rec = tb.nodeRec[NN - 1 + i];
        const uint32_t br = tb.blkRec[bi];
        const int par = (int)(rec & 0xffffu), st = (int)((rec >> 16) & 0xffffu), cof = TUCK ? (int)((rec >> 32) & 0xffffu) : (int)(rec >> 32);
        const int cst = TUCK ? (int)(rec >> 48) : 16 * NBO;  // the child's granule arrays
        const int a16 = (int)((br >> 16) & 0xffu), b16 = (int)(br >> 24), h16 = (int)(br & 0xffffu);
        Piv<S> pq;
        RT<S> *qpa, *qpg;
        S *qpb;
        pivot_slots<S, R, J, BL, L>(tb, i, qpa, qpg, qpb);
        pq.inv_a = *qpa;
        pq.inv_g = *qpg;
        pq.ba = *qpb;
        S A[4], Bk[4], H[4], o[4];
        const char *pa = lb + par + a16 + 16 * NB(m), *pb = lb + par + b16 + 16 * NB(m), *ph = lb + par + h16;
#pragma unroll
        for (int g = 0; g < GPB; ++g) {
            const Gran<S> qa = *reinterpret_cast<const Gran<S> *>(pa + g * st);
            const Gran<S> qb = *reinterpret_cast<const Gran<S> *>(pb + g * st);
            const Gran<S> qh = *reinterpret_cast<const Gran<S> *>(ph + g * st);
#pragma unroll
            for (int j = 0; j < EPG((int)sizeof(S)); ++j) {
                A[g * EPG((int)sizeof(S)) + j] = qa.e[j];
                Bk[g * EPG((int)sizeof(S)) + j] = qb.e[j];
                H[g * EPG((int)sizeof(S)) + j] = qh.e[j];
            }
        }
        elim_math(A, Bk, H, a16 == b16, pq, o);
        // the include child i of level J is view 2i+1 of that level
        char *pc = lb + cof + 16 * bi;
#pragma unroll
        for (int g = 0; g < GPB; ++g) {
            Gran<S> q;
#pragma unroll
            for (int j = 0; j < EPG((int)sizeof(S)); ++j)
                q.e[j] = o[g * EPG((int)sizeof(S)) + j];
            *reinterpret_cast<Gran<S> *>(pc + g * cst) = q;
        }
    };
    constexpr int TOT = NN * NS, FULL = TOT / 64;
    // real path: an empty asm hides that the lane index is the same in every
    // leaf, so the node and block indices of the passes of levels 3 and 4 are
    // recomputed per leaf instead of being held in registers across the whole
    // leaf loop (levels 1 and 2 fit: 254 registers; with the others the
    // kernel passes 256 and half the waves go).  The 16-byte paths have
    // registers to spare.
    int ln = lane;
    if constexpr (std::is_same<S, double>::value && J > 2)
        __asm__ volatile("" : "+v"(ln));
    __builtin_assume((unsigned)ln < 64u);  // node and block by 24-bit products
#pragma unroll 2
    for (int it0 = 0; it0 < 64 * FULL; it0 += 64)
        pass(it0 + ln);
    if constexpr (TOT % 64 != 0) {
        if (64 * FULL + ln < TOT)
            pass(64 * FULL + ln);
    }
    __syncthreads();
}

// real path: the include step in place on LDS node 0 (R + 1 modes) that makes
// every second leaf, block coordinates from the table
template <class S, int R>
__device__ __forceinline__ void elim_leaf(const TierB<S> &tb, int lane, RT<S> &pdet, int &bad)
{
    constexpr int G = EPG((int)sizeof(S)), GPB = 4 / G, ST = 16 * NB(R + 1);
    char *const lb = reinterpret_cast<char *>(tb.buf);
    const Piv<S> pv = node_pivot(tb.buf, NB(R + 1), R);
    pdet = pv.pdet;
    if (!is_pos(pv.pdet) || !is_pos(pv.inv_a))
        bad = 1;
    for (int bi = lane; bi < NB(R); bi += 64) {
        const uint32_t br = tb.blkRec[bi];
        const int a16 = (int)((br >> 16) & 0xffu), b16 = (int)(br >> 24);
        S A[4], Bk[4], H[4], o[4];
#pragma unroll
        for (int g = 0; g < GPB; ++g) {
            const Gran<S> qa = *reinterpret_cast<const Gran<S> *>(lb + a16 + 16 * NB(R) + g * ST);
            const Gran<S> qb = *reinterpret_cast<const Gran<S> *>(lb + b16 + 16 * NB(R) + g * ST);
            const Gran<S> qh = *reinterpret_cast<const Gran<S> *>(lb + 16 * bi + g * ST);
#pragma unroll
            for (int j = 0; j < G; ++j) {
                A[g * G + j] = qa.e[j];
                Bk[g * G + j] = qb.e[j];
                H[g * G + j] = qh.e[j];
            }
        }
        elim_math(A, Bk, H, a16 == b16, pv, o);
        put_block(tb.buf, NB(R + 1), bi, o);
    }
    __syncthreads();
}

template <class S, int R, int J, int BL, int L>
__device__ __forceinline__ void tierB(const TierB<S> &tb, RT<S> leafDet, int lane, int &bad)
{
    if constexpr (J <= BL) {
        tierB_level<S, R, J, BL, L>(tb, leafDet, lane, bad);
        tierB<S, R, J + 1, BL, L>(tb, leafDet, lane, bad);
    }
}

// ---------------------------------------------------------------------------
// register-resident include step (packed lower triangle): h has M modes, hn
// receives M-1 modes
template <class S, int M>
__device__ __forceinline__ void elim_regs(const S *h, const Piv<S> &pq, S *hn)
{
    constexpr int p = 2 * M - 2;
    S u1[p], r1[p], u2[p], r2[p];
#pragma unroll
    for (int y = 0; y < p; ++y) {
        r1[y] = h[pidx(p, y)];
        r2[y] = sub_mul(h[pidx(p + 1, y)], r1[y], pq.ba);
        u1[y] = scale(r1[y], pq.inv_a);
        u2[y] = scale(r2[y], pq.inv_g);
    }
#pragma unroll
    for (int x = 0; x < p; ++x)
#pragma unroll
        for (int y = 0; y <= x; ++y) {
            if (x == y)
                hn[pidx(x, y)] = upd_diag(h[pidx(x, y)], u1[x], r1[y], u2[x], r2[y]);
            else
                hn[pidx(x, y)] = upd(h[pidx(x, y)], u1[x], r1[y], u2[x], r2[y]);
        }
}

// all 2^M subsets below a register-resident node of M modes.  SG is the sign
// (-1)^(#excluded) of its subsets relative to the lane's frame (see the
// accumulators); det is the running determinant.
template <class S, int M, int SG, class Acc, int TB = 0>
__device__ __forceinline__ void tail(const S *h, RT<S> det, Acc &acc, int &bad)
{
    if constexpr (M == 0) {
        acc.template add<SG, TB>(rsqrt_nr(det));
    } else if constexpr (M == 1) {
        // exclude (sign -SG) and include (sign SG) of the last mode
        const RT<S> a = re(h[0]);
        const S b = h[1];
        const RT<S> g = re(h[2]);
        const RT<S> pd = det_last(a, b, g);  // det of the last 2x2 block
        acc.template add_pair<SG, TB>(rsqrt_nr(det), rsqrt_nr(rmul(det, pd)));
    } else {
        tail<S, M - 1, -SG, Acc, TB>(h, det, acc, bad);  // exclude the next mode
        constexpr int p = 2 * M - 2;
        const RT<S> a = re(h[pidx(p, p)]);
        const S b = h[pidx(p + 1, p)];
        const RT<S> g = re(h[pidx(p + 1, p + 1)]);
        const Piv<S> pq = pivot(a, b, g);
        S hn[E(M - 1)];
        elim_regs<S, M>(h, pq, hn);
        tail<S, M - 1, SG, Acc, TB | (1 << (M - 1))>(hn, rmul(det, pq.pdet), acc, bad);
    }
}

// The include chain of a register-resident node of M modes: its 2x2 pivots
// in turn, each tested (alpha > 0, alpha gamma1 > 0), down to the last mode.
// Run on the lane that holds the all-include subset, this completes the test
// of every pivot of the factorisation of I - O itself: positive definiteness
// of I - O is equivalent to all of them passing (the block form of
// Sylvester's criterion), and it implies it for every other subset.
template <class S, int M>
__device__ __forceinline__ void include_chain_test(const S *h, int &bad)
{
    if constexpr (M == 1) {
        const RT<S> a = re(h[0]);
        if (!is_pos(a) || !is_pos(det_last(a, h[1], re(h[2]))))
            bad = 1;
    } else if constexpr (M > 1) {
        constexpr int p = 2 * M - 2;
        const RT<S> a = re(h[pidx(p, p)]);
        const Piv<S> pq = pivot(a, h[pidx(p + 1, p)], re(h[pidx(p + 1, p + 1)]));
        if (!is_pos(a) || !is_pos(pq.pdet))
            bad = 1;
        S hn[E(M - 1)];
        elim_regs<S, M>(h, pq, hn);
        include_chain_test<S, M - 1>(hn, bad);
    }
}

// element (x, y), y <= x, of a node with nb blocks per granule array
template <class S>
__device__ __forceinline__ S node_el(const S *node, int nb, int x, int y)
{
    return blk(node, nb, bidx(x >> 1, y >> 1), ((x & 1) << 1) + (y & 1));
}

// pivot of one lane-level decision: an include lane takes the 2x2 pivot, an
// exclude lane a zero update (inverses and beta/alpha zero, determinant 1),
// which leaves the prefix exactly as it is, so that both kinds of lanes run
// the same instructions.
template <class S>
__device__ __forceinline__ Piv<S> lane_pivot(RT<S> a, S b, RT<S> g, bool inc, int &bad)
{
    Piv<S> pq = pivot(a, b, g);
    if (inc && (!is_pos(a) || !is_pos(pq.pdet)))
        bad = 1;
    if (!inc) {
        pq.inv_a = rconst<RT<S>>(0.0);
        pq.inv_g = rconst<RT<S>>(0.0);
        pq.ba = zero_of(b);
        pq.pdet = rconst<RT<S>>(1.0);
    }
    return pq;
}

// tier C: lane l finishes node l of level B.  Its ancestor of level B-L is an
// LDS node of T+L modes; the lane takes the last L decisions itself (bit
// L-1-j of l is the decision at level B-L+1+j) and then the last T modes.
// The L lane levels are fused into one pass over the LDS node: the pivot
// rows of every level are formed first, then each remaining entry is read
// once and receives the L rank-2 updates in turn, so only the pivot rows and
// the T-mode result are held in registers.
template <class S, int T, int B, int L, class Acc>
__device__ __forceinline__ void tierC_terms(const TierB<S> &tb, RT<S> leafDet, int leafInc, int N, int lane, Acc &acc,
                                            int &bad, bool full_leaf, double &sign, double &anchor)
{
    static_assert(L == 1 || L == 2, "one or two lane levels");
    constexpr int NP = (1 << (B - L)) - 1;  // table base of level B-L
    constexpr int pT = 2 * T;               // rows of the T-mode result
    constexpr int p1 = 2 * (T + L) - 2;     // pivot rows of the first lane level
    const int ip = lane >> L;
    const S *src = tb.buf + tb.srcOff[NP + ip];
    const int snb = tb.srcNB[NP + ip];
    const int di = tb.srcDet[NP + ip];
    RT<S> det = di == 0xff ? leafDet : *det_at<S, T + B, B - L, L>(tb, di);
    const bool inc1 = (lane >> (L - 1)) & 1;  // first lane level
    const bool inc0 = lane & 1;               // second (L == 2)

    // first level: pivot of mode T+L-1 and its rows, r2 in LDL form
    const Piv<S> q1 = lane_pivot(re(node_el(src, snb, p1, p1)), node_el(src, snb, p1 + 1, p1),
                                 re(node_el(src, snb, p1 + 1, p1 + 1)),
                                 inc1, bad);
    S r1[p1], r2[p1];
#pragma unroll
    for (int y = 0; y < p1; ++y) {
        r1[y] = node_el(src, snb, p1, y);
        r2[y] = sub_mul(node_el(src, snb, p1 + 1, y), r1[y], q1.ba);
    }
    det = rmul(det, q1.pdet);
    int includes = leafInc + __popc(ip) + inc1;

    // second level (L == 2): its pivot rows are rows pT, pT+1 of the first
    // child, formed here from the node and the first level's rows
    Piv<S> q2;
    S s1[pT], s2[pT];
    if constexpr (L == 2) {
        S c[2][pT + 2];
#pragma unroll
        for (int x = pT; x < pT + 2; ++x) {
            const S u1 = scale(r1[x], q1.inv_a), u2 = scale(r2[x], q1.inv_g);
#pragma unroll
            for (int y = 0; y <= x; ++y) {
                const S v = node_el(src, snb, x, y);
                c[x - pT][y] = (x == y) ? upd_diag(v, u1, r1[y], u2, r2[y]) : upd(v, u1, r1[y], u2, r2[y]);
            }
        }
        q2 = lane_pivot(re(c[0][pT]), c[1][pT], re(c[1][pT + 1]), inc0, bad);
#pragma unroll
        for (int y = 0; y < pT; ++y) {
            s1[y] = c[0][y];
            s2[y] = sub_mul(c[1][y], s1[y], q2.ba);
        }
        det = rmul(det, q2.pdet);
        includes += inc0;
    }

    // the T-mode result: every entry read once, updated level by level
    S hT[E(T)];
#pragma unroll
    for (int x = 0; x < pT; ++x) {
        const S u1 = scale(r1[x], q1.inv_a), u2 = scale(r2[x], q1.inv_g);
        S w1, w2;
        if constexpr (L == 2) {
            w1 = scale(s1[x], q2.inv_a);
            w2 = scale(s2[x], q2.inv_g);
        }
#pragma unroll
        for (int y = 0; y <= x; ++y) {
            const S v = node_el(src, snb, x, y);
            S o = (x == y) ? upd_diag(v, u1, r1[y], u2, r2[y]) : upd(v, u1, r1[y], u2, r2[y]);
            if constexpr (L == 2)
                o = (x == y) ? upd_diag(o, w1, s1[y], w2, s2[y]) : upd(o, w1, s1[y], w2, s2[y]);
            hT[pidx(x, y)] = o;
        }
    }
    const int excluded = (N - T) - includes;
    sign = (excluded & 1) ? -1.0 : 1.0;
    acc.set_frame(sign);
    if constexpr (Acc::kAnchored) {
        anchor = acc.anchor(det);
        acc.open(anchor);
    }
    if (full_leaf)  // wave-uniform: the leaf that holds the all-include subset
        include_chain_test<S, T>(hT, bad);
    tail<S, T, 1, Acc>(hT, det, acc, bad);
}

template <class S, int T, int B, int L, class Acc>
__device__ __forceinline__ void tierC(const TierB<S> &tb, RT<S> leafDet, int leafInc, int N, int lane, Acc &acc,
                                      int &bad, bool full_leaf)
{
    double sign, anchor;
    if constexpr (Acc::kAnchored) {
        if (acc.usable()) {
            tierC_terms<S, T, B, L, Acc>(tb, leafDet, leafInc, N, lane, acc, bad, full_leaf, sign, anchor);
            if (acc.close(sign, anchor))
                return;
            // once more from the LDS nodes, which are as they were (the empty
            // asm: nothing of the first run is kept for this one)
            __asm__ volatile("" : "+v"(lane));
        }
        if constexpr (Acc::kDD) {
            AccDD leaf;
            tierC_terms<S, T, B, L, AccDD>(tb, leafDet, leafInc, N, lane, leaf, bad, full_leaf, sign, anchor);
            acc.fold(sign, leaf.hi, leaf.lo, leaf.abs_sum);
        }
    } else {
        tierC_terms<S, T, B, L, Acc>(tb, leafDet, leafInc, N, lane, acc, bad, full_leaf, sign, anchor);
    }
}

// ---------------------------------------------------------------------------
// Host memory is written by system-scope stores, and the number the host waits
// for last, behind a release of that scope: the host reads the result as soon
// as it is there, without the end-of-kernel signal and the runtime's wait for
// it (3 to 5 us of a call).
template <class V>
__device__ __forceinline__ void st_host(V *p, V v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
// one lane: the verdict, and then the evaluation's number
__device__ __forceinline__ void announce(EvalResult *r, const StageInfo *gate, unsigned long long done)
{
    st_host(&r->status, gate->status);
    st_host(&r->path, gate->path);
    st_host(&r->N, gate->N);
    __hip_atomic_store(&r->done, done, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Agent-scope accesses: what another wave of the same launch reads, on
// whichever die it runs.
template <class V>
__device__ __forceinline__ void st_agent(V *p, V v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <class V>
__device__ __forceinline__ V ld_agent(const V *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <bool DD>
__device__ inline void red_step(double &h, double &l, double &ab, double &bad, int off)
{
    const double oh = __shfl_xor(h, off), ol = __shfl_xor(l, off);
    if (DD)
        dd_add2(h, l, oh, ol);
    else
        h += oh;
    ab += __shfl_xor(ab, off);
    bad = fmax(bad, __shfl_xor(bad, off));
}

// The end of a root of a lone evaluation with at most RESULT_ROOTS of them
// (its slot is written): the wave that ends last sums the slots, in
// the order of the reduction kernel (whose threads and waves beyond them add
// zeros), and announces the result if it is the last launch of its chain, instead
// of a launch for that alone: 13 Hermitian modes 29.5 us a call against 31.9.
// More roots than lanes keep the kernel of their own: they would all meet at
// this one counter (13 ns each), and one wave would add several slots a lane
// (256 roots, real n = 19: 37.0 us a call against 35.3; 128, n = 18: 33.3
// against 33.6, with 0.4 us more for those of up to 64).
template <bool DD>
__device__ __forceinline__ void finish_root(const __attribute__((address_space(4))) MainParams *prm, const double *slots, int lane)
{
    const int nroots = (int)prm->total_items;
    if (nroots > 1) {
        // the slot is out before it is counted
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_s_waitcnt(0);
        unsigned long long before = 0;
        if (lane == 0)
            before = __hip_atomic_fetch_add(prm->finished, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (bcast_first(before) + 1 < (unsigned long long)nroots)
            return;
    }
    double h = 0.0, l = 0.0, ab = 0.0, bad = 0.0;
    if (lane < nroots) {
        const double *s = slots + 4 * lane;
        const double s0 = ld_agent(s), s1 = ld_agent(s + 1);
        ab = ld_agent(s + 2);
        bad = ld_agent(s + 3);
        if (DD)
            dd_add2(h, l, s0, s1);
        else
            h = s0;
    }
#pragma unroll 1
    for (int off = 32; off >= 1; off >>= 1)
        red_step<DD>(h, l, ab, bad, off);
    if (DD)
        dd_add2(h, l, 0.0, 0.0);
    if (lane == 0) {
        st_host(&prm->result->v[0], h);
        st_host(&prm->result->v[1], l);
        st_host(&prm->result->v[2], ab);
        st_host(&prm->result->v[3], bad);
        st_host(&prm->result->ms, (double)(wall_clock64() - ld_agent(prm->clock)) * prm->ms_per_tick);
        if (prm->done)
            announce(prm->result, prm->gate, prm->done);
    }
}

// one wave of a launch; prm is the first of the kernel's arguments
template <class S, int T, int B, int L, class Acc>
__device__ __forceinline__ void main_wave(const MainParams &prm)
{
    constexpr int R = T + B;
    constexpr int BL = B - L;                // levels expanded in LDS
    constexpr int NN_MAX = 1 << (BL - 1);    // include nodes of the last LDS level
    // real path: node 0 holds the level-(LA-1) node (R+1 modes), whose
    // exclude view is the tier-A leaf and whose include child the next one
    constexpr int X0 = std::is_same<S, double>::value ? 1 : 0;
    constexpr int kBufScalars = NodePlacement<R, BL, (int)sizeof(S), L, X0>{}.off[1 << BL] / (int)sizeof(S);
    __shared__ S bufB[kBufScalars];
    __shared__ S nBa[NN_MAX];          // real path alone (TuckedPivots)
    __shared__ RT<S> nInv[2 * NN_MAX];
    __shared__ RT<S> ndet[std::is_same<S, ddr>::value ? NN_MAX - 1 : (1 << BL) - 1];
    __shared__ uint16_t srcOff[(1 << (BL + 1)) - 1];
    __shared__ uint8_t srcNB[(1 << (BL + 1)) - 1];
    __shared__ uint8_t srcDet[(1 << (BL + 1)) - 1];
    __shared__ uint32_t blkRec[NB(R - 1 + X0)];
    __shared__ unsigned long long nodeRec[(1 << BL) - 1];

    const int lane = threadIdx.x;
    if (prm.gate && prm.gate->path != prm.gate_path) {
        // the matrix has another path, or is not valid.  The block that looks
        // last announces it: behind the end nothing may touch the workspace,
        // which may be the caller's (their looks come first in each block, and
        // a count of one address for up to RESULT_ROOTS blocks)
        if (prm.done_gated && lane == 0 &&
            __hip_atomic_fetch_add(prm.finished, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1 == gridDim.x)
            announce(prm.result, prm.gate, prm.done);
        return;
    }
    if (prm.clock && blockIdx.x == 0 && lane == 0)
        st_agent(prm.clock, (long long)wall_clock64());
    build_tables<S, R, BL + 1, L>(srcOff, srcNB, srcDet, nodeRec, blkRec, lane);
    __syncthreads();
    const TierB<S> tb{bufB, srcOff, srcNB, srcDet, nodeRec, blkRec, ndet, X0 ? nInv : nullptr, X0 ? nBa : nullptr};
    S *wscr = reinterpret_cast<S *>(prm.scratch + (long long)blockIdx.x * prm.scratch_stride);

    // The first item of each wave is its own block's; the queue counter hands
    // out the ones after the grid's.  A launch of no more items than waves
    // touches no counter at all (its one address serves the whole device's
    // waves one by one: 1024 of them took 13 to 17 us to get their first
    // tickets).  Not where blocks may start late (prm.tickets_only: launches on
    // part of the device, beside others): there the first items come from the
    // counter too, for an item that waits for its block ends the launch late
    // (a saturated stream of requests 1130 -> 1020 per second).
    const long long nfirst = prm.tickets_only ? 0 : (long long)gridDim.x;
    auto ticket = [&]() -> long long {
        return nfirst < prm.total_items ? nfirst + (long long)take_ticket(prm.counter, lane) : prm.total_items;
    };
    // the descriptors are read where they lie, by scalar loads: prm.one in the
    // kernel's arguments (prm is the first of them) unless there is a list
    typedef const __attribute__((address_space(4))) ProblemDesc CDesc;
    CDesc *probs = prm.probs ? (CDesc *)prm.probs
                             : (CDesc *)((const __attribute__((address_space(4))) char *)__builtin_amdgcn_kernarg_segment_ptr() +
                                         offsetof(MainParams, one));
    for (long long item = prm.tickets_only ? ticket() : blockIdx.x; item < prm.total_items; item = ticket()) {
        int lo = 0, hi = prm.nprob - 1;  // last problem with item_begin <= item
        while (lo < hi) {
            int mid = (lo + hi + 1) >> 1;
            if (probs[mid].item_begin <= item)
                lo = mid;
            else
                hi = mid - 1;
        }
        const ProblemDesc P = {probs[lo].C,          probs[lo].slots,      probs[lo].N,     probs[lo].k,
                               probs[lo].root_begin, probs[lo].item_begin, probs[lo].nroots};
        const long long root = P.root_begin + (item - P.item_begin);
        const int N = P.N, k = P.k, LA = N - R, D = LA - k;
        const S *C = reinterpret_cast<const S *>(P.C);
        // the wave's stack (tslot_off): the root node, tier-A slots k+1 ..
        // LA-1, and the running determinants of the tier-A levels on the
        // current path (used only when the root has more than one leaf)
        RT<S> *sdet = reinterpret_cast<RT<S> *>(wscr + tslot_off(N, k, LA));
        int bad = 0;

        // root: decisions on modes 0..k-1 given by the bits of root.  When
        // the node at the first included level fits the LDS buffer (free
        // until the first leaf), it is copied there, every include
        // eliminates in place in LDS, and only the final root node (N-k
        // modes, stride NB(N-k)) is written to the wave's stack.  Otherwise
        // the first include reads the matrix and the later ones rewrite the
        // root node in place in the stack with the matrix's stride NB(N).
        const S *rsrc = C;
        int rnb = NB(N);
        RT<S> rdet = rconst<RT<S>>(1.0);
        int rinc = 0;
        bool in_lds = false;  // the first leaf's node is in place in LDS
        const unsigned long long rbits = (unsigned long long)root & ((1ull << k) - 1);
        const int l0 = rbits ? __builtin_ctzll(rbits) : k;  // first included level
        if (rbits && NSZ(N - l0) <= kBufScalars) {
            const int nb0 = NB(N - l0);
            copy_node<S, true, false>(C, NB(N), bufB, nb0, N - l0, lane);
            __syncthreads();
            for (int l = l0; l < k; ++l) {
                if ((rbits >> l) & 1) {
                    RT<S> pd;
                    elim_lds<S>(bufB, nb0, N - l, lane, pd, bad);
                    rdet = rmul(rdet, pd);
                    ++rinc;
                }
            }
            // later leaves read the root node from the stack (a root of one
            // leaf has none); the first one is already here
            if (D > 0)
                copy_node<S, false, true>(bufB, nb0, wscr, NB(N - k), N - k, lane);
            restride_node<S, R + X0>(bufB, nb0, min(R + X0, N - k), lane);
            rsrc = wscr;
            rnb = NB(N - k);
            in_lds = true;
        } else {
            for (int l = 0; l < k; ++l) {
                if ((rbits >> l) & 1) {
                    RT<S> pd;
                    elim_inplace<S>(rsrc, rnb, wscr, rnb, N - l, lane, pd, bad);
                    rdet = rmul(rdet, pd);
                    ++rinc;
                    rsrc = wscr;
                }
            }
        }

        Acc acc;
        const long long nleaf = 1ll << D;
        for (long long x = 0; x < nleaf; ++x) {
            // double-double factor: an empty asm hides that the lane index
            // is the same in every leaf, so what the tiers derive from it
            // (block and node indices, table entries) is recomputed in each
            // leaf instead of being held in registers across the whole loop.
            // That brings the kernel to 252 registers, two waves per SIMD
            // (the real FP64 kernel does the same for tier B only).
            int lane = threadIdx.x;
            if constexpr (std::is_same<S, ddr>::value)
                __asm__ volatile("" : "+v"(lane));
            __builtin_assume((unsigned)lane < 64u);
            RT<S> ldet;
            int linc;
            if (x == 0) {
                // the first R modes of the root node (real path R + 1, or R
                // when the root is the leaf), restrided
                if (!in_lds)
                    copy_node<S, true, false>(rsrc, rnb, bufB, NB(R + X0), min(R + X0, N - k), lane);
                ldet = rdet;
                linc = rinc;
            } else {
                // leaf x differs from leaf x-1 from level lvl on: lvl becomes an
                // include, every deeper tier-A level an exclude
                const int t = __builtin_ctzll(x);
                const int lvl = LA - 1 - t;
                const long long xr = x >> (t + 1);
                const S *s;
                int snb;
                RT<S> sd;
                int si;
                if (xr == 0) {
                    s = rsrc;
                    snb = rnb;
                    sd = rdet;
                    si = rinc;
                } else {
                    const int sl = LA - (__builtin_ctzll(xr) + t + 1);
                    s = wscr + tslot_off(N, k, sl);
                    snb = NB(N - sl);
                    sd = sdet[sl];
                    // includes on the path down to level sl: the root's and
                    // the tier-A decisions above sl, bits LA-1-l of x
                    si = rinc + __popcll((unsigned long long)x >> (LA - sl));
                }
                RT<S> pd;
                if (X0 && t == 0) {
                    // the include at level LA-1: its source, the level-(LA-1)
                    // node of this path, is LDS node 0, updated in place
                    elim_leaf<S, R>(tb, lane, pd, bad);
                } else {
                    // the deepest slot a later step reads (level LA, or LA-1
                    // when node 0 holds that level) gets the child in LDS
                    // only; shallower ones also go to their stack slot
                    S *dst = (lvl + 1 < LA - X0) ? wscr + tslot_off(N, k, lvl + 1) : nullptr;
                    elim_global<S>(s, snb, dst, NB(N - lvl - 1), bufB, NB(R + X0), N - lvl, lane, pd, bad);
                }
                ldet = rmul(sd, pd);
                linc = si + 1;
                if (lane == 0)
                    sdet[lvl + 1] = ldet;
            }
            __syncthreads();
            if constexpr (std::is_same<Acc, AccStore>::value) {
                // subset index of the lane's first term: bit N-1-l is the
                // decision at level l, so the root's k bits reversed on top,
                // then the leaf index x (tier A, level LA-1 lowest), then the
                // lane (tier B's view bits and tier C's two lane levels), then
                // the T bits of the tail
                const unsigned long long rrev = k ? __builtin_bitreverse64((unsigned long long)root) >> (64 - k) : 0ull;
                acc.begin_leaf(prm.terms + ((rrev << (N - k)) | ((unsigned long long)x << R) | ((unsigned long long)lane << T)));
            }
            tierB<S, R, 1, BL, L>(tb, ldet, lane, bad);
            tierC<S, T, B, L, Acc>(tb, ldet, linc, N, lane, acc, bad, root == (1ll << k) - 1 && x == nleaf - 1);
            __syncthreads();
        }

        double h = acc.hi * acc.frame, l = acc.lo * acc.frame, ab = acc.abs_sum;
        constexpr bool is_dd = Acc::kDD;
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            double oh = __shfl_xor(h, off), ol = __shfl_xor(l, off), oa = __shfl_xor(ab, off);
            if constexpr (is_dd)
                dd_add2(h, l, oh, ol);
            else
                h += oh;
            ab += oa;
        }
        const int anybad = __any(bad);
        if (lane == 0) {
            // slots are overwritten, never accumulated, so running a root
            // again (the host's recovery from a numeric failure) is idempotent
            const bool forced = item + 1 == prm.fail_item1;
            double *sl = P.slots + 4 * root;
            const double v[4] = {forced ? __builtin_nan("") : h, l, ab,
                                 anybad ? SLOT_NOT_PD : (forced || !__builtin_isfinite(h)) ? SLOT_NUMERIC : 0.0};
#pragma unroll
            for (int j = 0; j < 4; ++j)
                st_agent(&sl[j], v[j]);
        }
        if constexpr (!std::is_same<Acc, AccStore>::value) {
            // these arguments are read here, not held from the kernel's start
            typedef const __attribute__((address_space(4))) MainParams CParams;
            CParams *late = (CParams *)__builtin_amdgcn_kernarg_segment_ptr();
            __asm__ volatile("" : "+s"(late));
            if (late->result)
                finish_root<Acc::kDD>(late, P.slots, lane);
        }
    }
}

template <class S, int T, int B, int L, class Acc>
__global__ void __launch_bounds__(64) tor_main(MainParams prm)
{
    main_wave<S, T, B, L, Acc>(prm);
}

// ---------------------------------------------------------------------------
// per-matrix sum of the root slots: thread t takes roots t, t + RED_THREADS,
// ... in index order, then the threads are combined by a fixed tree (within
// each wave, then across the waves), so the result does not depend on timing.
constexpr int RED_THREADS = 1024;

template <bool DD>
__device__ __forceinline__ void reduce_matrix(const ProblemDesc &P, double *result)
{
    constexpr int NW = RED_THREADS / 64;
    __shared__ double part[4][NW];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const long long nroots = 1ll << P.k;
    double h = 0.0, l = 0.0, ab = 0.0, bad = 0.0;
    for (long long r = t; r < nroots; r += RED_THREADS) {
        const double *s = P.slots + 4 * r;
        if (DD)
            dd_add2(h, l, s[0], s[1]);
        else
            h += s[0];
        ab += s[2];
        bad = fmax(bad, s[3]);
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1)
        red_step<DD>(h, l, ab, bad, off);
    if (lane == 0) {
        part[0][w] = h;
        part[1][w] = l;
        part[2][w] = ab;
        part[3][w] = bad;
    }
    __syncthreads();
    if (w == 0) {
        const bool in = lane < NW;
        h = in ? part[0][lane] : 0.0;
        l = in ? part[1][lane] : 0.0;
        ab = in ? part[2][lane] : 0.0;
        bad = in ? part[3][lane] : 0.0;
#pragma unroll
        for (int off = NW / 2; off >= 1; off >>= 1)
            red_step<DD>(h, l, ab, bad, off);
        if (lane == 0) {
            result[0] = h;
            result[1] = l;
            result[2] = ab;
            result[3] = bad;
        }
    }
}

template <bool DD>
__global__ void __launch_bounds__(RED_THREADS) tor_reduce(const ProblemDesc *probs, double *results)
{
    reduce_matrix<DD>(probs[blockIdx.x], results + 4 * blockIdx.x);
}

// one matrix, of the path the staging kernel gave it (a or b); the end of its
// chain
template <bool DD>
__global__ void __launch_bounds__(RED_THREADS) tor_reduce_one(const StageInfo *gate, int path_a, ProblemDesc a, int path_b,
                                                              ProblemDesc b, const long long *clock, double ms_per_tick,
                                                              EvalResult *result, unsigned long long done)
{
    __shared__ double r[4];
    const int path = gate->path;
    const bool mine = path == path_a || path == path_b;
    double ms = 0.0;
    if (threadIdx.x == 0 && mine)
        ms = (double)(wall_clock64() - *clock) * ms_per_tick;
    if (path == path_a)
        reduce_matrix<DD>(a, r);
    else if (path == path_b)
        reduce_matrix<DD>(b, r);
    if (threadIdx.x == 0) {  // the thread that wrote r
        if (mine) {
            for (int j = 0; j < 4; ++j)
                st_host(&result->v[j], r[j]);
            st_host(&result->ms, ms);
        }
        announce(result, gate, done);
    }
}

#ifndef TOR_KERNELS_TEMPLATES_ONLY
// Everything below is built once, in this translation unit; the
// double-double factor's kernel is instantiated and launched from
// tor_kernels_quad.hip, which includes the templates above on their own.
__global__ void tor_zero(unsigned long long *p, int count)
{
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count)
        p[i] = 0ull;
}

// ---------------------------------------------------------------------------
hipError_t launch_main_store(const MainParams &p, int grid, hipStream_t s)
{
    hipLaunchKernelGGL((tor_main<double, REAL_T, REAL_B, REAL_L, AccStore>), dim3(grid), dim3(64), 0, s, p);
    return hipGetLastError();
}

int main_store_occupancy()
{
    int n = 0;
    const hipError_t e =
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, tor_main<double, REAL_T, REAL_B, REAL_L, AccStore>, 64, 0);
    return e == hipSuccess ? n : 0;
}

hipError_t launch_main(int path, bool dd, const MainParams &p, int grid, hipStream_t s)
{
    if (path == PATH_QUAD) {
        return launch_main_quad(p, grid, s);
    } else if (path == PATH_REAL) {
        if (dd)
            hipLaunchKernelGGL((tor_main<double, REAL_T, REAL_B, REAL_L, AccAnchor>), dim3(grid), dim3(64), 0, s, p);
        else
            hipLaunchKernelGGL((tor_main<double, REAL_T, REAL_B, REAL_L, AccF64>), dim3(grid), dim3(64), 0, s, p);
    } else {
        if (dd)
            hipLaunchKernelGGL((tor_main<c64, CPLX_T, CPLX_B, CPLX_L, AccDD>), dim3(grid), dim3(64), 0, s, p);
        else
            hipLaunchKernelGGL((tor_main<c64, CPLX_T, CPLX_B, CPLX_L, AccF64>), dim3(grid), dim3(64), 0, s, p);
    }
    return hipGetLastError();
}

// ms per tick of the device's constant-rate clock (wall_clock64)
static double wall_ms_per_tick()
{
    static const double v = [] {
        int dev = 0, khz = 0;
        (void)hipGetDevice(&dev);
        (void)hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev);
        return khz > 0 ? 1.0 / khz : 0.0;
    }();
    return v;
}

// roots of a lone evaluation up to which its last wave forms the result
// (finish_root): one a lane
constexpr int RESULT_ROOTS = 64;

hipError_t launch_eval_one(const EvalOne &e, hipStream_t s)
{
    if (e.nrun < 1 || e.nrun > 2)
        return hipErrorInvalidValue;
    // one leaf: the first path's kernel stages the matrix itself (the FP64 sum,
    // an option, has no such kernel)
    const bool small = e.stage && e.dd && e.run[0].P.nroots == 1 && e.st.n <= SMALL_MODES;
    hipError_t err = small      ? hipSuccess
                     : e.stage ? launch_stage_one(e.st, e.counters, 4, s)
                               : launch_zero(e.counters, 4, s);
    // the paths whose roots a kernel of their own has to sum
    int red[2] = {-2, -2};
    for (int i = 0; i < e.nrun; ++i)
        // (fewer waves than roots would still look for tickets behind the end)
        if (e.run[i].P.nroots > RESULT_ROOTS || e.run[i].grid < e.run[i].P.nroots)
            red[i] = e.run[i].path;
    const bool reduce = red[0] >= 0 || red[1] >= 0;
    for (int i = 0; i < e.nrun && err == hipSuccess; ++i) {
        const EvalOne::Run &r = e.run[i];
        const bool last = !reduce && i == e.nrun - 1;
        MainParams p{};
        p.nprob = 1;
        p.one = r.P;
        p.total_items = r.P.nroots;
        p.counter = e.counters + i;
        p.scratch = r.scratch;
        p.scratch_stride = r.stride;
        p.fail_item1 = e.fail_root + 1;
        p.gate = e.st.info;
        p.gate_path = r.path;
        if (red[i] < 0) {
            p.result = e.result;
            p.finished = e.counters + 2 + i;
            p.done = last ? e.done : 0;
        }
        p.done_gated = last;
        p.clock = e.clock;
        p.ms_per_tick = wall_ms_per_tick();
        err = small && i == 0 ? launch_small(r.path, p, e.st, e.counters, 4, s) : launch_main(r.path, e.dd, p, r.grid, s);
    }
    if (err != hipSuccess || !reduce)
        return err;
    const ProblemDesc &a = e.run[0].P, &b = e.run[e.nrun - 1].P;
    if (e.dd)
        hipLaunchKernelGGL((tor_reduce_one<true>), dim3(1), dim3(RED_THREADS), 0, s, e.st.info, red[0], a, red[1], b, e.clock,
                           wall_ms_per_tick(), e.result, e.done);
    else
        hipLaunchKernelGGL((tor_reduce_one<false>), dim3(1), dim3(RED_THREADS), 0, s, e.st.info, red[0], a, red[1], b, e.clock,
                           wall_ms_per_tick(), e.result, e.done);
    return hipGetLastError();
}

// the slots of a click_all launch; sets whether the outputs may be written
template <bool DD>
__global__ void __launch_bounds__(RED_THREADS) tor_reduce_click(const StageInfo *gate, ProblemDesc P, double *det,
                                                                long long *clock, double ms_per_tick, ClickResult *result)
{
    __shared__ double r[4];
    const bool mine = gate->path == PATH_REAL;
    if (mine)
        reduce_matrix<DD>(P, r);
    if (threadIdx.x == 0) {  // the thread that wrote r
        const double sq = det[0], bad = det[1];
        det[2] = mine && gate->status == 0 && r[3] == 0.0 && bad == 0.0 && sq > 0.0 ? 1.0 : 0.0;
        const long long now = wall_clock64();
        if (mine) {
            for (int j = 0; j < 4; ++j)
                st_host(&result->v[j], r[j]);
            st_host(&result->ms[0], (double)(now - clock[0]) * ms_per_tick);
        }
        clock[1] = now;
        st_host(&result->det[0], sq);
        st_host(&result->det[1], bad);
        st_host(&result->status, gate->status);
        st_host(&result->path, gate->path);
    }
}

// the end of a click_all call: the transform's time (an event at either end
// would put packets of its own between the kernels)
__global__ void tor_click_end(const long long *clock, double ms_per_tick, ClickResult *result)
{
    if (threadIdx.x == 0)
        st_host(&result->ms[1], (double)(wall_clock64() - clock[1]) * ms_per_tick);
}

// What bounds a small call is the chain of its launches: six kernels and
// nothing between them.  A copy each for the state, the descriptors,
// sqrt(det) and the verdict, an event on either side of two of the kernels and
// a wait before the transform made the 15 modes' call 111 us, against 70 so
// (25 modes: 777 and 745).
hipError_t launch_click_all(const ClickAll &c, hipStream_t s)
{
    hipError_t err = launch_stage_det(c.st, c.counter, c.det, s);
    if (err != hipSuccess)
        return err;
    MainParams p{};
    p.nprob = 1;
    p.one = c.P;
    p.total_items = c.P.nroots;
    p.counter = c.counter;
    p.scratch = c.scratch;
    p.scratch_stride = c.stride;
    p.gate = c.st.info;
    p.gate_path = PATH_REAL;
    p.terms = c.terms;
    p.clock = c.clock;
    err = launch_main_store(p, c.grid, s);
    if (err != hipSuccess)
        return err;
    const double tick = wall_ms_per_tick();
    if (c.dd)
        hipLaunchKernelGGL((tor_reduce_click<true>), dim3(1), dim3(RED_THREADS), 0, s, c.st.info, c.P, c.det, c.clock, tick,
                           c.result);
    else
        hipLaunchKernelGGL((tor_reduce_click<false>), dim3(1), dim3(RED_THREADS), 0, s, c.st.info, c.P, c.det, c.clock, tick,
                           c.result);
    err = hipGetLastError();
    if (err == hipSuccess)
        err = launch_click_transform(c.terms, c.g, c.N, c.M, c.det, c.probs, c.tor_hi, c.tor_lo, &c.result->full, s);
    if (err != hipSuccess)
        return err;
    hipLaunchKernelGGL(tor_click_end, dim3(1), dim3(64), 0, s, c.clock, tick, c.result);
    return hipGetLastError();
}

int main_occupancy(int path)
{
    int n = 0;
    hipError_t e;
    if (path == PATH_QUAD)
        return main_occupancy_quad();
    if (path == PATH_REAL)
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, tor_main<double, REAL_T, REAL_B, REAL_L, AccAnchor>, 64, 0);
    else
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, tor_main<c64, CPLX_T, CPLX_B, CPLX_L, AccDD>, 64, 0);
    return e == hipSuccess ? n : 0;
}

hipError_t launch_reduce(const ProblemDesc *probs, int nprob, double *results, bool dd, hipStream_t s)
{
    if (dd)
        hipLaunchKernelGGL((tor_reduce<true>), dim3(nprob), dim3(RED_THREADS), 0, s, probs, results);
    else
        hipLaunchKernelGGL((tor_reduce<false>), dim3(nprob), dim3(RED_THREADS), 0, s, probs, results);
    return hipGetLastError();
}

hipError_t launch_zero(unsigned long long *p, int count, hipStream_t s)
{
    hipLaunchKernelGGL(tor_zero, dim3((count + 63) / 64), dim3(64), 0, s, p, count);
    return hipGetLastError();
}
#endif  // TOR_KERNELS_TEMPLATES_ONLY

}  // namespace tor
