// tor_small.hip -- a lone evaluation of a matrix that is one tier-A leaf (at most
// 11 modes on the real path, 9 on the others) as one launch: a workgroup
// stages the matrix, and its first wave goes on as the recursive kernel's only
// one.  What bounds such a call is the chain of latencies, not the work, so the
// end of a kernel, the start of the next and the matrix's way through another die's
// cache are taken out of it: 10 modes 26.3 us a call against 27.5.  The rest is
// one wave's 22 000 cycles (9 us), the staging's one pass over the bus, and the
// launch and the answer on their way.
#define TOR_KERNELS_TEMPLATES_ONLY
#include "tor_kernels.hip"
#include "tor_stage.hpp"

namespace tor {

constexpr int SMALL_THREADS = 256;  // as the staging kernel of so few modes
constexpr int SMALL_ENTRIES = NB(2 * SMALL_MODES);

template <class S, int T, int B, int L, class Acc>
__global__ void __launch_bounds__(SMALL_THREADS) tor_small(MainParams prm, StageDesc D, unsigned long long *zero, int nzero)
{
    __shared__ c64 tri[SMALL_ENTRIES];
    if ((int)threadIdx.x < nzero)
        zero[threadIdx.x] = 0ull;
    stage_matrix<SMALL_THREADS, SMALL_ENTRIES>(D, tri);
    __syncthreads();
    if (__builtin_amdgcn_readfirstlane((int)threadIdx.x) >= 64)
        return;  // whole waves: the barriers that follow wait for the first alone
    main_wave<S, T, B, L, Acc>(prm);
}

hipError_t launch_small(int path, const MainParams &p, const StageDesc &d, unsigned long long *zero, int nzero, hipStream_t s)
{
    if (p.total_items != 1 || p.probs || d.n > SMALL_MODES)
        return hipErrorInvalidValue;
    const dim3 one(1), nt(SMALL_THREADS);
    if (path == PATH_REAL)
        hipLaunchKernelGGL((tor_small<double, REAL_T, REAL_B, REAL_L, AccAnchor>), one, nt, 0, s, p, d, zero, nzero);
    else if (path == PATH_QUAD)
        hipLaunchKernelGGL((tor_small<ddr, QUAD_T, QUAD_B, QUAD_L, AccQ>), one, nt, 0, s, p, d, zero, nzero);
    else
        hipLaunchKernelGGL((tor_small<c64, CPLX_T, CPLX_B, CPLX_L, AccDD>), one, nt, 0, s, p, d, zero, nzero);
    return hipGetLastError();
}

}  // namespace tor
