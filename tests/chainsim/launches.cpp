// The launches of a lone evaluation's chain, looked at on the CPU: links the
// built library, takes the place of hipLaunchKernel, and records every launch of
// launch_eval_one with its first argument (MainParams of the recursive kernels,
// which are the ones with workgroups of one wave).
// Prints nothing and exits with 0 if in every chain the last launch alone
// announces the end, and ends the chain whatever the verdict.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstring>
#include <vector>

#include "../../paper_2109_04528_amd/csrc/tor_internal.hpp"

struct Launch {
    dim3 grid, block;
    tor::MainParams p;
    bool main;
};
static std::vector<Launch> g_launches;

extern "C" hipError_t hipLaunchKernel(const void *, dim3 grid, dim3 block, void **args, size_t, hipStream_t)
{
    Launch l{grid, block, {}, block.x == 64 && grid.x > 0};
    if (l.main)
        std::memcpy(&l.p, args[0], sizeof l.p);
    g_launches.push_back(l);
    return hipSuccess;
}
extern "C" hipError_t hipGetLastError() { return hipSuccess; }
// what a launch's host stub asks the runtime for (which fails without a device)
static dim3 g_grid, g_block;
extern "C" hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t, hipStream_t)
{
    g_grid = grid;
    g_block = block;
    return hipSuccess;
}
extern "C" hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *shared, hipStream_t *s)
{
    *grid = g_grid;
    *block = g_block;
    *shared = 0;
    *s = nullptr;
    return hipSuccess;
}

static int g_bad = 0;
static void check(bool ok, const char *what, long long a, long long b, int path)
{
    if (!ok) {
        std::fprintf(stderr, "check failed: %s (roots %lld %lld, first path %d)\n", what, a, b, path);
        g_bad = 1;
    }
}

int main()
{
    using namespace tor;
    // roots of the two paths a matrix may take (0: no second path)
    const long long roots[] = {0, 1, 2, 64, 128, 2048};
    for (int first : {PATH_REAL, PATH_CPLX})
        for (long long a : roots)
            for (long long b : roots)
                for (int waves : {2048, 32}) {
                    if (a == 0)
                        continue;
                    static char mem[4096];
                    static EvalResult res;
                    EvalOne e{};
                    e.stage = true;
                    e.st.n = e.st.M = 14;
                    e.st.info = (StageInfo *)mem;
                    e.counters = (unsigned long long *)(mem + 256);
                    e.clock = (long long *)(mem + 512);
                    e.nrun = b ? 2 : 1;
                    e.dd = true;
                    e.result = &res;
                    e.done = 7;
                    e.fail_root = -1;
                    const long long n[2] = {a, b};
                    for (int i = 0; i < e.nrun; i++) {
                        e.run[i].path = i ? (first == PATH_REAL ? PATH_CPLX : PATH_REAL) : first;
                        e.run[i].P.nroots = n[i];
                        e.run[i].grid = (int)(n[i] < waves ? n[i] : waves);
                    }
                    g_launches.clear();
                    check(launch_eval_one(e, nullptr) == hipSuccess, "launched", a, b, first);
                    const size_t last = g_launches.size() - 1;
                    bool reduced = !g_launches[last].main;
                    for (size_t i = 0; i < g_launches.size(); i++) {
                        const Launch &l = g_launches[i];
                        if (!l.main)
                            continue;
                        check(l.p.gate != nullptr, "looks at the verdict", a, b, first);
                        check(i == last || (l.p.done == 0 && !l.p.done_gated), "announced before the chain's end", a, b, first);
                        if (i == last)
                            check(l.p.done == 7 && l.p.done_gated && l.p.result && l.p.finished && l.grid.x == l.p.total_items,
                                  "the end is announced once by every block", a, b, first);
                        else
                            check(reduced || l.p.result, "a sum for every path", a, b, first);
                        if (l.p.result)
                            check(l.p.total_items <= 64 && l.grid.x == l.p.total_items, "a wave for each root", a, b, first);
                    }
                }
    return g_bad;
}
