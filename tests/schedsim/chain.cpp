// A lone evaluation's one chain (launch_eval_one) on the CPU, against the HIP
// stand-in: what the host does around it.  The chain's stand-in runs on the
// stream like the kernels do, forms the slots as the recursive stand-in of
// stubs.cpp does, and can
//   fail    make root g_fail_root of its first run report a numeric failure;
//   late    write the slots after it has announced the result, as a host that
//           does not wait for the stream may find them.
// hipMalloc (linked with --wrap) refuses allocations above g_alloc_limit.
// Exit status 0 when every scenario passes.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <thread>
#include <vector>

#include "../../include/tor.h"
#include "../../paper_2109_04528_amd/csrc/tor_internal.hpp"

namespace {
std::atomic<long long> g_fail_root{-1};
std::atomic<bool> g_late{false};
std::atomic<int> g_chains{0};
std::atomic<size_t> g_alloc_limit{~(size_t)0};
int g_failed = 0;

void check(bool ok, const char *what, int i = -1)
{
    if (!ok) {
        std::fprintf(stderr, "check failed: %s (%d)\n", what, i);
        g_failed = 1;
    }
}
}  // namespace

hipError_t real_malloc(void **p, size_t bytes) __asm__("__real__Z9hipMallocPPvm");
hipError_t wrap_malloc(void **p, size_t bytes) __asm__("__wrap__Z9hipMallocPPvm");
hipError_t wrap_malloc(void **p, size_t bytes)
{
    return bytes > g_alloc_limit ? (hipError_t)hipErrorOutOfMemory : real_malloc(p, bytes);
}

namespace tor {

hipError_t launch_eval_one(const EvalOne &e, hipStream_t s)
{
    ++g_chains;
    const EvalOne ev = e;
    const long long fail = g_fail_root.exchange(-1);
    const bool late = g_late;
    fake_enqueue(s, [=] {
        double c = ev.st.O[0];
        const bool general = ev.st.O[1] > 0.0;
        const int path = (ev.st.flags & STAGE_DD) ? PATH_QUAD : general || (ev.st.flags & STAGE_FORCE_CPLX) ? PATH_CPLX : PATH_REAL;
        if (ev.stage) {
            std::memcpy(ev.st.out, &c, sizeof c);
            ev.st.info->status = 0;
            ev.st.info->path = path;
        }
        std::memcpy(&c, ev.st.out, sizeof c);
        const EvalOne::Run *run = nullptr;
        for (int i = 0; i < ev.nrun; i++)
            if (ev.run[i].path == ev.st.info->path)
                run = &ev.run[i];
        double v[4] = {0.0, 0.0, 0.0, 0.0};
        std::vector<double> slots;
        if (run) {
            const double per = std::ldexp(1.0, run->P.N - run->P.k);
            for (long long r = 0; r < run->P.nroots; r++) {
                const bool bad = r == fail;
                const double sl[4] = {bad ? NAN : c * per, 0.0, per, bad ? SLOT_NUMERIC : 0.0};
                slots.insert(slots.end(), sl, sl + 4);
                v[0] += sl[0];
                v[2] += sl[2];
                v[3] = std::max(v[3], sl[3]);
            }
            ev.st.info->N = run->P.N;
        }
        auto put = [&] {
            if (run)
                std::memcpy(run->P.slots, slots.data(), sizeof(double) * slots.size());
        };
        if (!late)
            put();
        std::memcpy(ev.result->v, v, sizeof v);
        ev.result->ms = 0.01;
        ev.result->status = ev.st.info->status;
        ev.result->path = ev.st.info->path;
        ev.result->N = ev.st.info->N;
        __atomic_store_n(&ev.result->done, ev.done, __ATOMIC_RELEASE);
        if (late) {
            std::this_thread::sleep_for(std::chrono::milliseconds(20));
            put();
        }
    });
    return hipSuccess;
}

}  // namespace tor

int main()
{
    // one root, few, many; the real and the complex path
    for (int n : {5, 14, 20})
        for (bool general : {false, true})
            for (bool late : {false, true}) {
                tor_ctx *ctx = nullptr;
                check(tor_create(&ctx, nullptr) == TOR_OK, "create");
                std::vector<double> O(8 * (size_t)n * n, 0.0);
                O[0] = 0.5 + n;
                O[1] = general ? 1.0 : 0.0;
                if (!general)  // what the host looks at to guess the path
                    O[2 * ((size_t)n * 2 * n + n)] = O[0];
                tor_result clean{}, r{};
                check(tor_eval(ctx, n, O.data(), 2L * n, &clean) == TOR_OK && clean.launches == 1, "clean", n);
                g_late = late;
                g_fail_root = n == 5 ? 0 : 3;
                check(tor_eval(ctx, n, O.data(), 2L * n, &r) == TOR_OK && r.launches == 2, late ? "recovery, late slots" : "recovery", n);
                check(r.tor == clean.tor && r.sum_abs == clean.sum_abs && r.path == clean.path, "recovered value", n);
                g_late = false;
                check(tor_eval(ctx, n, O.data(), 2L * n, &r) == TOR_OK && r.launches == 1 && r.tor == clean.tor, "after it", n);
                // a forced failure goes through the same chain and is used up
                const int before = g_chains;
                check(tor_debug_fail_root(ctx, 0, 2) == TOR_OK, "debug");
                check(tor_eval(ctx, n, O.data(), 2L * n, &r) == TOR_OK && g_chains > before, "forced failure's chain", n);
                check(tor_eval(ctx, n, O.data(), 2L * n, &r) == TOR_OK && r.launches == 1, "used up", n);
                tor_destroy(ctx);
            }
    // device memory for one path's launch but not for either's: whatever a batch
    // of one is given, a lone evaluation is given too
    int refused = 0, general_path = 0;
    for (int n : {14, 22, 30})
        for (size_t limit = (size_t)1 << 20; limit <= (size_t)400 << 20; limit += limit / 8) {
            g_alloc_limit = limit;
            std::vector<double> O(8 * (size_t)n * n, 0.0);
            O[0] = 0.25;
            O[2 * ((size_t)n * 2 * n + n)] = O[0];
            const double *ptr = O.data();
            const long ld = 2L * n;
            tor_ctx *a = nullptr, *b = nullptr;
            check(tor_create(&a, nullptr) == TOR_OK && tor_create(&b, nullptr) == TOR_OK, "create");
            tor_result ra{}, rb{};
            const int before = g_chains;
            const int rca = tor_eval(a, n, ptr, ld, &ra), rcb = tor_eval_batch(b, 1, &n, &ptr, &ld, &rb);
            check(rca == rcb || rca == TOR_OK, "served within the limit", n);
            if (rca == TOR_OK && rcb == TOR_OK) {
                check(ra.tor == rb.tor && ra.path == rb.path, "value within the limit", n);
                general_path += g_chains == before;
            } else {
                ++refused;
            }
            tor_destroy(a);
            tor_destroy(b);
        }
    check(refused > 0 && general_path > 0, "limits on both sides");
    std::printf("done %d\n", g_failed);
    return g_failed;
}
