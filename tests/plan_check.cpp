// Host checks of csrc/kspace_plan.h; one check per run, named by argv[1].  Prints what is
// wrong and returns 1, or returns 0.
#include <algorithm>
#include <chrono>
#include <cstdio>
#include <cstring>

#include "kspace_plan.h"

using namespace sse;

static Dims dims(int64_t nkz, int64_t ne, int64_t nw, int64_t na, int64_t nb, int64_t norb) {
    return Dims{nkz, ne, nkz, nw, na, nb, norb, 1};
}

// every task of the three products of a step is taken by exactly one wave, whatever the
// steps before left over
static int first_task() {
    constexpr int kWaves = ks::kCorrWaves;
    for (int ncb = 1; ncb <= 7; ++ncb)
        for (int rows = 1; rows <= 3; ++rows)
            for (int from = 0; from < kWaves; ++from)
                for (int j = 0; j < 3; ++j) {
                    int taken[32] = {};
                    const int tasks = rows * ncb;
                    for (int wave = 0; wave < kWaves; ++wave) {
                        const int first = ks::first_task<kWaves>(wave, from + j * ncb);
                        if (first < 0 || first >= kWaves) {
                            printf("first task %d: %d passes, from %d, direction %d, wave %d\n", first, ncb, from, j, wave);
                            return 1;
                        }
                        for (int t = first; t < tasks; t += kWaves) ++taken[t];
                    }
                    for (int t = 0; t < tasks; ++t)
                        if (taken[t] != 1) {
                            printf("task %d taken %d times: %d passes, from %d, direction %d\n", t, taken[t], ncb, from, j);
                            return 1;
                        }
                }
    return 0;
}

// the planes of Y that a lane of corr_kspace_kernel reads: those of its energies shifted by
// w0 + 1 .. w0 + wb up and down
static int corr_window() {
    for (int both = 0; both < 2; ++both)
        for (int n = 1; n <= 25; n += n < 12 ? 1 : 4)
            for (int nw = 1; nw <= 130; nw += nw < 50 ? 1 : 9)
                for (int ne : {7, 64}) {
                    ks::CorrTile t;
                    if (!ks::corr_tile(dims(2, ne, nw, 4, 2, n), true, both, &t)) continue;
                    const int planes = t.eb + t.halo_lo + t.halo_hi, tail = n % t.rc ? n % t.rc * n : t.nel;
                    for (int wg = 0; wg < t.nwg; ++wg)
                        for (int tid = 0; tid < ks::kCorrThreads; ++tid)
                            for (int e_n : {t.eb, 1})
                                for (int nel : {t.nel, tail}) {
                                    const ks::CorrLane l = ks::corr_lane(t, tid, wg);
                                    const int cnt = ks::corr_energies(t, l, nw, nel, e_n);
                                    if (cnt <= 0) continue;
                                    const int first = l.es * (t.eb / t.es) + t.halo_lo, last = first + cnt - 1;
                                    if (last + l.w0 + t.wb >= planes || (both && first - l.w0 - t.wb < 0)) {
                                        printf("norb %d nw %d ne %d both %d: group %d of %d, frequencies from %d, planes %d\n", n, nw,
                                               ne, both, wg, t.nwg, l.w0, planes);
                                        return 1;
                                    }
                                }
                }
    return 0;
}

// Time of the searches that five small and middling calls do once each, the least of
// thirty: microseconds, where trying every combination took 0.4 ms for the five
static int corr_search_time() {
    using Clock = std::chrono::steady_clock;
    double sum = 0.0;
    for (const Dims& d : {dims(3, 16, 2, 16, 4, 4), dims(5, 64, 6, 200, 4, 8), dims(7, 128, 10, 512, 4, 10), dims(3, 48, 5, 250, 3, 6),
                          dims(3, 101, 4, 500, 3, 5)}) {
        double least = 1e9;
        for (int rep = 0; rep < 30; ++rep) {
            const auto t0 = Clock::now();
            ks::CorrTile t;
            if (!ks::corr_tile(d, true, false, &t)) return 1;
            least = std::min(least, std::chrono::duration<double, std::micro>(Clock::now() - t0).count());
        }
        sum += least;
    }
    printf("%.1f us\n", sum);
    return sum < 200.0 ? 0 : 1;
}

// the smallest tile fits exactly where the search finds one
static int corr_support() {
    for (int both = 0; both < 2; ++both)
        for (int n = 1; n <= 32; ++n)
            for (int nw = 1; nw <= 400; nw += nw < 20 ? 1 : 17) {
                ks::CorrTile t;
                const Dims d = dims(2, 64, nw, 4, 2, n);
                if (ks::corr_fits(d, true, both) == ks::corr_tile(d, true, both, &t)) continue;
                printf("norb %d nw %d both %d\n", n, nw, both);
                return 1;
            }
    return 0;
}

// the parts of a launch hold every (atom, workgroup of an atom) once, in at most 2^32 - 1
// work-items each
static int launch_parts() {
    for (int threads : {256, 512})
        for (int64_t na : {1LL, 9LL, 4864LL, 1100000LL, 300000000LL})
            for (int64_t per : {1LL, 28LL, 1000LL, 3000000LL, 2000000000LL}) {
                if (na > 10000 && per > 10000) continue;  // beyond any card's memory, and many parts
                int64_t next_a = 0, next = 0;
                bool ok = true;
                ks::launch_parts(na, per, threads, [&](ks::LaunchPart p) {
                    const int64_t atoms = (int64_t)p.groups / p.n;
                    ok = ok && p.a0 == next_a && p.first == next && (int64_t)p.groups == atoms * p.n && atoms % 8 == 0 && atoms > 0 &&
                         (int64_t)p.groups * threads < (int64_t(1) << 32);
                    next += p.n;
                    if (next == per) next_a += atoms, next = 0;
                });
                if (ok && next == 0 && next_a >= na) continue;
                printf("%lld atoms of %lld workgroups of %d\n", (long long)na, (long long)per, threads);
                return 1;
            }
    return 0;
}

int main(int argc, char** argv) {
    const struct {
        const char* name;
        int (*run)();
    } checks[] = {{"first_task", first_task}, {"corr_window", corr_window}, {"corr_search_time", corr_search_time}, {"corr_support", corr_support}, {"launch_parts", launch_parts}};
    for (const auto& c : checks)
        if (argc > 1 && !strcmp(argv[1], c.name)) return c.run();
    printf("no such check\n");
    return 2;
}
