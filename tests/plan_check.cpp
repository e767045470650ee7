// Host checks of csrc/kspace_plan.h; one check per run, named by argv[1].  Prints what is
// wrong and returns 1, or returns 0.
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

int main(int argc, char** argv) {
    const struct {
        const char* name;
        int (*run)();
    } checks[] = {{"first_task", first_task}};
    for (const auto& c : checks)
        if (argc > 1 && !strcmp(argv[1], c.name)) return c.run();
    printf("no such check\n");
    return 2;
}
