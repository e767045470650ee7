// Plans of the kernels of kspace.h: tiles, their searches on the host, and the deal of work
// to waves and lanes, apart from the kernels so that the host can check them for any shape.
#pragma once

#include <algorithm>
#include <cstddef>

#include "sse_common.h"

namespace sse {
namespace ks {

constexpr size_t kLdsBytes = 160 * 1024;
constexpr size_t kEntry = 16;  // bytes of a complex entry

// x / d for 0 <= x < 2^16, 1 <= d < 2^16, with the reciprocal taken on the host
struct Div {
    uint32_t m, one;  // one: d == 1
    __host__ __device__ Div() : m(0), one(0) {}
    __host__ explicit Div(int d) : m(d == 1 ? 0u : (uint32_t)(0xffffffffu / (uint32_t)d) + 1u), one(d == 1 ? 0xffffffffu : 0u) {}
    __host__ __device__ __forceinline__ int quot(int x) const {
        return (int)((uint32_t)(((uint64_t)(uint32_t)x * m) >> 32) | ((uint32_t)x & one));
    }
};

// LDS row of norb complex entries: an odd number of 16-byte entries, so that
// lanes that read down a column hit distinct banks
__host__ __device__ __forceinline__ int row_len(int n) { return n | 1; }

// The first task of a wave when the tasks from `shift` on go to waves 0, 1, ...: the
// tasks of one step are dealt on from where the last step's ended.  A mask, since
// wave - shift is negative as soon as the steps before had more tasks than waves.
template <int WAVES>
__host__ __device__ __forceinline__ int first_task(int wave, int shift) {
    static_assert((WAVES & (WAVES - 1)) == 0, "a power of two");
    return (wave - shift) & (WAVES - 1);
}

// ------------------------------------------------------------------ corr_kspace_kernel
constexpr int kCorrThreads = 512, kCorrWaves = kCorrThreads / 64;
constexpr int kCorrCB = 5, kCorrXB = 5;  // columns per pass of Y, outputs (i, r) per pass of X

struct CorrTile {
    int wb;                    // frequencies of a lane
    int eb, rc, es, nwb, nwg;  // energies, rows, shares of the energies, frequency blocks of a workgroup and groups of them
    int halo_lo, halo_hi;      // planes of Y before and after the tile
    int ncb;
    ks::Div by_n, by_ncb, by_xb[2], by_rc[2], by_row[2], by_nn;
    int nel, y_entries, x_entries, g_entries;
    size_t lds;
};

// What a thread sums: entry el, direction j, frequencies w0 + 1 .. w0 + wb, share es of the energies
struct CorrLane {
    int el, j, es, w0;
};
__host__ __device__ __forceinline__ CorrLane corr_lane(const CorrTile& t, int tid, int wg) {
    const int rest = tid / t.nel;
    return CorrLane{tid % t.nel, rest / t.nwb % 3, rest / t.nwb / 3, (wg * t.nwb + rest % t.nwb) * t.wb};
}
// Energies it sums of a tile with e_n of them, in a chunk with nel entries.  A lane whose
// frequencies all lie beyond nw (the last group may have fewer blocks than the others) has
// none: its window would leave the planes of Y.
__host__ __device__ __forceinline__ int corr_energies(const CorrTile& t, const CorrLane& l, int nw, int nel, int e_n) {
    const int share = t.eb / t.es, mine = e_n - l.es * share;
    return l.es < t.es && l.el < nel && l.w0 < nw && mine > 0 ? (mine < share ? mine : share) : 0;
}

// the tile with the least time under the quantisation of each step
inline bool corr_tile(const Dims& d, bool hi, bool lo, CorrTile* best) {
    const int n = (int)d.norb, np = row_len(n);
    if (d.norb > 32 || d.nkz > 128 || d.nw > 4096 || d.ne >= (int64_t(1) << 28) || d.nb >= (1 << 20)) return false;
    auto up = [](double a, double b) { return (double)(int64_t)((a + b - 1) / b); };
    double best_cost = 0.0;
    bool found = false;
    // both branches' windows of five frequencies do not fit the registers
    for (int wb = 2; wb <= (hi && lo ? 4 : 5); ++wb)
    for (int rc = 1; rc <= n && 3 * rc * n <= kCorrThreads; ++rc) {
        CorrTile t{};
        const int64_t nwb_all = (d.nw + wb - 1) / wb;
        t.wb = wb;
        const int nel = rc * n;
        t.rc = rc;
        t.nel = nel;
        t.nwb = (int)std::min<int64_t>(nwb_all, kCorrThreads / (3 * nel));
        t.nwg = (int)((nwb_all + t.nwb - 1) / t.nwb);
        const int max_es = kCorrThreads / (3 * nel * t.nwb);
        t.halo_lo = lo ? (int)nwb_all * wb : 0;
        t.halo_hi = hi ? (int)nwb_all * wb : 0;
        t.ncb = (n + kCorrCB - 1) / kCorrCB;
        const int tail = n % rc ? n % rc : rc;
        t.by_n = Div(n);
        t.by_ncb = Div(t.ncb);
        t.by_xb[0] = Div((3 * rc + kCorrXB - 1) / kCorrXB);
        t.by_xb[1] = Div((3 * tail + kCorrXB - 1) / kCorrXB);
        t.by_rc[0] = Div(rc);
        t.by_rc[1] = Div(tail);
        t.by_row[0] = Div(nel);
        t.by_row[1] = Div(tail * n);
        t.by_nn = Div(n * n);
        for (int es = 1; es <= max_es; ++es)
            for (int eb = es; eb <= 128; eb += es) {
                if (eb > es && eb - es >= d.ne) break;
                const int64_t y = (int64_t)(eb + t.halo_lo + t.halo_hi) * 3 * nel, x = (int64_t)eb * 3 * nel;
                const int64_t gr = (int64_t)eb * rc * np, bt = (int64_t)eb * n * np;
                const int64_t all = std::max<int64_t>(y + x + gr + bt + 3 * n * n, wb * kCorrThreads) + d.nkz + 1;
                if (all > (int64_t)(kLdsBytes / kEntry)) break;
                t.eb = eb;
                t.es = es;
                t.y_entries = (int)y;
                t.x_entries = (int)x;
                t.g_entries = (int)gr;
                t.lds = kEntry * (size_t)all;
                const int occ = t.lds <= kLdsBytes / 2 ? 2 : 1;
                const int r = eb * rc <= 64 ? 1 : 2;
                // vector instructions of the busiest SIMD (its share of the waves, rounded up) per
                // tile and chunk, the waits of a step, and the prologue of a chunk; the steps left
                // over from groups of wb energies wait for their operands
                const double halo = t.halo_lo + t.halo_hi;
                const double s1 = (eb / es + eb / es % wb * 5.0) * (wb * (hi && lo ? 14.0 : 12.0) + 10);
                const double r1 = n * kCorrCB * 4.4 * r + 80, rt = 3 * up((double)eb * rc, 64 * r) * t.ncb;
                const double l1 = n * kCorrXB * 8.8 + 100, lt = up((double)eb * n, 128) * up(3.0 * rc, kCorrXB);
                const double fixed = 400 + 25 * (up((double)eb * nel, kCorrThreads) + up((double)eb * n * n, kCorrThreads)) +
                                     4 * up(halo * 3 * nel, kCorrThreads);
                const double tile = up(up(3.0 * nel * t.nwb * es, 64), 4) * s1 + up(rt, 4) * r1 + up(lt, 4) * l1 +
                                    kCorrWaves / 4 * fixed + 3000.0 / occ;
                const double fill = up(halo, eb) * (up(rt, 4) * r1 + 1000);
                const double cost = up(n, rc) * (up((double)d.ne, eb) * tile + fill) * t.nwg;
                if (!found || cost < best_cost) {
                    best_cost = cost;
                    *best = t;
                    found = true;
                }
            }
    }
    return found;
}

}  // namespace ks
}  // namespace sse
