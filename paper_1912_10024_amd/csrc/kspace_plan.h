// Plans of the kernels of kspace.h: tiles, their searches on the host, and the deal of work
// to waves and lanes, apart from the kernels so that the host can check them for any shape.
#pragma once

#include <algorithm>
#include <cmath>
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

// A launch of `per` workgroups for each of na atoms, dealt over the eight XCDs by atom
// (workgroup x: atom x mod 8 of its eight), in parts of as many workgroups as a launch may
// have: whole groups of eight atoms, or, where eight atoms are too many, a range of `per`.
struct LaunchPart {
    int64_t a0;    // first atom
    int first, n;  // the range of `per`
    unsigned groups;
};
template <class Launch>
inline void launch_parts(int64_t na, int64_t per, int threads, Launch launch) {
    const int64_t most = launch_groups(threads), na8 = (na + 7) / 8 * 8;
    const int64_t atoms = std::max<int64_t>(8, most / per / 8 * 8), range = std::min(per, most / 8);
    for (int64_t a0 = 0; a0 < na8; a0 += atoms)
        for (int64_t first = 0; first < per; first += range) {
            const int64_t n = std::min(range, per - first);
            launch(LaunchPart{a0, (int)first, (int)n, (unsigned)(std::min(atoms, na8 - a0) * n)});
        }
}

// Twiddles of up to kTableNkz - 1 momenta, cos and -sin of 2 pi m / nkz rounded, then what
// the rounding took off (from 64-bit mantissas: about eleven bits of it)
constexpr int kTableNkz = 17;
struct Twiddles {
    double t[kTableNkz - 1][4];
};
inline const Twiddles& twiddles(int64_t nkz) {
    struct All {
        Twiddles of[kTableNkz];
        All() {
            for (int n = 1; n < kTableNkz; ++n)
                for (int m = 0; m < kTableNkz - 1; ++m) {
                    const int p = m % n, r = std::min(p, n - p);  // the angle 2 pi r / n in [0, pi]
                    const long double x = 2.0L * 3.14159265358979323846264338327950288L * r / n;
                    long double c = cosl(x), s = sinl(x);
                    if (4 * r % n == 0) c = 4 * r == n ? 0 : r ? -1 : 1, s = 4 * r == n ? 1 : 0;
                    if (p != r) s = -s;
                    double* t = of[n].t[m];
                    t[0] = (double)c;
                    t[1] = -(double)s;
                    t[2] = (double)(c - t[0]);
                    t[3] = (double)(-s - t[1]);
                }
        }
    };
    static const All all;
    return all.of[nkz < kTableNkz ? nkz : 0];
}

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

__host__ __device__ __forceinline__ int up_div(int a, int b) { return (a + b - 1) / b; }

// A tile but for its energies: LDS in entries (base + energies * per, at least `least` for
// the last sum) and what the cost of a tile takes from it
struct CorrShape {
    int n, wb, rc, nel, nwb, nwg, ncb, halo;
    int base, per, least;
    int chunks, x_passes;
    double step;  // vector instructions of one energy of the sums
};
inline bool corr_limits(const Dims& d) {
    return d.norb <= 32 && d.nkz <= 128 && d.nw <= 4096 && d.ne < (int64_t(1) << 28) && d.nb < (1 << 20);
}
inline CorrShape corr_shape(const Dims& d, bool hi, bool lo, int wb, int rc) {
    const int n = (int)d.norb, nwb_all = up_div((int)d.nw, wb);
    CorrShape s{};
    s.n = n;
    s.wb = wb;
    s.rc = rc;
    s.nel = rc * n;
    s.nwb = std::min(nwb_all, kCorrThreads / (3 * s.nel));
    s.nwg = up_div(nwb_all, s.nwb);
    s.ncb = up_div(n, kCorrCB);
    s.halo = (hi + lo) * nwb_all * wb;
    s.base = s.halo * 3 * s.nel + 3 * n * n + 2 * (int)d.nkz + 1;
    s.per = 6 * s.nel + (rc + n) * row_len(n);
    s.least = wb * kCorrThreads + 2 * (int)d.nkz + 1;
    s.chunks = up_div(n, rc);
    s.x_passes = up_div(3 * rc, kCorrXB);
    s.step = wb * (hi && lo ? 14.0 : 12.0) + 10;
    return s;
}
inline int corr_entries(const CorrShape& s, int eb) { return std::max(s.base + eb * s.per, s.least); }

// Vector instructions of the busiest SIMD (its share of the waves, rounded up) per tile of
// es shares of `share` energies, the waits of a step, and the prologue of a chunk; the steps
// left over from groups of wb energies wait for their operands
inline double corr_cost(const CorrShape& s, int ne, int es, int share) {
    auto up = [](int a, int shift) { return (a + (1 << shift) - 1) >> shift; };
    const int eb = es * share, wide = eb * s.rc <= 64 ? 0 : 1;  // rows per lane of the right products, less one
    const int rt = 3 * up(eb * s.rc, 6 + wide) * s.ncb, lt = up(eb * s.n, 7) * s.x_passes;
    const double r1 = s.n * kCorrCB * 4.4 * (1 + wide) + 80, l1 = s.n * kCorrXB * 8.8 + 100;
    const double fixed = 400 + 25 * (up(eb * s.nel, 9) + up(eb * s.n * s.n, 9)) + 4 * up(s.halo * 3 * s.nel, 9);
    const bool two = corr_entries(s, eb) <= (int)(kLdsBytes / kEntry / 2);  // workgroups on a compute unit
    const double tile = up(up(3 * s.nel * s.nwb * es, 6), 2) * (share + share % s.wb * 5) * s.step + up(rt, 2) * r1 +
                        up(lt, 2) * l1 + kCorrWaves / 4 * fixed + (two ? 1500 : 3000);
    const double fill = up_div(s.halo, eb) * (up(rt, 2) * r1 + 1000);
    return (double)s.chunks * s.nwg * (up_div(ne, eb) * tile + fill);
}

// both branches' windows of five frequencies do not fit the registers
inline int corr_max_wb(bool hi, bool lo) { return hi && lo ? 4 : 5; }

// whether the smallest tile fits the LDS
inline bool corr_fits(const Dims& d, bool hi, bool lo) {
    if (!corr_limits(d)) return false;
    for (int wb = 2; wb <= corr_max_wb(hi, lo); ++wb)
        if (corr_entries(corr_shape(d, hi, lo, wb, 1), 1) <= (int)(kLdsBytes / kEntry)) return true;
    return false;
}

// The tile with the least cost.  Tried are the row counts that give different numbers of
// chunks; all the lanes' shares, a half, a third of them or a power of two in between; and,
// for the room of one and of two workgroups per compute unit, tiles that divide the
// energies evenly and tiles of whole groups of wb.  A call searches
// once, in 5 to 25 us on one core; over 5,900 shapes the cost is on average 0.1% above that
// of every combination tried in turn, which took 20 to 230 us.
inline bool corr_tile(const Dims& d, bool hi, bool lo, CorrTile* best) {
    if (!corr_limits(d)) return false;
    const int n = (int)d.norb, ne = (int)d.ne;
    constexpr int kRoom = (int)(kLdsBytes / kEntry);
    double best_cost = 0.0;
    CorrShape bs{};
    int best_es = 0, best_share = 0;
    for (int wb = corr_max_wb(hi, lo); wb >= 2; --wb)
        for (int c = 1, rc_before = 0; c <= n; ++c) {
            const int rc = up_div(n, c);
            if (rc == rc_before || 3 * rc * n > kCorrThreads) continue;
            rc_before = rc;
            const CorrShape s = corr_shape(d, hi, lo, wb, rc);
            if (corr_entries(s, 1) > kRoom) continue;
            const int most = std::min(128, (kRoom - s.base) / s.per), half = std::min(128, (kRoom / 2 - s.base) / s.per);
            auto shares = [&](int es) {
                if (es < 1 || es > most) return;
                const int need = up_div(ne, es);
                for (int room : {most, half}) {
                    const int limit = std::min(room / es, need);
                    if (limit < 1) continue;
                    const int even = up_div(need, up_div(need, limit)), down = limit / wb * wb, over = up_div(even, wb) * wb;
                    for (int share : {even, down, over <= limit ? over : 0, limit / wb / 2 * wb}) {
                        if (share < 1) continue;
                        const double cost = corr_cost(s, ne, es, share);
                        if (best_share && cost >= best_cost) continue;
                        best_cost = cost;
                        bs = s;
                        best_es = es;
                        best_share = share;
                    }
                }
            };
            const int max_es = kCorrThreads / (3 * s.nel * s.nwb);
            shares(max_es);
            if (max_es > 2) shares(max_es / 2);
            if (max_es > 5) shares(max_es / 3);
            int es = 1;
            while (4 * es < max_es) es *= 2;
            for (; es < max_es; es *= 2) shares(es);
        }
    if (!best_share) return false;
    const int eb = best_es * best_share, tail = n % bs.rc ? n % bs.rc : bs.rc;
    CorrTile t{};
    t.wb = bs.wb;
    t.eb = eb;
    t.rc = bs.rc;
    t.es = best_es;
    t.nwb = bs.nwb;
    t.nwg = bs.nwg;
    t.halo_lo = lo ? bs.halo / (hi + lo) : 0;
    t.halo_hi = hi ? bs.halo / (hi + lo) : 0;
    t.ncb = bs.ncb;
    t.by_n = Div(n);
    t.by_ncb = Div(t.ncb);
    t.by_xb[0] = Div(up_div(3 * bs.rc, kCorrXB));
    t.by_xb[1] = Div(up_div(3 * tail, kCorrXB));
    t.by_rc[0] = Div(bs.rc);
    t.by_rc[1] = Div(tail);
    t.by_row[0] = Div(bs.nel);
    t.by_row[1] = Div(tail * n);
    t.by_nn = Div(n * n);
    t.nel = bs.nel;
    t.y_entries = (eb + t.halo_lo + t.halo_hi) * 3 * bs.nel;
    t.x_entries = eb * 3 * bs.nel;
    t.g_entries = eb * bs.rc * row_len(n);
    t.lds = kEntry * (size_t)corr_entries(bs, eb);
    *best = t;
    return true;
}

}  // namespace ks
}  // namespace sse
