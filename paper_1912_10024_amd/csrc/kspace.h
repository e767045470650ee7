// Building blocks of the kernels that work in the momentum transform.
//
// The sum over phonon momenta of Eq. 3 is a cyclic convolution over kz, and the
// products with grad H do not touch the momentum, so with
//   hat X[m] = sum_k X[k] exp(-2 pi i k m / Nkz)
// every transformed momentum m is a problem of its own with one momentum:
//   hat Sigma[m, E, a] = sum_n sum_i A_i . U_i,   U_i[E] = sum_{j, w} hat D_ij[m, w] (H_j[E-w] + H_j[E+w]),
//   H_j[E] = hat G[m, E, b] . A_j^H.
// Against the sum over (q, w) of whole products this is Nkz times fewer
// multiplications, and taking the right factor before and the left factor after
// the filter over the frequencies costs 6 block products per (edge, momentum,
// energy) instead of the 12 of all nine A_i . G . A_j^H.
//
// All of it runs on the fp64 vector ALUs, whose peak on this chip is that of the
// fp64 matrix cores: in each step one operand is the same for every lane (a
// grad H entry, broadcast from a register, or a coefficient, broadcast from LDS), so a lane needs one
// LDS read for 12 to 24 multiply-adds, nothing is padded to a tile, and every size
// takes the same code.
#pragma once

#include <type_traits>

#include "kspace_plan.h"
#include "sse_common.h"

namespace sse {
namespace ks {

constexpr int kEBlk = 4;  // energies of one lane in the filter

// one complex entry of an LDS array (16-byte aligned)
__device__ __forceinline__ cd ld(const cd* p) {
    const double2 v = *reinterpret_cast<const double2*>(p);
    return cd{v.x, v.y};
}
__device__ __forceinline__ void st(cd* p, cd v) { *reinterpret_cast<double2*>(p) = make_double2(v.re, v.im); }

// exp(-2 pi i m / nkz), m = 0 .. nkz-1, each as a rounded value and what rounding took off.
// The same twiddle enters the transform of G, that of D and the inverse: with few momenta
// its rounding would be one error with one sign in all terms (at three momenta it made dG
// 1.1 times further off than the direct sum).  From kTableNkz on there are enough different
// ones for that not to matter, and the second parts are zero.
__device__ __forceinline__ void stage_twiddles(cd* tw, const Twiddles& table, int nkz, int tid, int threads) {
    for (int m = tid; m < nkz; m += threads) {
        if (nkz < kTableNkz) {
            st(tw + 2 * m, cd{table.t[m][0], table.t[m][1]});
            st(tw + 2 * m + 1, cd{table.t[m][2], table.t[m][3]});
        } else {
            double s, c;
            sincospi(2.0 * (double)m / (double)nkz, &s, &c);
            st(tw + 2 * m, cd{c, -s});
            st(tw + 2 * m + 1, cd{0.0, 0.0});
        }
    }
}

// One pair of terms, k and nkz - k, of a sum over the momenta: the twiddle tw[0] + tw[1] and
// its conjugate times a and b, as Re (a + b) + i Im (a - b).  Half the products of the two terms
// by themselves, and a chain half as long to round.  CONJ: with the conjugate twiddles.
template <bool CONJ = false>
__device__ __forceinline__ void pair_fma(cd& s, cd a, cd b, cd hi, cd lo) {
    const cd p{a.re + b.re, a.im + b.im}, q{a.re - b.re, a.im - b.im};
    if (CONJ) hi.im = -hi.im, lo.im = -lo.im;
    s.re = fma(lo.re, p.re, s.re);
    s.im = fma(lo.re, p.im, s.im);
    s.re = fma(-lo.im, q.im, s.re);
    s.im = fma(lo.im, q.re, s.im);
    s.re = fma(hi.re, p.re, s.re);
    s.im = fma(hi.re, p.im, s.im);
    s.re = fma(-hi.im, q.im, s.re);
    s.im = fma(hi.im, q.re, s.im);
}
// the term at nkz / 2 (even nkz), whose twiddle is (-1)^m
__device__ __forceinline__ void middle_add(cd& s, cd a, int m) {
    s.re += m & 1 ? -a.re : a.re;
    s.im += m & 1 ? -a.im : a.im;
}
// sum_k load(k) tw[k m mod nkz]
template <bool CONJ = false, class Load>
__device__ __forceinline__ cd momentum_sum(int nkz, int m, const cd* tw, Load load) {
    cd s = load(0);
    int j = m;
#pragma unroll 2
    for (int k = 1; 2 * k < nkz; ++k) {
        pair_fma<CONJ>(s, load(k), load(nkz - k), ld(tw + 2 * j), ld(tw + 2 * j + 1));
        j += m;
        j -= j >= nkz ? nkz : 0;
    }
    if (!(nkz & 1)) middle_add(s, load(nkz / 2), m);
    return s;
}

// A block array, or its transform: complex elements between momenta, atoms and energies,
// and the energies that it holds
struct Blocks {
    const double* p;
    int64_t kst, atom, est;
    int first, count;
};
// an array [nkz][ne][na][slots][norb][norb], its slot 0
inline Blocks array_blocks(const double* p, const Dims& d, int64_t slots) {
    const int64_t atom = slots * d.norb * d.norb;
    return Blocks{p, d.ne * d.na * atom, atom, d.na * atom, 0, (int)d.ne};
}
// a transform of its energies [first, first + count), [nkz][na][count][norb][norb]
inline Blocks hat_blocks(const double* p, const Dims& d, int64_t first, int64_t count) {
    const int64_t nn = d.norb * d.norb;
    return Blocks{p, d.na * count * nn, count * nn, nn, (int)first, (int)count};
}
// Where a tile of energies x rows of it is loaded from
struct Source {
    const double* p;   // block of the wanted atom at momentum 0, energy `first`
    int64_t kst, est;
    int first, count;
};
__device__ __forceinline__ Source source(const Blocks& b, int64_t a) {
    return Source{b.p + 2 * a * b.atom, b.kst, b.est, b.first, b.count};
}

// Transform or direct sum.  The transform rounds every value of a cyclic sum relative to the
// largest of its Nkz values, the direct sum each relative to its own terms.  The two are
// alike (within about kSpread) as soon as one of the arrays under the sum has blocks of like
// size at all momenta, whatever the others hold: spread_kernel finds out for every block of
// one array, and of a second and third only where those before are not like that, and sets a
// bit per array in a word of the workspace.  Where all the bits of a sum are set, the kernels of
// the transform leave at once and the direct ones run; else the other way round.
constexpr double kSpread = 32.0;
constexpr int kSpreadD = 1, kSpreadG = 2, kSpreadSigma = 4;  // bits: coefficients, G (or Go), dSigma (or Gs)
constexpr int64_t kWordBytes = 16;  // of the workspace, so that what follows stays aligned
inline void* aligned(void* p) { return reinterpret_cast<void*>((reinterpret_cast<uintptr_t>(p) + 15) & ~uintptr_t(15)); }
struct Gate {
    const int* word;  // NULL: open, whatever the kernel
    int mask;
};
__device__ __forceinline__ bool all_spread(const Gate& g) { return (__builtin_amdgcn_readfirstlane(*g.word) & g.mask) == g.mask; }
template <bool DIRECT>
__device__ __forceinline__ bool shut(const Gate& g) {
    return g.word && all_spread(g) != DIRECT;
}
// workgroups of a direct launch behind a gate: few, since they mostly find it shut, each
// with several tiles if not
constexpr unsigned kGatedGroups = 1024;

// The blocks of one energy and atom at the nkz momenta, nn entries each, are of like size: the
// largest part of the largest is at most kSpread times that of the smallest, and finite.
// L lanes (a power of two, aligned in the wave) work on one block, l the lane's number.
__device__ __forceinline__ bool like_blocks(const double* p, int64_t kst, int nkz, int nn, int l, int L) {
    double least = __builtin_inf(), most = 0.0;
    auto part = [](double v) { return fabs(v) <= 1.7976931348623157e308 ? fabs(v) : __builtin_inf(); };
    for (int k0 = 0; k0 < nkz; k0 += 4) {
        double m[4] = {0.0, 0.0, 0.0, 0.0};
        for (int x = l; x < nn; x += L) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const cd v = cload(p, (k0 + u < nkz ? k0 + u : k0) * kst + x);
                m[u] = fmax(m[u], fmax(part(v.re), part(v.im)));
            }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            for (int o = 1; o < L; o <<= 1) m[u] = fmax(m[u], __shfl_xor(m[u], o));
            least = fmin(least, m[u]);
            most = fmax(most, m[u]);
        }
    }
    return most <= 1.7976931348623157e308 && most <= kSpread * least;
}
// lanes for blocks of nn entries
inline int block_lanes(int64_t nn) {
    int l = 1;
    while (l < 64 && l < nn) l *= 2;
    return l;
}

// Without a workspace Pi keeps the finding in its output: a workgroup's first output holds
// kMarker until the direct kernel writes it.  A signalling NaN, which no operation returns.
constexpr unsigned long long kMarker = 0x7ff4535345306b73ull;
__device__ __forceinline__ bool marked(const double* out, int64_t entry) {
    return *reinterpret_cast<const unsigned long long*>(out + 2 * entry) == kMarker;
}

constexpr int kDirect = 0;  // blocks of one momentum as they are, from an array or from its transform
constexpr int kTrans = 1;   // transformed over the momenta while they are loaded, from an array


// Rows r0 .. r0+rc-1 of the source blocks of energies e_first .. e_first+new_-1 into
// LDS, entry (ew, r, u) of [ew][rc][row_len].  CT: of the conjugate transpose of
// every block (whose transform at m is that of the block at -m, conjugate transposed:
// kt = -m).  Energies outside the grid give zeros.  U entries per thread are
// loaded together, which is what hides the latency.
template <int THREADS, int SRC, bool CT>
__device__ __forceinline__ void load_rows(const Source& s, const cd* tw, int nkz, int kt, int e_first, int new_,
                                          int r0, int rc, int n, Div by_row, Div by_n, cd* sG, int tid) {
    constexpr int U = SRC == kTrans ? 4 : 8;
    const int nrow = rc * n, total = new_ * nrow, np = row_len(n);
    const double* base = s.p + (SRC == kTrans ? 0 : 2 * kt * s.kst);
    for (int x0 = tid; x0 < total; x0 += U * THREADS) {
        const double* p[U];
        bool ok[U];
        int dst[U];
        cd acc[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int x = x0 + u * THREADS;
            const int xx = x < total ? x : 0;
            const int ew = by_row.quot(xx), rem = xx - ew * nrow, r = by_n.quot(rem), c = rem - r * n;
            const int e = e_first + ew - s.first;
            ok[u] = e >= 0 && e < s.count;
            dst[u] = x < total ? (ew * rc + r) * np + c : -1;
            p[u] = base + 2 * ((ok[u] ? e : 0) * s.est + (CT ? c * n + r0 + r : r0 * n + rem));
            acc[u] = cd{0.0, 0.0};
        }
        if constexpr (SRC == kTrans) {
            // momentum_sum of U entries at a time
#pragma unroll
            for (int u = 0; u < U; ++u) acc[u] = cload(p[u], 0);
            int m = kt;  // k * kt mod nkz
#pragma unroll 2
            for (int k = 1; 2 * k < nkz; ++k) {
                const cd hi = ld(tw + 2 * m), lo = ld(tw + 2 * m + 1);
#pragma unroll
                for (int u = 0; u < U; ++u) pair_fma(acc[u], cload(p[u], k * s.kst), cload(p[u], (nkz - k) * s.kst), hi, lo);
                m += kt;
                m -= m >= nkz ? nkz : 0;
            }
            if (!(nkz & 1)) {
#pragma unroll
                for (int u = 0; u < U; ++u) middle_add(acc[u], cload(p[u], nkz / 2 * s.kst), kt);
            }
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u) acc[u] = cload(p[u], 0);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (dst[u] < 0) continue;
            st(sG + dst[u], ok[u] ? (CT ? cd{acc[u].re, -acc[u].im} : acc[u]) : cd{0.0, 0.0});
        }
    }
}

// The same rows through registers: ask() issues the loads, put() stores them later, so that
// other work hides their latency.  U entries per thread; what is left is loaded by put().
template <int THREADS, int U, int SRC, bool CT>
struct RowsAhead {
    cd v[U];
    __device__ __forceinline__ cd get(const Source& s, const cd* tw, int nkz, int kt, int e, int at) const {
        e -= s.first;
        const bool ok = e >= 0 && e < s.count;
        const double* p = s.p + 2 * ((SRC == kTrans ? 0 : kt * s.kst) + (ok ? e : 0) * s.est + at);
        cd a;
        if constexpr (SRC == kTrans)
            a = momentum_sum(nkz, kt, tw, [&](int k) { return cload(p, k * s.kst); });
        else
            a = cload(p, 0);
        if (!ok) a = cd{0.0, 0.0};
        return CT ? cd{a.re, -a.im} : a;
    }
    __device__ __forceinline__ void ask(const Source& s, const cd* tw, int nkz, int kt, int e_first, int new_, int r0,
                                        int rc, int n, Div by_row, Div by_n, int tid) {
        const int nrow = rc * n, total = new_ * nrow;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int x = tid + u * THREADS < total ? tid + u * THREADS : 0;
            const int ew = by_row.quot(x), rem = x - ew * nrow, r = by_n.quot(rem), c = rem - r * n;
            v[u] = get(s, tw, nkz, kt, e_first + ew, CT ? c * n + r0 + r : r0 * n + rem);
        }
    }
    __device__ __forceinline__ void put(const Source& s, const cd* tw, int nkz, int kt, int e_first, int new_, int r0,
                                        int rc, int n, Div by_row, Div by_n, cd* dst, int tid) const {
        const int nrow = rc * n, total = new_ * nrow, np = row_len(n);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int x = tid + u * THREADS;
            const int ew = by_row.quot(x), rem = x - ew * nrow, r = by_n.quot(rem), c = rem - r * n;
            if (x < total) st(dst + (ew * rc + r) * np + c, v[u]);
        }
        for (int x = tid + U * THREADS; x < total; x += THREADS) {
            const int ew = by_row.quot(x), rem = x - ew * nrow, r = by_n.quot(rem), c = rem - r * n;
            st(dst + (ew * rc + r) * np + c, get(s, tw, nkz, kt, e_first + ew, CT ? c * n + r0 + r : r0 * n + rem));
        }
    }
};

// Products with a uniform operand.  The 2 CB doubles of a step's uniform operands
// (CB complex entries of grad H) sit in one register, double l of them in lane l of
// every row of 16 lanes, and the multiply-adds read them with the DPP row broadcast,
// which costs nothing.  Through scalar registers they took a scalar load per entry, whose
// results return out of order and from a cache that four workgroups share: the
// products then ran at 40% of the rate they reach from the vector memory path.
// All 64 lanes have to be active.  The wait states are those that a DPP read needs
// after a vector write of its source.
#define SSE_FMAC(D, S, X, K) "v_fmac_f64_dpp " D ", " S ", " X " row_newbcast:" K " row_mask:0xf bank_mask:0xf\n"
// p0 += f[K0] x0, p1 += f[K0] x1, p2 += f[K1] x0, p3 += f[K1] x1 (CONJ: conj(f))
template <bool CONJ, int K0, int K1>
__device__ __forceinline__ void fma4(cd& p0, cd& p1, cd& p2, cd& p3, double f, cd x0, cd x1) {
#define SSE_FMA4(SR, SI)                                                                                            \
    asm("s_nop 1\n" SSE_FMAC("%0", "%8", "%9", "%13") SSE_FMAC("%1", "%8", "%10", "%13")                            \
            SSE_FMAC("%2", "%8", "%11", "%13") SSE_FMAC("%3", "%8", "%12", "%13") SSE_FMAC("%4", "%8", "%9", "%15")  \
                SSE_FMAC("%5", "%8", "%10", "%15") SSE_FMAC("%6", "%8", "%11", "%15")                                \
                    SSE_FMAC("%7", "%8", "%12", "%15") SSE_FMAC("%0", SR, "%10", "%14")                              \
                        SSE_FMAC("%1", SI, "%9", "%14") SSE_FMAC("%2", SR, "%12", "%14")                             \
                            SSE_FMAC("%3", SI, "%11", "%14") SSE_FMAC("%4", SR, "%10", "%16")                        \
                                SSE_FMAC("%5", SI, "%9", "%16") SSE_FMAC("%6", SR, "%12", "%16")                     \
                                    SSE_FMAC("%7", SI, "%11", "%16")                                                 \
        : "+&v"(p0.re), "+&v"(p0.im), "+&v"(p1.re), "+&v"(p1.im), "+&v"(p2.re), "+&v"(p2.im), "+&v"(p3.re),          \
          "+&v"(p3.im)                                                                                               \
        : "v"(f), "v"(x0.re), "v"(x0.im), "v"(x1.re), "v"(x1.im), "n"(2 * K0), "n"(2 * K0 + 1), "n"(2 * K1),         \
          "n"(2 * K1 + 1))
    if constexpr (CONJ)
        SSE_FMA4("%8", "-%8");
    else
        SSE_FMA4("-%8", "%8");
#undef SSE_FMA4
}
// p0 += f[K] x0, p1 += f[K] x1
template <bool CONJ, int K>
__device__ __forceinline__ void fma2(cd& p0, cd& p1, double f, cd x0, cd x1) {
#define SSE_FMA2(SR, SI)                                                                                           \
    asm("s_nop 1\n" SSE_FMAC("%0", "%4", "%5", "%9") SSE_FMAC("%1", "%4", "%6", "%9") SSE_FMAC("%2", "%4", "%7", "%9") \
            SSE_FMAC("%3", "%4", "%8", "%9") SSE_FMAC("%0", SR, "%6", "%10") SSE_FMAC("%1", SI, "%5", "%10")       \
                SSE_FMAC("%2", SR, "%8", "%10") SSE_FMAC("%3", SI, "%7", "%10")                                    \
        : "+&v"(p0.re), "+&v"(p0.im), "+&v"(p1.re), "+&v"(p1.im)                                                   \
        : "v"(f), "v"(x0.re), "v"(x0.im), "v"(x1.re), "v"(x1.im), "n"(2 * K), "n"(2 * K + 1))
    if constexpr (CONJ)
        SSE_FMA2("%4", "-%4");
    else
        SSE_FMA2("-%4", "%4");
#undef SSE_FMA2
}
// p0 += f[K0] x, p1 += f[K1] x (K1 == K0: p0 only)
template <bool CONJ, int K0, int K1>
__device__ __forceinline__ void fma2r(cd& p0, cd& p1, double f, cd x) {
#define SSE_FMA2R(SR, SI, TR, TI)                                                                                       \
    if constexpr (K1 != K0)                                                                                     \
        asm("s_nop 1\n" SSE_FMAC("%0", "%4", "%5", "%7") SSE_FMAC("%1", "%4", "%6", "%7")                       \
                SSE_FMAC("%2", "%4", "%5", "%9") SSE_FMAC("%3", "%4", "%6", "%9")                               \
                    SSE_FMAC("%0", SR, "%6", "%8") SSE_FMAC("%1", SI, "%5", "%8")                               \
                        SSE_FMAC("%2", SR, "%6", "%10") SSE_FMAC("%3", SI, "%5", "%10")                         \
            : "+&v"(p0.re), "+&v"(p0.im), "+&v"(p1.re), "+&v"(p1.im)                                            \
            : "v"(f), "v"(x.re), "v"(x.im), "n"(2 * K0), "n"(2 * K0 + 1), "n"(2 * K1), "n"(2 * K1 + 1));        \
    else                                                                                                        \
        asm("s_nop 1\n" SSE_FMAC("%0", "%2", "%3", "%5") SSE_FMAC("%1", "%2", "%4", "%5")                       \
                SSE_FMAC("%0", TR, "%4", "%6") SSE_FMAC("%1", TI, "%3", "%6")                                   \
            : "+&v"(p0.re), "+&v"(p0.im)                                                                        \
            : "v"(f), "v"(x.re), "v"(x.im), "n"(2 * K0), "n"(2 * K0 + 1))
    if constexpr (CONJ) {
        SSE_FMA2R("%4", "-%4", "%2", "-%2");
    } else {
        SSE_FMA2R("-%4", "%4", "-%2", "%2");
    }
#undef SSE_FMA2R
}
#undef SSE_FMAC

// acc[r][c] += f_c x_r (CONJ: conj(f_c)) for two operands x per lane
template <int CB, bool CONJ, int C = 0>
__device__ __forceinline__ void fma_block(cd (&acc)[2][CB], double f, const cd (&x)[2]) {
    static_assert(CB <= 8, "16 doubles per row of lanes");
    if constexpr (C + 2 <= CB) {
        fma4<CONJ, C, C + 1>(acc[0][C], acc[1][C], acc[0][C + 1], acc[1][C + 1], f, x[0], x[1]);
        fma_block<CB, CONJ, C + 2>(acc, f, x);
    } else if constexpr (C < CB) {
        fma2<CONJ, C>(acc[0][C], acc[1][C], f, x[0], x[1]);
    }
}
// the same for one operand per lane
template <int CB, bool CONJ, int C = 0>
__device__ __forceinline__ void fma_block(cd (&acc)[1][CB], double f, const cd (&x)[1]) {
    static_assert(CB <= 8, "16 doubles per row of lanes");
    if constexpr (C < CB) {
        cd none{0.0, 0.0};
        constexpr int D = C + 1 < CB ? C + 1 : C;
        fma2r<CONJ, C, D>(acc[0][C], C + 1 < CB ? acc[0][D] : none, f, x[0]);
        fma_block<CB, CONJ, C + 2>(acc, f, x);
    }
}

// double `comp` of the uniform operand this lane holds: entry min(l / 2, CB - 1), re or im
template <int CB>
__device__ __forceinline__ int uniform_entry(int lane) {
    const int c = (lane & 15) >> 1;
    return c < CB ? c : CB - 1;
}

// acc[r][c] += f_c(k) x_r(k) for k in [0, len).  factor(k): this lane's double of step k's
// uniform operands, asked for TB steps ahead; operand(k, x): the lane's own from LDS,
// asked for one step ahead.
template <int R, int CB, bool CONJ, class Factor, class Operand>
__device__ __forceinline__ void uniform_product(cd (&acc)[R][CB], int len, Factor factor, Operand operand) {
    constexpr int TB = 4;
    double fa[TB], fb[TB];
    cd x[2][R];
    auto ask = [&](double (&f)[TB], int k0) {
#pragma unroll
        for (int u = 0; u < TB; ++u) f[u] = factor(k0 + u < len ? k0 + u : len - 1);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto mul = [&](const double (&f)[TB], int k0) {
#pragma unroll
        for (int u = 0; u < TB; ++u) {
            if (k0 + u < len) {
                operand(k0 + u + 1 < len ? k0 + u + 1 : len - 1, x[(u + 1) & 1]);
                __builtin_amdgcn_sched_barrier(0);
                fma_block<CB, CONJ>(acc, f[u], x[u & 1]);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    ask(fa, 0);
    operand(0, x[0]);
    for (int k0 = 0; k0 < len; k0 += 2 * TB) {
        ask(fb, k0 + TB);
        mul(fa, k0);
        if (k0 + TB >= len) break;
        ask(fa, k0 + 2 * TB);
        mul(fb, k0 + TB);
    }
}

// The three blocks of grad H of an edge into LDS (the uniform operands are read from
// there: from memory every pass of a product began with the latency of a load)
template <int THREADS>
__device__ __forceinline__ void stage_factor(const double* __restrict__ A, int64_t edge, int nn, cd* sA, int tid) {
    for (int x = tid; x < 3 * nn; x += THREADS) st(sA + x, cload(A, 3 * edge * nn + x));
}

// out(row)[c] = sum_u sG[row][u] . f(u, c) for `rows` rows: a lane owns R rows, 64
// apart, of a group of 64 R, CB columns at a time.  RT: f(u, c) = conj(M[c][u]) (the
// right factor grad_j H^H), else f(u, c) = M[u][c].
template <int WAVES, int R, int CB, bool RT, class Out>
__device__ __forceinline__ void right_product(const cd* sG, const cd* sM, int rows, int n, int ncb,
                                              Div by_ncb, int first, int lane, Out out) {
    const int np = row_len(n);
    const int tasks = (rows + 64 * R - 1) / (64 * R) * ncb;
    for (int t = first; t < tasks; t += WAVES) {
        const int tr = by_ncb.quot(t), c0 = (t - tr * ncb) * CB;
        const int row = tr * 64 * R + lane;
        const cd* g[R];
        cd acc[R][CB];
#pragma unroll
        for (int r = 0; r < R; ++r) g[r] = sG + (row + 64 * r < rows ? row + 64 * r : 0) * np;
#pragma unroll
        for (int c = 0; c < CB; ++c)
#pragma unroll
            for (int r = 0; r < R; ++r) acc[r][c] = cd{0.0, 0.0};
        const int fc = c0 + uniform_entry<CB>(lane), cc = fc < n ? fc : n - 1;
        const double* f = reinterpret_cast<const double*>(sM) + 2 * (RT ? cc * n : cc) + (lane & 1);
        const int step = RT ? 2 : 2 * n;
        uniform_product<R, CB, RT>(
            acc, n, [&](int u) { return f[u * step]; },
            [&](int u, cd (&x)[R]) {
#pragma unroll
                for (int r = 0; r < R; ++r) x[r] = ld(g[r] + u);
            });
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (row + 64 * r >= rows) continue;
            cd* o = out(row + 64 * r);
#pragma unroll
            for (int c = 0; c < CB; ++c)
                if (c0 + c < n) st(o + c0 + c, acc[r][c]);
        }
    }
}

// acc += d * x
__device__ __forceinline__ void cacc(cd& acc, cd d, cd x) { cfma(acc, d, x); }

// One step of the filter for kEBlk energies: acc[i][e] += D_i (lo[e] + hi[e]), or
// with one table per branch Dl_i lo[e] + Dh_i hi[e]
template <bool TWO>
__device__ __forceinline__ void filter_step(cd (&acc)[3][kEBlk], const cd* lo, const cd* hi, const cd* Dl, const cd* Dh) {
#pragma unroll
    for (int e = 0; e < kEBlk; ++e) {
        if constexpr (TWO) {
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                cacc(acc[i][e], Dl[i], lo[e]);
                cacc(acc[i][e], Dh[i], hi[e]);
            }
        } else {
            const cd x{lo[e].re + hi[e].re, lo[e].im + hi[e].im};
#pragma unroll
            for (int i = 0; i < 3; ++i) cacc(acc[i][e], Dl[i], x);
        }
    }
}

// The filter over the frequencies for one direction j: X points at the lane's
// entry of the plane of its first energy minus nw (planes `es` entries apart), sL
// at the coefficients [w][i] of j for the E - w branch and sH for E + w (TWO).
// A window of kEBlk planes per branch slides with w through registers (slot
// index = plane mod kEBlk), so a step reads two planes and three coefficients
// from LDS for 12 kEBlk multiply-adds.
template <bool TWO>
__device__ __forceinline__ void filter(cd (&acc)[3][kEBlk], const cd* X, int es, int nw, const cd* sL, const cd* sH) {
    static_assert(kEBlk == 4, "slot arithmetic");
    const cd* pl = X + (nw - 1) * es;  // plane of e = 0 at E - 1
    const cd* ph = X + (nw + 1) * es;
    cd lo[kEBlk], hi[kEBlk];
#pragma unroll
    for (int e = 1; e < kEBlk; ++e) lo[e] = ld(pl + e * es);
#pragma unroll
    for (int e = 0; e + 1 < kEBlk; ++e) hi[e] = ld(ph + e * es);
    ph += (kEBlk - 1) * es;
    auto step = [&](auto T) {
        constexpr int t = decltype(T)::value;
        lo[(0 - t) & 3] = ld(pl);
        hi[(3 + t) & 3] = ld(ph);
        cd l[kEBlk], h[kEBlk], Dl[3], Dh[3];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            Dl[i] = ld(sL + i);
            if constexpr (TWO) Dh[i] = ld(sH + i);
        }
#pragma unroll
        for (int e = 0; e < kEBlk; ++e) {
            l[e] = lo[(e - t) & 3];
            h[e] = hi[(e + t) & 3];
        }
        filter_step<TWO>(acc, l, h, Dl, Dh);
        pl -= es;
        ph += es;
        sL += 3;
        if constexpr (TWO) sH += 3;
    };
    int left = nw;
    for (; left >= 4; left -= 4) {
        step(std::integral_constant<int, 0>{});
        step(std::integral_constant<int, 1>{});
        step(std::integral_constant<int, 2>{});
        step(std::integral_constant<int, 3>{});
    }
    if (left > 0) step(std::integral_constant<int, 0>{});
    if (left > 1) step(std::integral_constant<int, 1>{});
    if (left > 2) step(std::integral_constant<int, 2>{});
}

// The same sums where a coefficient is not finite: a term outside the energy grid
// is left out instead of multiplied by a zero block, which would spread the
// coefficient to energies that have no term with it.
template <bool TWO>
__device__ __forceinline__ void filter_masked(cd (&acc)[3][kEBlk], const cd* X, int es, int nw, const cd* sL, const cd* sH,
                                              int e_first, int ne) {
    for (int w = 1; w <= nw; ++w, sL += 3, sH += 3) {
#pragma unroll
        for (int e = 0; e < kEBlk; ++e) {
            const int E = e_first + e;
            const bool l_ok = E - w >= 0 && E - w < ne, h_ok = E + w >= 0 && E + w < ne;
            const cd l = X[(nw + e - w) * es], h = X[(nw + e + w) * es];
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                if constexpr (TWO) {
                    if (l_ok) cacc(acc[i][e], sL[i], l);
                    if (h_ok) cacc(acc[i][e], sH[i], h);
                } else {
                    if (l_ok || h_ok) cacc(acc[i][e], sL[i], cd{l.re + h.re, l.im + h.im});
                }
            }
        }
    }
}

// Coefficients of one edge into LDS, [j][w][i] (nine per frequency): the transform
// over the phonon momenta at kt, or (DIRECT) those of momentum kt.  CONJ: conjugated
// (the adjoint).  SWAP: [i][w][j].  Sets *bad where one is not finite.
template <int THREADS, bool DIRECT, bool CONJ, bool SWAP = false>
__device__ __forceinline__ void stage_coeff(const double* __restrict__ D, const cd* tw, int nkz, int kt, int nw, int ne,
                                            int64_t edges, int64_t edge, cd* sD, int* bad, int tid) {
    for (int x = tid; x < nw * 9; x += THREADS) {
        const int w = x / 9, ij = x % 9;
        cd v;
        const int64_t o = ((int64_t)w * edges + edge) * 9 + ij, qst = (int64_t)nw * edges * 9;
        if constexpr (DIRECT)
            v = cload(D, o + kt * qst);
        else
            v = momentum_sum(nkz, kt, tw, [&](int q) { return cload(D, o + q * qst); });
        if (w + 1 >= ne) v = cd{0.0, 0.0};  // a frequency that no pair of energies differs by has no term
        if constexpr (CONJ) v.im = -v.im;
        if (!(fabs(v.re) <= 1.7976931348623157e308 && fabs(v.im) <= 1.7976931348623157e308)) *bad = 1;
        const int in = SWAP ? ij / 3 : ij % 3, out = SWAP ? ij % 3 : ij / 3;
        st(sD + (in * nw + w) * 3 + out, v);
    }
}

}  // namespace ks
}  // namespace sse
