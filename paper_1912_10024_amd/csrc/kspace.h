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
// grad H entry, read through the scalar cache into scalar registers, or a
// coefficient, broadcast from LDS), so a lane needs one LDS read for 12 to 24
// multiply-adds, nothing is padded to a tile, and every size takes the same code.
#pragma once

#include <type_traits>

#include "sse_common.h"

namespace sse {
namespace ks {

constexpr int kEBlk = 4;  // energies of one lane in the filter
constexpr int kWaitLgkm = 0xc07f;  // s_waitcnt lgkmcnt(0), the other counters as they are

// memory that no kernel in flight writes, read at a uniform address: the constant
// address space makes the compiler use the scalar cache
typedef const double __attribute__((address_space(4)))* uptr;
__device__ __forceinline__ uptr uniform_ptr(const double* p) { return (uptr)(uintptr_t)p; }

// one complex entry of an LDS array (16-byte aligned)
__device__ __forceinline__ cd ld(const cd* p) {
    const double2 v = *reinterpret_cast<const double2*>(p);
    return cd{v.x, v.y};
}
__device__ __forceinline__ void st(cd* p, cd v) { *reinterpret_cast<double2*>(p) = make_double2(v.re, v.im); }

// x / d for 0 <= x < 2^16, 1 <= d < 2^16, with the reciprocal taken on the host
struct Div {
    uint32_t m, one;  // one: d == 1
    __host__ __device__ Div() : m(0), one(0) {}
    __host__ explicit Div(int d) : m(d == 1 ? 0u : (uint32_t)(0xffffffffu / (uint32_t)d) + 1u), one(d == 1 ? 0xffffffffu : 0u) {}
    __device__ __forceinline__ int quot(int x) const { return (int)(__umulhi((uint32_t)x, m) | ((uint32_t)x & one)); }
};

// LDS row of norb complex entries: an odd number of 16-byte entries, so that
// lanes that read down a column hit distinct banks
__host__ __device__ __forceinline__ int row_len(int n) { return n | 1; }

// exp(-2 pi i m / nkz), m = 0 .. nkz-1
__device__ __forceinline__ void stage_twiddles(cd* tw, int nkz, int tid, int threads) {
    for (int m = tid; m < nkz; m += threads) {
        double s, c;
        sincospi(2.0 * (double)m / (double)nkz, &s, &c);
        st(tw + m, cd{c, -s});
    }
}

// Where a tile of energies x rows of a source block array is loaded from
struct Source {
    const double* p;   // block of the wanted atom at momentum 0, energy 0
    int64_t kst, est;  // complex elements between momenta and energies
};
constexpr int kDirect = 0;  // blocks of one momentum as they are, from an array or from its transform
constexpr int kTrans = 1;   // transformed over the momenta while they are loaded

// Rows r0 .. r0+rc-1 of the source blocks of energies e_first .. e_first+new_-1 into
// LDS, entry (ew, r, u) of [ew][rc][row_len].  CT: of the conjugate transpose of
// every block (whose transform at m is that of the block at -m, conjugate transposed:
// kt = -m).  Energies outside the grid give zeros.  U entries per thread are
// loaded together, which is what hides the latency.
template <int THREADS, int SRC, bool CT>
__device__ __forceinline__ void load_rows(const Source& s, const cd* tw, int nkz, int kt, int e_first, int new_, int ne,
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
            const int e = e_first + ew;
            ok[u] = e >= 0 && e < ne;
            dst[u] = x < total ? (ew * rc + r) * np + c : -1;
            p[u] = base + 2 * ((ok[u] ? e : 0) * s.est + (CT ? c * n + r0 + r : r0 * n + rem));
            acc[u] = cd{0.0, 0.0};
        }
        if constexpr (SRC == kTrans) {
            int m = 0;  // k * kt mod nkz
#pragma unroll 4
            for (int k = 0; k < nkz; ++k) {
                const cd t = ld(tw + m);
#pragma unroll
                for (int u = 0; u < U; ++u) cfma(acc[u], cload(p[u], k * s.kst), t);
                m += kt;
                m -= m >= nkz ? nkz : 0;
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

// acc[r][c] += x_r(k) * f_c(k) (CONJ: conj(f)) for k in [0, len): R operands per
// lane from LDS, CB of them uniform from memory.  The operands of step k + 1 are on
// their way while step k multiplies (4 R CB multiply-adds per lane): scalar loads
// return out of order, so a wave can only wait for all of them, and without this
// every step paid the scalar cache's latency.
// at(k, x, f): addresses of step k's operands; off[c]: doubles between the uniform ones.
template <int R, int CB, bool CONJ, class At>
__device__ __forceinline__ void uniform_product(cd (&acc)[R][CB], int len, const int (&off)[CB], At at) {
    cd x[2][R], f[2][CB];
    auto fetch = [&](int buf, int k) {
        const cd* p[R];
        uptr u;
        at(k < len ? k : len - 1, p, u);
        __builtin_amdgcn_s_waitcnt(kWaitLgkm);  // the other buffer has arrived, before more is asked for
#pragma unroll
        for (int c = 0; c < CB; ++c) f[buf][c] = cd{u[off[c]], u[off[c] + 1]};
#pragma unroll
        for (int r = 0; r < R; ++r) x[buf][r] = ld(p[r]);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto mul = [&](int buf) {
#pragma unroll
        for (int c = 0; c < CB; ++c)
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if constexpr (CONJ)
                    cfma_conj(acc[r][c], x[buf][r], f[buf][c]);
                else
                    cfma(acc[r][c], x[buf][r], f[buf][c]);
            }
        __builtin_amdgcn_sched_barrier(0);
    };
    fetch(0, 0);
    int k = 0;
    for (; k + 2 <= len; k += 2) {
        fetch(1, k + 1);
        mul(0);
        fetch(0, k + 2);
        mul(1);
    }
    if (k < len) mul(0);
}

// out(row)[c] = sum_u sG[row][u] . f(u, c) for `rows` rows: a lane owns R rows, 64
// apart, of a group of 64 R, CB columns at a time.  RT: f(u, c) = conj(M[c][u]) (the
// right factor grad_j H^H), else f(u, c) = M[u][c].
template <int WAVES, int R, int CB, bool RT, class Out>
__device__ __forceinline__ void right_product(const cd* sG, uptr M, int rows, int n, int ncb, Div by_ncb, int first,
                                              int lane, Out out) {
    const int np = row_len(n);
    const int tasks = (rows + 64 * R - 1) / (64 * R) * ncb;
    for (int t = first; t < tasks; t += WAVES) {
        const int tr = by_ncb.quot(t), c0 = (t - tr * ncb) * CB;
        const int row = tr * 64 * R + lane;
        const cd* g[R];
        cd acc[R][CB];
        int off[CB];
#pragma unroll
        for (int r = 0; r < R; ++r) g[r] = sG + (row + 64 * r < rows ? row + 64 * r : 0) * np;
#pragma unroll
        for (int c = 0; c < CB; ++c) {
#pragma unroll
            for (int r = 0; r < R; ++r) acc[r][c] = cd{0.0, 0.0};
            const int cc = c0 + c < n ? c0 + c : n - 1;
            off[c] = 2 * (RT ? cc * n : cc);
        }
        const int step = RT ? 2 : 2 * n;
        uniform_product<R, CB, RT>(acc, n, off, [&](int u, const cd* (&p)[R], uptr& f) {
#pragma unroll
            for (int r = 0; r < R; ++r) p[r] = g[r] + u;
            f = M + u * step;
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
// over the phonon momenta at kt (TRANS) or those of momentum kt.  CONJ: conjugated
// (the adjoint).  Sets *bad where one is not finite.
template <int THREADS, bool TRANS, bool CONJ>
__device__ __forceinline__ void stage_coeff(const double* __restrict__ D, const cd* tw, int nkz, int kt, int nw, int ne,
                                            int64_t edges, int64_t edge, cd* sD, int* bad, int tid) {
    for (int x = tid; x < nw * 9; x += THREADS) {
        const int w = x / 9, ij = x % 9;
        cd v{0.0, 0.0};
        const int64_t o = ((int64_t)w * edges + edge) * 9 + ij, qst = (int64_t)nw * edges * 9;
        if constexpr (TRANS) {
            int m = 0;
#pragma unroll 4
            for (int q = 0; q < nkz; ++q) {
                cfma(v, cload(D, o + q * qst), ld(tw + m));
                m += kt;
                m -= m >= nkz ? nkz : 0;
            }
        } else {
            v = cload(D, o + kt * qst);
        }
        if (w + 1 >= ne) v = cd{0.0, 0.0};  // a frequency that no pair of energies differs by has no term
        if constexpr (CONJ) v.im = -v.im;
        if (!(fabs(v.re) <= 1.7976931348623157e308 && fabs(v.im) <= 1.7976931348623157e308)) *bad = 1;
        st(sD + ((ij % 3) * nw + w) * 3 + ij / 3, v);
    }
}

}  // namespace ks
}  // namespace sse
