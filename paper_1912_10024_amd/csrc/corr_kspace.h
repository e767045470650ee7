// fp64 correlations over energy in the momentum transform (kspace.h), any shape:
// the phonon self-energy (Eq. 4) and the D gradient of Eq. 3.
//
//   dD_ij[q, w]  = conj(alpha) sum_{k, E, +-} sum_rc conj((A_i B[k, E] A_j^H)[r][c]) g[k+q, E +- w][r][c]
//                = conj(alpha) sum_{k, E, +-} < X_i[k, E], Y_j[k+q, E +- w] >,   X_i = A_i B,  Y_j = g A_j
// over the entries of a block, with B the neighbour's block of G; the sum over k is a
// correlation, so in the transform hat dD[m, w] needs hat X[m] and hat Y[m] only:
// Nkz times fewer products than the sum over (q, k), and 6 block products per (edge,
// momentum, energy) instead of 12.  Pi_ij is the same sum over the upper branch with
// g = Gs and B = Go^H: tr(A_i^H Gs A_j Go) = < A_i Go^H, Gs A_j >.
//
// One workgroup per (edge, transformed momentum), sweeping the energies in tiles of
// eb, for one chunk of rc rows of the blocks after another:
//   load   rows of g of the energies that enter the window, all of B of the tile's energies
//   right  Y_j rows                                        (lane = a row)
//   left   X_i rows                                        (lane = (energy, column))
//   sums   acc[i][w] += conj(X_i[E]) Y_j[E +- w]           (lane = an entry, one j, WB
//          frequencies, a share of the energies)
// A lane's window of WB energies per branch slides with E through registers, so a
// step reads 3 + 1 (or 2) entries from LDS for 12 WB multiply-adds.  The planes
// of Y that the next tile still needs move to the front of the buffer.  The lanes'
// sums are added in LDS in a fixed order at the end.
//
// YSRC, XSRC = kTrans transform g and B while they load; the direct sum takes k as it stands,
// one workgroup per (edge, q) (exact for integer-valued inputs, Nkz times the work).
//
// This header holds the kernel; Pi and dD have a source file each, compiled side by side.
#pragma once

#include <algorithm>

#include "kspace.h"
#include "sse_kernels.h"

namespace sse {
namespace corr {

constexpr int kThreads = ks::kCorrThreads, kWaves = kThreads / 64;
constexpr int kCB = ks::kCorrCB, kXB = ks::kCorrXB;
using ks::corr_tile;
using ks::CorrTile;

struct CorrArgs {
    ks::Blocks y, x;  // g (or Gs) and B (or Go), or their transforms
    int lo, hi;       // energies of X that are summed
    bool add;         // add to the output instead of writing it
};

// HI, LO: the branches; CT: B is the conjugate transpose of the array's blocks
// One (edge, momentum, group of frequencies): block x of a launch's part
template <int YSRC, int XSRC, bool DIRECT, bool HI, bool LO, bool CT, int WB>
__device__ __forceinline__ void corr_block(int block, const Dims& d, bool marks, const CorrArgs& g, const double* __restrict__ A,
                                           const int32_t* __restrict__ nbr, cd scale, const CorrTile& t,
                                           const ks::LaunchPart& part, const ks::Twiddles& table, double* __restrict__ out) {
    extern __shared__ __align__(16) double smem[];
    const int n = (int)d.norb, nkz = (int)d.nkz, nw = (int)d.nw, ne = (int)d.ne, nb = (int)d.nb;
    const int nn = n * n, np = ks::row_len(n), eb = t.eb;
    cd* sY = reinterpret_cast<cd*>(smem);  // [plane][j][r][c], plane 0 at energy e0 - halo_lo
    cd* sX = sY + t.y_entries;             // [e][i][r][c]
    cd* sG = sX + t.x_entries;             // rows of g [e][r][np]
    cd* sB = sG + t.g_entries;             // B [e][t][np]
    cd* sA = sB + eb * n * np;             // grad H of the edge
    cd* tw = sA + 3 * nn;
    int* bad = reinterpret_cast<int*>(tw + 2 * nkz);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // the workgroups of an atom on one XCD: they read the same blocks of g
    const int s = block >> 3;
    const int64_t a = part.a0 + s / part.n * 8 + (block & 7);
    if (a >= d.na) return;  // uniform, before any barrier
    int rem = part.first + s % part.n;
    const int wg = rem % t.nwg;
    rem /= t.nwg;
    const int m = rem / nkz, kt = rem % nkz;
    const int64_t edge = a * nb + m, edges = d.na * nb;
    const int32_t b = __builtin_amdgcn_readfirstlane(nbr[edge]);
    const bool valid = b >= 0 && b < d.na;
    // an edge marked for the direct kernel (uniform, and only this workgroup writes the entry)
    if (marks && ks::marked(out, (((int64_t)kt * nw + wg * t.nwb * WB) * edges + edge) * 9) != DIRECT) return;

    const ks::CorrLane own = ks::corr_lane(t, tid, wg);
    const int el = own.el, j = own.j, es = own.es, w0 = own.w0;
    cd acc[3][WB];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int u = 0; u < WB; ++u) acc[i][u] = cd{0.0, 0.0};

    if (valid) {
        if constexpr (YSRC == ks::kTrans || XSRC == ks::kTrans) ks::stage_twiddles(tw, table, nkz, tid, kThreads);
        if (tid == 0) *bad = 0;
        ks::stage_factor<kThreads>(A, edge, nn, sA, tid);
        const ks::Source ys = ks::source(g.y, a);
        const ks::Source xs = ks::source(g.x, b);
        for (int kp = 0; kp < (DIRECT ? nkz : 1); ++kp) {
            const int ky = DIRECT ? (kp + kt) % nkz : kt;
            const int kx = DIRECT ? kp : CT ? (nkz - kt) % nkz : kt;
            for (int r0 = 0; r0 < n; r0 += t.rc) {
                const int rc = n - r0 < t.rc ? n - r0 : t.rc, last = rc < t.rc;
                const int nel = rc * n, ps = 3 * nel;  // entries of a plane
                auto load = [&](int energy, int count) {
                    ks::load_rows<kThreads, YSRC, false>(ys, tw, nkz, ky, energy, count, r0, rc, n, t.by_row[last], t.by_n,
                                                         sG, tid);
                };
                // Y of the loaded rows of `count` energies into the planes from `plane` on; the first
                // task goes to wave `from`
                auto right = [&](int plane, int count, int from) {
                    const int rows = count * rc;
                    for (int jj = 0; jj < 3; ++jj) {
                        auto dst = [&](int row) {
                            const int ew = t.by_rc[last].quot(row);
                            return sY + (plane + ew) * ps + jj * nel + (row - ew * rc) * n;
                        };
                        const int w = ks::first_task<kWaves>(wave, from + jj * t.ncb);
                        if (rows <= 64)
                            ks::right_product<kWaves, 1, kCB, false>(sG, sA + jj * nn, rows, n, t.ncb, t.by_ncb, w, lane, dst);
                        else
                            ks::right_product<kWaves, 2, kCB, false>(sG, sA + jj * nn, rows, n, t.ncb, t.by_ncb, w, lane, dst);
                    }
                };
                for (int p = 0; p < t.halo_lo + t.halo_hi; p += eb) {
                    const int left = t.halo_lo + t.halo_hi - p, count = left < eb ? left : eb;
                    __syncthreads();
                    load(g.lo - t.halo_lo + p, count);
                    __syncthreads();
                    right(p, count, 0);
                }
                ks::RowsAhead<kThreads, 2, YSRC, false> y_next;
                ks::RowsAhead<kThreads, 4, XSRC, CT> x_next;
                auto ask = [&](int e0) {
                    const int e_n = g.hi - e0 < eb ? g.hi - e0 : eb;
                    y_next.ask(ys, tw, nkz, ky, e0 + t.halo_hi, eb, r0, rc, n, t.by_row[last], t.by_n, tid);
                    x_next.ask(xs, tw, nkz, kx, e0, e_n, 0, n, n, t.by_nn, t.by_n, tid);
                };
                ask(g.lo);
                for (int e0 = g.lo; e0 < g.hi; e0 += eb) {
                    const int e_n = g.hi - e0 < eb ? g.hi - e0 : eb;
                    __syncthreads();
                    y_next.put(ys, tw, nkz, ky, e0 + t.halo_hi, eb, r0, rc, n, t.by_row[last], t.by_n, sG, tid);
                    x_next.put(xs, tw, nkz, kx, e0, e_n, 0, n, n, t.by_nn, t.by_n, sB, tid);
                    __syncthreads();
                    // X_i[e][r][c] = sum_t A_i[r0 + r][t] B[e][t][c]; two columns (e, c) per lane
                    const int ncol = e_n * n, nout = 3 * rc, nob = (nout + kXB - 1) / kXB;
                    const int tasks = (ncol + 127) / 128 * nob;
                    for (int task = wave; task < tasks; task += kWaves) {
                        const int tc = t.by_xb[last].quot(task), o0 = (task - tc * nob) * kXB;
                        const cd* p[2];
                        int col[2], e[2];
#pragma unroll
                        for (int h = 0; h < 2; ++h) {
                            col[h] = tc * 128 + 64 * h + lane;
                            const int x = col[h] < ncol ? col[h] : 0;
                            e[h] = t.by_n.quot(x);
                            p[h] = sB + e[h] * n * np + x - e[h] * n;
                        }
                        cd v[2][kXB];
#pragma unroll
                        for (int o = 0; o < kXB; ++o) v[0][o] = v[1][o] = cd{0.0, 0.0};
                        const int fo = o0 + ks::uniform_entry<kXB>(lane), oo = fo < nout ? fo : nout - 1;
                        const int fi = oo >= 2 * rc ? 2 : oo >= rc ? 1 : 0;
                        const double* f = reinterpret_cast<const double*>(sA) + 2 * (fi * nn + (r0 + oo - fi * rc) * n) + (lane & 1);
                        ks::uniform_product<2, kXB, false>(v, n, [&](int q) { return f[2 * q]; }, [&](int q, cd (&x)[2]) {
                            x[0] = ks::ld(p[0] + q * np);
                            x[1] = ks::ld(p[1] + q * np);
                        });
#pragma unroll
                        for (int h = 0; h < 2; ++h) {
                            if (col[h] >= ncol) continue;
                            cd* dst = sX + e[h] * ps + col[h] - e[h] * n;
                            bool fin = true;
#pragma unroll
                            for (int o = 0; o < kXB; ++o) {
                                if (o0 + o >= nout) continue;
                                ks::st(dst + (o0 + o) * n, v[h][o]);
                                fin = fin && fabs(v[h][o].re) <= 1.7976931348623157e308 && fabs(v[h][o].im) <= 1.7976931348623157e308;
                            }
                            if (!fin) *bad = 1;
                        }
                    }
                    right(t.halo_lo + t.halo_hi, eb, tasks % kWaves);
                    __syncthreads();
                    // on its way while the sums run (after the last tile: that one again, so that the
                    // registers are dead in between)
                    ask(e0 + eb < g.hi ? e0 + eb : e0);
                    __builtin_amdgcn_sched_barrier(0);
                    const int share = eb / t.es, cnt = ks::corr_energies(t, own, nw, nel, e_n);
                    const cd* X = sX + es * share * ps + el;
                    const cd* Yc = sY + (es * share + t.halo_lo) * ps + j * nel + el;  // plane of the first energy
                    if (*bad == 0) {
                        const cd* ph = Yc + (w0 + 1) * ps;
                        const cd* pl = Yc - (w0 + 1) * ps;
                        cd hi[WB], lo[WB];
                        if (cnt > 0) {
                            if constexpr (HI) {
#pragma unroll
                                for (int u = 0; u + 1 < WB; ++u) hi[u] = ks::ld(ph + u * ps);
                            }
                            if constexpr (LO) {
#pragma unroll
                                for (int u = 1; u < WB; ++u) lo[(WB - u) % WB] = ks::ld(pl - u * ps);
                            }
                        }
                        ph += (WB - 1) * ps;
                        auto step = [&](auto S) {
                            constexpr int st = decltype(S)::value;
                            if constexpr (HI) hi[(st + WB - 1) % WB] = ks::ld(ph);
                            if constexpr (LO) lo[st % WB] = ks::ld(pl);
                            cd x[3];
#pragma unroll
                            for (int i = 0; i < 3; ++i) x[i] = ks::ld(X + i * nel);
#pragma unroll
                            for (int u = 0; u < WB; ++u) {
                                cd y;
                                if constexpr (HI && LO) {
                                    const cd h = hi[(st + u) % WB], l = lo[(st + WB - u) % WB];
                                    y = cd{h.re + l.re, h.im + l.im};
                                } else if constexpr (HI) {
                                    y = hi[(st + u) % WB];
                                } else {
                                    y = lo[(st + WB - u) % WB];
                                }
#pragma unroll
                                for (int i = 0; i < 3; ++i) cfma_conja(acc[i][u], x[i], y);
                            }
                            X += ps;
                            ph += ps;
                            pl += ps;
                        };
                        int left = cnt;
                        for (; left >= WB; left -= WB) {
                            step(std::integral_constant<int, 0>{});
                            if constexpr (WB > 1) step(std::integral_constant<int, 1>{});
                            if constexpr (WB > 2) step(std::integral_constant<int, 2>{});
                            if constexpr (WB > 3) step(std::integral_constant<int, 3>{});
                            if constexpr (WB > 4) step(std::integral_constant<int, 4>{});
                        }
                        if (left > 0) step(std::integral_constant<int, 0>{});
                        if constexpr (WB > 2)
                            if (left > 1) step(std::integral_constant<int, 1>{});
                        if constexpr (WB > 3)
                            if (left > 2) step(std::integral_constant<int, 2>{});
                        if constexpr (WB > 4)
                            if (left > 3) step(std::integral_constant<int, 3>{});
                    } else {
                        // a term outside the grid is left out instead of multiplied by a zero block
                        for (int e = 0; e < cnt; ++e) {
                            const int E = e0 + es * share + e;
#pragma unroll
                            for (int u = 0; u < WB; ++u) {
                                const int w = w0 + 1 + u;
                                if (w > nw) continue;
#pragma unroll
                                for (int i = 0; i < 3; ++i) {
                                    const cd x = ks::ld(X + e * ps + i * nel);
                                    if (HI && E + w < ne) cfma_conja(acc[i][u], x, ks::ld(Yc + (e + w) * ps));
                                    if (LO && E - w >= 0) cfma_conja(acc[i][u], x, ks::ld(Yc + (e - w) * ps));
                                }
                            }
                        }
                    }
                    // the planes that the next tile's window keeps
                    const int keep = (t.halo_lo + t.halo_hi) * ps, from = eb * ps;
                    for (int x0 = 0; x0 < keep; x0 += 4 * kThreads) {
                        cd v[4];
                        __syncthreads();
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            const int x = x0 + u * kThreads + tid;
                            if (x < keep) v[u] = ks::ld(sY + from + x);
                        }
                        __syncthreads();
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            const int x = x0 + u * kThreads + tid;
                            if (x < keep) ks::st(sY + x, v[u]);
                        }
                    }
                }
            }
        }
    }
    // the lanes' sums, one direction i at a time, in the order of (share, entry)
    cd* red = sY;
    const int outs = 3 * t.nwb * WB;
    for (int i = 0; i < 3; ++i) {
        __syncthreads();
#pragma unroll
        for (int u = 0; u < WB; ++u) ks::st(red + u * kThreads + tid, i == 0 ? acc[0][u] : i == 1 ? acc[1][u] : acc[2][u]);
        __syncthreads();
        // eight lanes per output: every eighth entry each, then a tree over the eight
        for (int o0 = 0; o0 < outs; o0 += kThreads / 8) {
            const int o = o0 + tid / 8, oo = o < outs ? o : 0;
            const int u = oo % WB, wo = oo / WB % t.nwb, jo = oo / WB / t.nwb;
            const int w = (wg * t.nwb + wo) * WB + u;
            cd sum{0.0, 0.0};
            for (int se = 0; se < t.es; ++se) {
                const cd* p = red + u * kThreads + ((se * 3 + jo) * t.nwb + wo) * t.nel;
                for (int x = tid & 7; x < t.nel; x += 8) {
                    const cd v = ks::ld(p + x);
                    sum.re += v.re;
                    sum.im += v.im;
                }
            }
#pragma unroll
            for (int h = 4; h > 0; h >>= 1) {
                sum.re += __shfl_down(sum.re, h, 8);
                sum.im += __shfl_down(sum.im, h, 8);
            }
            if (o >= outs || w >= nw || (tid & 7)) continue;
            const int64_t at = (((int64_t)kt * nw + w) * edges + edge) * 9 + i * 3 + jo;
            if (DIRECT) sum = cmul(scale, sum);
            if (g.add) {
                const cd old = cload(out, at);
                sum = cd{old.re + sum.re, old.im + sum.im};
            }
            cstore(out, at, sum);
        }
    }
}

template <int YSRC, int XSRC, bool DIRECT, bool HI, bool LO, bool CT, int WB>
__global__ __launch_bounds__(kThreads) void corr_kspace_kernel(Dims d, ks::Gate gate, bool marks, CorrArgs g,
                                                               const double* __restrict__ A, const int32_t* __restrict__ nbr,
                                                               cd scale, CorrTile t, ks::LaunchPart part, ks::Twiddles table,
                                                               double* __restrict__ out) {
    if (ks::shut<DIRECT>(gate)) return;
    auto run = [&](int block) {
        corr_block<YSRC, XSRC, DIRECT, HI, LO, CT, WB>(block, d, marks, g, A, nbr, scale, t, part, table, out);
    };
    if constexpr (DIRECT) {
        for (unsigned block = blockIdx.x; block < part.groups; block += gridDim.x) {
            __syncthreads();  // the LDS of the block before
            run((int)block);
        }
    } else {
        run((int)blockIdx.x);
    }
}

template <int YSRC, int XSRC, bool DIRECT, bool HI, bool LO, bool CT, int WB>
hipError_t launch_corr_wb(const Dims& d, ks::Gate gate, bool marks, const CorrArgs& g, const double* A, const int32_t* nbr, cd scale,
                                 const CorrTile& t, double* out, hipStream_t stream) {
    auto kern = corr_kspace_kernel<YSRC, XSRC, DIRECT, HI, LO, CT, WB>;
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)t.lds);
    if (e != hipSuccess) return e;
    const int64_t per = d.nb * d.nkz * t.nwg;
    if (per > INT32_MAX) return hipErrorInvalidValue;
    ks::launch_parts(d.na, per, kThreads, [&](ks::LaunchPart part) {
        const unsigned groups = DIRECT && (gate.word || marks) ? std::min(part.groups, ks::kGatedGroups) : part.groups;
        hipLaunchKernelGGL(kern, dim3(groups), dim3(kThreads), t.lds, stream, d, gate, marks, g, A, nbr, scale, t, part,
                           ks::twiddles(d.nkz), out);
    });
    return hipGetLastError();
}

template <int YSRC, int XSRC, bool DIRECT, bool HI, bool LO, bool CT, class... Args>
hipError_t launch_corr_shape(int wb, Args... args) {
    switch (wb) {
        case 2: return launch_corr_wb<YSRC, XSRC, DIRECT, HI, LO, CT, 2>(args...);
        case 3: return launch_corr_wb<YSRC, XSRC, DIRECT, HI, LO, CT, 3>(args...);
        case 4: return launch_corr_wb<YSRC, XSRC, DIRECT, HI, LO, CT, 4>(args...);
    }
    if constexpr (!(HI && LO)) return launch_corr_wb<YSRC, XSRC, DIRECT, HI, LO, CT, 5>(args...);  // corr_max_wb
    return hipErrorInvalidValue;
}

}  // namespace corr
}  // namespace sse
