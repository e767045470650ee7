// fp64 Sigma (Eq. 3) in the momentum transform (kspace.h), any shape.
//
// transform_kernel writes hat G, atom by atom, into the workspace (a slab of
// energies at a time where the workspace is smaller than G), then one workgroup per
// (atom, transformed momentum, tile of eb energies) sums hat Sigma.  Per edge and
// per chunk of rc rows of the neighbour's blocks:
//   load   rows r0 .. r0+rc of hat G[E, b] for the eb + 2 nw energies the tile meets;
//   for j in 0..2:
//     right  H_j = rows . grad_j H^H            (lane = a row)
//     filter U_i += sum_w D_ij[w] (H_j[E-w] + H_j[E+w])   (lane = an entry, 4 energies)
//   left   Sigma[E] += sum_i A_i[:, rows] . U_i  (lane = (energy, column), sums in registers)
// The rows of a block do not meet before the last step, so a chunk of them is all
// that LDS holds; U_i stays in registers through the three directions and takes
// the place of the rows in LDS for the last step.  inverse_kernel transforms the
// output back in place.
//
// SRC = kTrans transforms while it loads (Nkz loads per entry, the same sums): for a
// workspace without room.  The direct sum takes the sum over source momenta as it stands
// (a loop over k' around the steps, Nkz times the work): every product and sum
// is then one of Eq. 3's own, so integer-valued inputs give exact results.
// Small problems and Nkz = 1 run it.
//
// This header holds the kernel; Sigma and dG have a source file each, compiled side by side.
#pragma once

#include <algorithm>

#include "kspace.h"
#include "sse_kernels.h"

namespace sse {
namespace fwd {

constexpr int kThreads = 256, kWaves = kThreads / 64;
constexpr size_t kLdsMax = 160 * 1024;

struct Tile {
    int eb, rc;  // energies and rows of a workgroup's tile
    int ncb;     // passes of the products over norb columns
    ks::Div by_n, by_ncb, by_row[2];  // norb, ncb, entries of a chunk of rows (the last one may be shorter)
    int rows;    // complex entries of one row buffer
    int body;    // of both, or of U_i
    size_t lds;
};

inline Tile make_tile(const Dims& d, int eb, int rc, int cb, bool two, bool stored) {
    const int n = (int)d.norb, tail = n % rc ? n % rc : rc;
    Tile t{eb, rc, (n + cb - 1) / cb, ks::Div(n), ks::Div((n + cb - 1) / cb), {ks::Div(rc * n), ks::Div(tail * n)}, 0, 0, 0};
    const int64_t rows = (eb + 2 * d.nw) * rc * ks::row_len(n);
    const int64_t body = std::max(2 * rows, (int64_t)eb * 3 * rc * n);
    const int64_t all = body + (two ? 18 : 9) * d.nw + (stored ? 6 : 3) * n * n + 2 * d.nkz + 1;
    t.lds = all < (1 << 20) ? sizeof(cd) * (size_t)all : (size_t)1 << 30;
    t.rows = (int)std::min<int64_t>(rows, 1 << 28);
    t.body = (int)std::min<int64_t>(body, 1 << 28);
    return t;
}

// The dG part of the adjoint is the same operation on the edges into an atom b, with
// g = dL/dSigma of the edge's own atom in place of G, the factors A_j on the right and
// A_i^H on the left, and conj(D) (MODE = kAdjoint; with two tables the E - w terms take Dm)
constexpr int kHermitian = 0;  // right factor grad_j H^H
constexpr int kStored = 1;     // right factor given
constexpr int kAdjoint = 2;

// the edges of kAdjoint: in-edges of every atom in edge order, atoms in decreasing
// in-degree (a workgroup's time grows with it, so the longest start first)
struct InEdges {
    const int32_t *offset, *edges, *order;
};

// CB columns per pass of the products, MT passes of the left product per wave
// One tile: block x of a launch's part
template <int SRC, bool DIRECT, bool TWO, int MODE, int CB, int MT>
__device__ __forceinline__ void fwd_tile(int block, const Dims& d, const ks::Blocks& blocks, const double* __restrict__ Dp,
                                         const double* __restrict__ Dm, const double* __restrict__ A,
                                         const double* __restrict__ B, const int32_t* __restrict__ nbr, const InEdges& in,
                                         cd alpha, const Tile& tile, int e_lo, int e_hi, const ks::LaunchPart& part,
                                         const ks::Twiddles& table, int s_slots, double* __restrict__ S) {
    constexpr bool ADJ = MODE == kAdjoint;
    extern __shared__ __align__(16) double smem[];
    const int n = (int)d.norb, nkz = (int)d.nkz, nw = (int)d.nw, ne = (int)d.ne, nb = (int)d.nb;
    const int np = ks::row_len(n), eb = tile.eb;
    cd* sG = reinterpret_cast<cd*>(smem);  // rows of G [ew][r][np]
    cd* sX = sG + tile.rows;               // H_j, same layout
    cd* sU = sG;                           // U_i [e][i][r][c], after the last filter
    cd* sD = sG + tile.body;               // [j][w][i]
    cd* sDm = sD + 9 * nw;                 // (TWO)
    cd* sA = sD + (TWO ? 18 : 9) * nw;     // grad H of the edge [i][r][c]
    cd* sR = sA + (MODE == kStored ? 3 * n * n : 0);  // right factor
    cd* tw = sR + 3 * n * n;
    int* bad = reinterpret_cast<int*>(tw + 2 * nkz);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // the workgroups of an atom get ids on one XCD, the tiles of a momentum next to
    // each other: their windows of energies overlap
    const int ntile = (e_hi - e_lo + eb - 1) / eb;
    const int s = block >> 3;
    const int64_t pos = part.a0 + s / part.n * 8 + (block & 7);
    if (pos >= d.na) return;  // uniform, before any barrier
    const int64_t a = ADJ ? __builtin_amdgcn_readfirstlane(in.order[pos]) : pos;
    const int rem = part.first + s % part.n, kt = rem / ntile, e0 = e_lo + (rem - kt * ntile) * eb;
    const int e_n = e_hi - e0 < eb ? e_hi - e0 : eb;  // energies of this tile
    const int ewin = eb + 2 * nw;
    const int nn = n * n;
    const int64_t edges = d.na * d.nb;

    if constexpr (!DIRECT) ks::stage_twiddles(tw, table, nkz, tid, kThreads);
    // this thread's entries of the output tile: columns (e, c) number l and l + 64 of
    // pass t's 128, rows rr .. rr + CB - 1
    const int ncol = e_n * n, nrb = tile.ncb;
    const int tasks = (ncol + 127) / 128 * nrb;
    cd sum[MT][2][CB];
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int r = 0; r < CB; ++r) sum[t][0][r] = sum[t][1][r] = cd{0.0, 0.0};
    const int m_lo = ADJ ? __builtin_amdgcn_readfirstlane(in.offset[a]) : 0;
    const int m_hi = ADJ ? __builtin_amdgcn_readfirstlane(in.offset[a + 1]) : nb;
    for (int m = m_lo; m < m_hi; ++m) {
        const int64_t edge = ADJ ? (int64_t)__builtin_amdgcn_readfirstlane(in.edges[m]) : a * nb + m;
        const int64_t b = ADJ ? edge / nb : (int64_t)__builtin_amdgcn_readfirstlane(nbr[edge]);
        if (b < 0 || b >= d.na) continue;
        const ks::Source src = ks::source(blocks, b);
        for (int r0 = 0; r0 < n; r0 += tile.rc) {
            const int rc = n - r0 < tile.rc ? n - r0 : tile.rc;
            // filter lanes: entry el = (r, c) of the chunk, energies 4 eq .. 4 eq + 3
            const ks::Div by_row = tile.by_row[rc < tile.rc];
            const int nel = rc * n, eq = by_row.quot(tid), el = tid - eq * nel;
            const bool f_lane = eq * ks::kEBlk < eb;
            const int f_r = tile.by_n.quot(el);
            const int f_off = f_lane ? (eq * ks::kEBlk * rc + f_r) * np + el - f_r * n : 0;
            cd acc[3][ks::kEBlk];
#pragma unroll
            for (int i = 0; i < 3; ++i)
#pragma unroll
                for (int e = 0; e < ks::kEBlk; ++e) acc[i][e] = cd{0.0, 0.0};
            for (int kp = 0; kp < (DIRECT ? nkz : 1); ++kp) {
                const int kg = DIRECT ? kp : kt;  // momentum of the blocks
                const int q = ADJ ? kp - kt : kt - kp, kd = !DIRECT ? kt : q < 0 ? q + nkz : q;  // of the coefficients
                const bool coeff = DIRECT || r0 == 0;  // this step's coefficients are new ones
                __syncthreads();                       // the buffers of the step before are read
                if (coeff && tid == 0) *bad = 0;
                ks::load_rows<kThreads, SRC, false>(src, tw, nkz, kg, e0 - nw, ewin, r0, rc, n, by_row, tile.by_n, sG,
                                                    tid);
                if (r0 == 0 && kp == 0) {
                    ks::stage_factor<kThreads>(A, edge, nn, sA, tid);
                    if constexpr (MODE == kStored) ks::stage_factor<kThreads>(B, edge, nn, sR, tid);
                }
                if (coeff) {
                    __syncthreads();  // *bad is cleared
                    ks::stage_coeff<kThreads, DIRECT, ADJ>(Dp, tw, nkz, kd, nw, ne, edges, edge, sD, bad, tid);
                    if constexpr (TWO)
                        ks::stage_coeff<kThreads, DIRECT, ADJ>(Dm, tw, nkz, kd, nw, ne, edges, edge, sDm, bad, tid);
                }
                __syncthreads();
                const bool finite = *bad == 0;
                for (int j = 0; j < 3; ++j) {
                    ks::right_product<kWaves, 2, CB, MODE == kHermitian>(sG, sR + j * nn, ewin * rc, n, tile.ncb, tile.by_ncb,
                                                              (wave + j) % kWaves, lane, [&](int row) { return sX + row * np; });
                    __syncthreads();
                    if (f_lane) {
                        const cd* Dl = sD + 3 * j * nw;
                        const cd* Dh = (TWO ? sDm : sD) + 3 * j * nw;
                        if (finite)
                            ks::filter<TWO>(acc, sX + f_off, rc * np, nw, Dl, Dh);
                        else
                            ks::filter_masked<TWO>(acc, sX + f_off, rc * np, nw, Dl, Dh, e0 + eq * ks::kEBlk, ne);
                    }
                    __syncthreads();
                }
            }
            if (f_lane) {
#pragma unroll
                for (int e = 0; e < ks::kEBlk; ++e)
#pragma unroll
                    for (int i = 0; i < 3; ++i) ks::st(sU + ((eq * ks::kEBlk + e) * 3 + i) * nel + el, acc[i][e]);
            }
            __syncthreads();
#pragma unroll
            for (int ti = 0; ti < MT; ++ti) {
                const int t = wave + ti * kWaves;
                if (t >= tasks) continue;
                const int tc = tile.by_ncb.quot(t), col = tc * 128 + lane, rr = (t - tc * nrb) * CB;
                const int x0 = col < ncol ? col : 0, x1 = col + 64 < ncol ? col + 64 : 0;
                const int ea = tile.by_n.quot(x0), eb_ = tile.by_n.quot(x1);
                const int fr = rr + ks::uniform_entry<CB>(lane);
                const int fc = fr < n ? fr : n - 1, f_step = ADJ ? 2 * n : 2;
                const double* f = reinterpret_cast<const double*>(sA) + 2 * (ADJ ? r0 * n + fc : fc * n + r0) + (lane & 1);
                const cd* ua = sU + ea * 3 * nel + x0 - ea * n;
                const cd* ub = sU + eb_ * 3 * nel + x1 - eb_ * n;
                auto operand = [&](int k, cd (&x)[2]) {
                    x[0] = ks::ld(ua + k * n);
                    x[1] = ks::ld(ub + k * n);
                };
                if constexpr (ADJ) {
                    // each direction's sum by itself: one chain over an atom's whole in-degree rounds
                    // more than the terms it adds
                    for (int i = 0; i < 3; ++i) {
                        cd part[2][CB];
#pragma unroll
                        for (int r = 0; r < CB; ++r) part[0][r] = part[1][r] = cd{0.0, 0.0};
                        const double* fi = f + 2 * i * nn;
                        ks::uniform_product<2, CB, ADJ>(
                            part, rc, [&](int k) { return fi[k * f_step]; },
                            [&](int k, cd (&x)[2]) { operand(i * rc + k, x); });
#pragma unroll
                        for (int h = 0; h < 2; ++h)
#pragma unroll
                            for (int r = 0; r < CB; ++r) {
                                sum[ti][h][r].re += part[h][r].re;
                                sum[ti][h][r].im += part[h][r].im;
                            }
                    }
                } else {
                    ks::uniform_product<2, CB, ADJ>(
                        sum[ti], 3 * rc,
                        [&](int k) {
                            const int i = k >= 2 * rc ? 2 : k >= rc ? 1 : 0;
                            return f[2 * i * nn + (k - i * rc) * f_step];
                        },
                        operand);
                }
            }
        }
    }
    const int64_t s_est = d.na * s_slots * nn;
    double* So = S + 2 * (((int64_t)kt * ne + e0) * s_est + a * s_slots * nn);
    if (ADJ && s_slots > 1) {  // the slots that the forward map does not read
        const int rest = (s_slots - 1) * nn;
        for (int e = 0; e < e_n; ++e)
            for (int x = tid; x < rest; x += kThreads) cstore(So, e * s_est + nn + x, cd{0.0, 0.0});
    }
#pragma unroll
    for (int ti = 0; ti < MT; ++ti) {
        const int t = wave + ti * kWaves;
        if (t >= tasks) continue;
        const int tc = tile.by_ncb.quot(t), rr = (t - tc * nrb) * CB;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int col = tc * 128 + 64 * h + lane;
            if (col >= ncol) continue;
            const int e = tile.by_n.quot(col), c = col - e * n;
            double* o = So + 2 * (e * s_est + c);
#pragma unroll
            for (int r = 0; r < CB; ++r)
                if (rr + r < n) cstore(o, (rr + r) * n, DIRECT ? cmul(alpha, sum[ti][h][r]) : sum[ti][h][r]);
        }
    }
}

template <int SRC, bool DIRECT, bool TWO, int MODE, int CB, int MT>
__global__ __launch_bounds__(kThreads, 2) void fwd_kspace_kernel(Dims d, ks::Gate gate, ks::Blocks blocks,
                                                                 const double* __restrict__ Dp,
                                                                 const double* __restrict__ Dm,
                                                                 const double* __restrict__ A,
                                                                 const double* __restrict__ B,
                                                                 const int32_t* __restrict__ nbr, InEdges in, cd alpha,
                                                                 Tile tile, int e_lo, int e_hi, ks::LaunchPart part,
                                                                 ks::Twiddles table, int s_slots,
                                                                 double* __restrict__ S) {
    if (ks::shut<DIRECT>(gate)) return;
    auto run = [&](int block) {
        fwd_tile<SRC, DIRECT, TWO, MODE, CB, MT>(block, d, blocks, Dp, Dm, A, B, nbr, in, alpha, tile, e_lo, e_hi, part, table,
                                                 s_slots, S);
    };
    if constexpr (DIRECT) {
        for (unsigned block = blockIdx.x; block < part.groups; block += gridDim.x) {
            __syncthreads();  // the LDS of the tile before
            run((int)block);
        }
    } else {
        run((int)blockIdx.x);
    }
}

// The tile with the least time per energy under the quantisation of each step:
// cycles of the busiest wave, 16 per complex multiply-add, and the number of
// rounds of workgroups on the chip.
inline bool pick_tile(const Dims& d, bool two, bool stored, int cb, int mt, int cus, Tile* best, double* best_cost) {
    const int n = (int)d.norb;
    bool found = false;
    auto up = [](double a, double b) { return (double)(int64_t)((a + b - 1) / b); };
    for (int rc = 1; rc <= n; ++rc)
        for (int eb = ks::kEBlk; eb <= 128 && eb / ks::kEBlk * rc * n <= kThreads; eb += ks::kEBlk) {
            if (eb > ks::kEBlk && eb - ks::kEBlk >= d.ne) break;
            const Tile t = make_tile(d, eb, rc, cb, two, stored);
            if (t.lds > kLdsMax) break;
            const double win = eb + 2.0 * d.nw;
            const double passes = up((double)eb * n, 128) * t.ncb;
            if (passes > mt * kWaves) break;
            const int occ = t.lds <= kLdsMax / 2 ? 2 : 1;
            // per chunk of rows, in vector instructions of a workgroup: the busiest wave of each
            // product and the filter, weighted by a fit to eleven tiles at 10 and 12 orbitals (within 10%)
            const double right = 3 * kWaves * up(up(win * rc, 128) * t.ncb, kWaves) * (n * cb * 8.4 + 60);
            const double filt = kWaves * 3.0 * d.nw * ks::kEBlk * (two ? 24 : 14);
            const double left = passes * (3 * rc * cb * 8.4 + 70);
            const double chunk = 1.7 * (right + filt) + 1.25 * left + 5500;
            const double groups = up(up((double)d.ne, eb) * (double)(d.nkz * d.na), cus * occ);
            const double cost = groups * up(n, rc) * chunk * (occ == 2 ? 2 : 1.5);
            if (!found || cost < *best_cost) {
                *best_cost = cost;
                *best = t;
                found = true;
            }
        }
    return found;
}

// columns per pass: the number that divides norb with the least left over
inline void passes_of(int n, int* cb, int* mt) {
    const int c6 = (n + 5) / 6 * 6, c5 = (n + 4) / 5 * 5, c4 = (n + 3) / 4 * 4;
    *cb = c4 <= c5 && c4 <= c6 ? 4 : c5 <= c6 ? 5 : 6;
    *mt = 2;
}

template <int SRC, bool DIRECT, bool TWO, int MODE, int CB, int MT>
hipError_t launch_cb(const Dims& d, ks::Gate gate, const ks::Blocks& blocks, const double* Dp, const double* Dm, const double* A,
                            const double* B, const int32_t* nbr, InEdges in, cd alpha, const Tile& t, int e_lo, int e_hi,
                            int s_slots, double* S, hipStream_t stream) {
    auto kern = fwd_kspace_kernel<SRC, DIRECT, TWO, MODE, CB, MT>;
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)t.lds);
    if (e != hipSuccess) return e;
    const int64_t per = d.nkz * ((e_hi - e_lo + t.eb - 1) / t.eb);
    if (per > INT32_MAX) return hipErrorInvalidValue;
    ks::launch_parts(d.na, per, kThreads, [&](ks::LaunchPart part) {
        const unsigned groups = DIRECT && gate.word ? std::min(part.groups, ks::kGatedGroups) : part.groups;
        hipLaunchKernelGGL(kern, dim3(groups), dim3(kThreads), t.lds, stream, d, gate, blocks, Dp, Dm, A, B, nbr, in, alpha, t,
                           e_lo, e_hi, part, ks::twiddles(d.nkz), s_slots, S);
    });
    return hipGetLastError();
}

template <int SRC, bool DIRECT, bool TWO, int MODE, class... Args>
hipError_t launch_shape(int cb, Args... args) {
    if (cb == 4) return launch_cb<SRC, DIRECT, TWO, MODE, 4, 2>(args...);
    if (cb == 5) return launch_cb<SRC, DIRECT, TWO, MODE, 5, 2>(args...);
    return launch_cb<SRC, DIRECT, TWO, MODE, 6, 2>(args...);
}

template <int SRC, bool DIRECT, int MODE, class... Args>
hipError_t launch_tables(bool two, int cb, Args... args) {
    return two ? launch_shape<SRC, DIRECT, true, MODE>(cb, args...) : launch_shape<SRC, DIRECT, false, MODE>(cb, args...);
}

template <int SRC>
using kFrom = std::integral_constant<int, SRC>;

// the tile for these dims on the current device
inline hipError_t choose_tile(const Dims& d, bool two, bool stored, int* cb, Tile* t) {
    int dev = 0, cus = 0, mt = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return e;
    passes_of((int)d.norb, cb, &mt);
    double cost = 0.0;
    return pick_tile(d, two, stored, *cb, mt, cus, t, &cost) ? hipSuccess : hipErrorInvalidValue;
}

}  // namespace fwd
}  // namespace sse
