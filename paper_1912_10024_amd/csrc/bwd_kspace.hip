// d gradH of the adjoint of Eq. 3 in the momentum transform (kspace.h), any shape.
//
// With g = dL/dSigma and B the neighbour's block of G, both transformed,
//   d gradH_i = conj(alpha) / Nkz sum_{m, E} U_i B^H,     U_i = sum_{j, w} conj(D_ij) (g A_j at E +- w)
//             + alpha / Nkz sum_{m, E} V_i B,             V_i = sum_{j, w} D_ji (g^H A_j at E +- w)
// The second line is the first one with g^H, B^H and D_ji(-m) in place of g, B and
// conj(D_ij(m)), so one piece of code runs twice.  Per pass, momentum and tile of eb
// energies, for one chunk of rc rows of the result:
//   rows of g, right product with A_j, filter over the frequencies: as in fwd_kspace_kernel
//   sums over (energy, column) of U_i[r][c] conj(B[t][c]): a contraction with 3 rc rows, 2 norb
//   columns and eb * 2 norb terms, on the fp64 matrix cores (16x16x4), the energies
//   dealt to the waves, whose sums are added in LDS at the end of a pass
// One workgroup per (edge, share): a share is all momenta of 32 energies or all energies of a
// momentum, as the workspace holds them; bwd_dh_reduce_kernel adds them in order.
#include <algorithm>

#include "kspace.h"
#include "sse_kernels.h"

namespace sse {

namespace {

constexpr int kThreads = 256, kWaves = kThreads / 64, kCB = 5;
constexpr int kNT = 4;  // column tiles: 2 norb <= 64
constexpr size_t kLdsMax = 160 * 1024;

typedef double f64x4 __attribute__((ext_vector_type(4)));

struct DhTile {
    int eb, rc, ncb;
    ks::Div by_n, by_ncb, by_row[2], by_nn;
    int rows, u_entries, body;
    size_t lds;
};

struct DhArgs {
    ks::Blocks g, G;  // dSigma and G, or their transforms
    bool by_energy;
};

}  // namespace

// One (edge, share): block x of a launch's part
template <int GSRC, int BSRC, bool DIRECT, bool TWO>
__device__ __forceinline__ void dh_block(int block, const Dims& d, const DhArgs& p, const double* __restrict__ Dp,
                                         const double* __restrict__ Dm, const double* __restrict__ A,
                                         const int32_t* __restrict__ nbr, cd alpha, const DhTile& t, int nshare,
                                         const ks::LaunchPart& part, const ks::Twiddles& table, double* __restrict__ out) {
    extern __shared__ __align__(16) double smem[];
    const int n = (int)d.norb, nkz = (int)d.nkz, nw = (int)d.nw, ne = (int)d.ne, nb = (int)d.nb;
    const int nn = n * n, np = ks::row_len(n), eb = t.eb;
    cd* sG = reinterpret_cast<cd*>(smem);  // rows of g [ew][r][np]
    cd* sX = sG + t.rows;                  // g A_j, same layout
    cd* sU = sG;                           // U_i [e][i][r][c]
    cd* sB = sG + t.u_entries;             // B [e][t][np], after the last filter
    cd* sD = sG + t.body;                  // [j][w][i]
    cd* sDm = sD + 9 * nw;                 // (TWO)
    cd* sO = sD + (TWO ? 18 : 9) * nw;     // the chunk's result
    cd* sA = sO + 3 * t.rc * n;            // grad H of the edge
    cd* tw = sA + 3 * nn;
    int* bad = reinterpret_cast<int*>(tw + 2 * nkz);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // the workgroups of an atom on one XCD
    const int s = block >> 3;
    const int64_t a = part.a0 + s / part.n * 8 + (block & 7);
    if (a >= d.na) return;  // uniform, before any barrier
    const int rem = part.first + s % part.n, share = rem % nshare;
    const int64_t edge = a * nb + rem / nshare, edges = d.na * nb;
    const int32_t b = __builtin_amdgcn_readfirstlane(nbr[edge]);
    if (b < 0 || b >= d.na) return;  // the reduction writes zero
    const int m_lo = p.by_energy ? 0 : share, m_hi = p.by_energy ? nkz : share + 1;
    const int e_lo = p.by_energy ? 32 * share : 0, e_hi = p.by_energy ? (e_lo + 32 < ne ? e_lo + 32 : ne) : ne;
    if constexpr (!DIRECT) ks::stage_twiddles(tw, table, nkz, tid, kThreads);
    ks::stage_factor<kThreads>(A, edge, nn, sA, tid);
    const ks::Source gs = ks::source(p.g, a);
    const ks::Source bs = ks::source(p.G, b);
    const int kk = lane >> 4, j16 = lane & 15;
    const int nt = (2 * n + 15) / 16;

    for (int r0 = 0; r0 < n; r0 += t.rc) {
        const int rc = n - r0 < t.rc ? n - r0 : t.rc, nrow = 3 * rc;
        const ks::Div by_row = t.by_row[rc < t.rc];
        const int nel = rc * n, eq = by_row.quot(tid), el = tid - eq * nel;
        const bool f_lane = eq * ks::kEBlk < eb;
        const int f_r = t.by_n.quot(el);
        const int f_off = f_lane ? (eq * ks::kEBlk * rc + f_r) * np + el - f_r * n : 0;
        auto pass = [&](auto second) {
            constexpr bool SECOND = decltype(second)::value;
            f64x4 sum[kNT];
#pragma unroll
            for (int c = 0; c < kNT; ++c) sum[c] = f64x4{0.0, 0.0, 0.0, 0.0};
            // the coefficients of transformed momentum, or (DIRECT) of phonon momentum, q
            auto coeff = [&](int q) {
                __syncthreads();
                if (tid == 0) *bad = 0;
                __syncthreads();
                ks::stage_coeff<kThreads, DIRECT, !SECOND, SECOND>(Dm, tw, nkz, q, nw, ne, edges, edge, sD, bad, tid);
                if constexpr (TWO)
                    ks::stage_coeff<kThreads, DIRECT, !SECOND, SECOND>(Dp, tw, nkz, q, nw, ne, edges, edge, sDm, bad, tid);
            };
            for (int m = m_lo; m < m_hi; ++m) {
                const int kt = !DIRECT && SECOND && m > 0 ? nkz - m : m;
                if constexpr (!DIRECT) coeff(kt);
                for (int e0 = e_lo; e0 < e_hi; e0 += eb) {
                    const int e_n = e_hi - e0 < eb ? e_hi - e0 : eb, ewin = eb + 2 * nw;
                    cd acc[3][ks::kEBlk];
#pragma unroll
                    for (int i = 0; i < 3; ++i)
#pragma unroll
                        for (int e = 0; e < ks::kEBlk; ++e) acc[i][e] = cd{0.0, 0.0};
                    for (int kp = 0; kp < (DIRECT ? nkz : 1); ++kp) {
                        // dSigma at k' + q meets B at k' = m with the coefficient of q
                        if constexpr (DIRECT) coeff(kp - m < 0 ? kp - m + nkz : kp - m);
                        __syncthreads();
                        ks::load_rows<kThreads, GSRC, SECOND>(gs, tw, nkz, DIRECT ? kp : kt, e0 - nw, ewin, r0, rc, n,
                                                              by_row, t.by_n, sG, tid);
                        __syncthreads();
                        const bool finite = *bad == 0;
                        for (int j = 0; j < 3; ++j) {
                            ks::right_product<kWaves, 2, kCB, false>(sG, sA + j * nn, ewin * rc, n, t.ncb, t.by_ncb,
                                                                     (wave + j) % kWaves, lane,
                                                                     [&](int row) { return sX + row * np; });
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
                    ks::load_rows<kThreads, BSRC, SECOND>(bs, tw, nkz, kt, e0, e_n, 0, n, n, t.by_nn, t.by_n, sB, tid);
                    __syncthreads();
                    // C[(i,r)][(t,re/im)] += sum over (e, c, re/im): K index kk = (c parity, re/im)
                    const bool row_ok = j16 < nrow;
                    const int rho = kk & 1, cpar = kk >> 1;
                    const double* Ua = reinterpret_cast<const double*>(sU) + 2 * ((row_ok ? j16 : 0) * n + cpar) + rho;
                    const double* Ba[kNT];
                    int b_neg[kNT];
#pragma unroll
                    for (int c = 0; c < kNT; ++c) {
                        const int col = 16 * c + j16, tt = col >> 1, tau = col & 1;
                        Ba[c] = reinterpret_cast<const double*>(sB) + 2 * ((tt < n ? tt : 0) * np + cpar) + (rho ^ tau);
                        b_neg[c] = rho == 0 && tau == 1 ? (int)0x80000000u : 0;
                    }
                    for (int e = wave; e < e_n; e += kWaves) {
                        const double* u = Ua + 2 * e * 3 * nel;
                        const int bo = 2 * e * n * np;
                        for (int c0 = 0; c0 < n; c0 += 2) {
                            // an odd norb ends with half a step: its second entry reads zero
                            const bool live = c0 + cpar < n;
                            const double x = row_ok && live ? u[2 * c0] : 0.0;
#pragma unroll
                            for (int c = 0; c < kNT; ++c) {
                                if (c >= nt) break;
                                const double y = live ? Ba[c][bo + 2 * c0] : 0.0;
                                sum[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(
                                    x, __hiloint2double(__double2hiint(y) ^ b_neg[c], __double2loint(y)), sum[c], 0, 0, 0);
                            }
                        }
                    }
                }
            }
            // the waves' sums in order, scaled
            __syncthreads();
            double* red = reinterpret_cast<double*>(sG);  // [wave][row][64]
#pragma unroll
            for (int c = 0; c < kNT; ++c) {
                if (c >= nt) break;
#pragma unroll
                for (int v = 0; v < 4; ++v) red[(wave * 16 + 4 * v + kk) * 64 + 16 * c + j16] = sum[c][v];
            }
            __syncthreads();
            const cd scale = SECOND ? alpha : cd{alpha.re, -alpha.im};
            for (int x = tid; x < nrow * n; x += kThreads) {
                const int row = t.by_n.quot(x), tt = x - row * n;
                cd v{0.0, 0.0};
                for (int w = 0; w < kWaves; ++w) {
                    v.re += red[(w * 16 + row) * 64 + 2 * tt];
                    v.im += red[(w * 16 + row) * 64 + 2 * tt + 1];
                }
                v = cmul(scale, v);
                if constexpr (SECOND) {
                    const cd o = ks::ld(sO + x);
                    const int i = row / rc;
                    cstore(out, ((int64_t)share * edges + edge) * 3 * nn + i * nn + (r0 + row - i * rc) * n + tt,
                           cd{o.re + v.re, o.im + v.im});
                } else {
                    ks::st(sO + x, v);
                }
            }
        };
        pass(std::integral_constant<bool, false>{});
        pass(std::integral_constant<bool, true>{});
    }
}

template <int GSRC, int BSRC, bool DIRECT, bool TWO>
__global__ __launch_bounds__(kThreads, 2) void dh_kspace_kernel(Dims d, ks::Gate gate, DhArgs p, const double* __restrict__ Dp,
                                                                const double* __restrict__ Dm, const double* __restrict__ A,
                                                                const int32_t* __restrict__ nbr, cd alpha, DhTile t,
                                                                int nshare, ks::LaunchPart part, ks::Twiddles table,
                                                                double* __restrict__ out) {
    if (ks::shut<DIRECT>(gate)) return;
    auto run = [&](int block) {
        dh_block<GSRC, BSRC, DIRECT, TWO>(block, d, p, Dp, Dm, A, nbr, alpha, t, nshare, part, table, out);
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

// LDS entries of a tile: its buffers, then everything
static int64_t dh_body(const Dims& d, int rc, int eb) {
    const int64_t n = d.norb, np = ks::row_len((int)n), rows = (eb + 2 * d.nw) * rc * np;
    return std::max(std::max(2 * rows, eb * 3 * rc * n + eb * n * np), (int64_t)kWaves * 16 * 64 / 2);
}
static int64_t dh_entries(const Dims& d, bool two, int rc, int eb) {
    return dh_body(d, rc, eb) + (two ? 18 : 9) * d.nw + 3 * rc * d.norb + 3 * d.norb * d.norb + 2 * d.nkz + 1;
}
static bool dh_fits(const Dims& d, bool two) {  // the smallest tile
    return d.norb <= 32 && d.nkz <= 128 && d.ne < (int64_t(1) << 28) && d.nw < (1 << 14) &&
           dh_entries(d, two, 1, ks::kEBlk) <= (int64_t)(kLdsMax / sizeof(cd));
}

static bool dh_tile(const Dims& d, bool two, DhTile* best) {
    const int n = (int)d.norb, np = ks::row_len(n);
    if (!dh_fits(d, two)) return false;
    auto up = [](double a, double b) { return (double)(int64_t)((a + b - 1) / b); };
    double best_cost = 0.0;
    bool found = false;
    for (int rc = 1; rc <= 5 && rc <= n; ++rc)
        for (int eb = ks::kEBlk; eb <= 64 && eb / ks::kEBlk * rc * n <= kThreads; eb += ks::kEBlk) {
            DhTile t{};
            const int tail = n % rc ? n % rc : rc;
            t.eb = eb;
            t.rc = rc;
            t.ncb = (n + kCB - 1) / kCB;
            t.by_n = ks::Div(n);
            t.by_ncb = ks::Div(t.ncb);
            t.by_row[0] = ks::Div(rc * n);
            t.by_row[1] = ks::Div(tail * n);
            t.by_nn = ks::Div(n * n);
            const int64_t all = dh_entries(d, two, rc, eb);
            if (all > (int64_t)(kLdsMax / sizeof(cd))) break;
            t.rows = (int)(eb + 2 * d.nw) * rc * np;
            t.u_entries = eb * 3 * rc * n;
            t.body = (int)dh_body(d, rc, eb);
            t.lds = sizeof(cd) * (size_t)all;
            const int occ = t.lds <= kLdsMax / 2 ? 2 : 1;
            const double win = eb + 2.0 * d.nw;
            const double rt = 3 * up(win * rc, 128) * t.ncb, r1 = n * kCB * 8.8 + 80;
            const double f1 = 3.0 * d.nw * ks::kEBlk * (two ? 24 : 14);
            const double c1 = up(eb, kWaves) * up(n, 2) * up(2.0 * n, 16) * 18;
            const double fixed = 600 + 25 * (up(win * rc * n, kThreads) + up((double)eb * n * n, kThreads));
            const double total = rt * r1 + up((double)eb / ks::kEBlk * rc * n, 64) * f1 + kWaves * (c1 + fixed);
            const double longest = up(rt, kWaves) * r1 + f1 + c1 + fixed + 2000;
            const double cost = up(n, rc) * up((double)std::min<int64_t>(d.ne, 32), eb) * (total / kWaves + longest / occ);
            if (!found || cost < best_cost) {
                best_cost = cost;
                *best = t;
                found = true;
            }
        }
    return found;
}

bool dh_kspace_supported(const Dims& d) { return dh_fits(d, true); }

template <int GSRC, int BSRC, bool DIRECT, bool TWO>
static hipError_t launch_dh(const Dims& d, ks::Gate gate, const DhArgs& p, const double* Dp, const double* Dm, const double* A,
                            const int32_t* nbr, cd alpha, const DhTile& t, int64_t nshare, double* shares,
                            hipStream_t stream) {
    auto kern = dh_kspace_kernel<GSRC, BSRC, DIRECT, TWO>;
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)t.lds);
    if (e != hipSuccess) return e;
    if (d.nb * nshare > INT32_MAX) return hipErrorInvalidValue;
    ks::launch_parts(d.na, d.nb * nshare, kThreads, [&](ks::LaunchPart part) {
        const unsigned groups = DIRECT && gate.word ? std::min(part.groups, ks::kGatedGroups) : part.groups;
        hipLaunchKernelGGL(kern, dim3(groups), dim3(kThreads), t.lds, stream, d, gate, p, Dp, Dm, A, nbr, alpha, t, (int)nshare,
                           part, ks::twiddles(d.nkz), shares);
    });
    return hipGetLastError();
}

hipError_t launch_dh_kspace(const Dims& d, ks::Gate gate, bool with_direct, const double* g, const double* g_hat, const double* G,
                            const double* G_hat, const double* Dp, const double* Dm, const double* A, const int32_t* nbr,
                            cd alpha, bool by_energy, double* shares, hipStream_t stream) {
    if (!gate.word && !with_direct) return hipSuccess;
    const bool two = Dm != Dp;
    DhTile t;
    if (!dh_tile(d, two, &t)) return hipErrorInvalidValue;
    const DhArgs raw{ks::array_blocks(g, d, 1), ks::array_blocks(G, d, d.gs), by_energy};
    const int64_t nshare = by_energy ? (d.ne + 31) / 32 : d.nkz;
#define SSE_DH(GS, BS, DIRECT, ARGS, SCALE)                                                                             \
    (two ? launch_dh<GS, BS, DIRECT, true>(d, gate, ARGS, Dp, Dm, A, nbr, SCALE, t, nshare, shares, stream)             \
         : launch_dh<GS, BS, DIRECT, false>(d, gate, ARGS, Dp, Dm, A, nbr, SCALE, t, nshare, shares, stream))
    if (gate.word) {
        DhArgs p = raw;
        if (G_hat && g_hat) p.g = ks::hat_blocks(g_hat, d, 0, d.ne);
        if (G_hat) p.G = ks::hat_blocks(G_hat, d, 0, d.ne);
        const cd a{alpha.re / (double)d.nkz, alpha.im / (double)d.nkz};
        const hipError_t e = G_hat && g_hat ? SSE_DH(ks::kDirect, ks::kDirect, false, p, a)
                             : G_hat        ? SSE_DH(ks::kTrans, ks::kDirect, false, p, a)
                                            : SSE_DH(ks::kTrans, ks::kTrans, false, p, a);
        if (e != hipSuccess) return e;
    }
    if (!with_direct) return hipSuccess;
    return SSE_DH(ks::kDirect, ks::kDirect, true, raw, alpha);
#undef SSE_DH
}

}  // namespace sse
