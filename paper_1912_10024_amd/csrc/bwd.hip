// Adjoint of the scattering self-energy (fp64): the workspace and the dispatch, and the
// kernels for shapes whose window of 2 nw energies does not fit the LDS of those in
// bwd_dg_kspace.hip (dG), bwd_kspace.hip (d gradH) and bwd_dd_kspace.hip (dD).
//
// With g = dL/dSigma (PyTorch's complex-gradient convention) define, for an
// edge (a, n) with neighbour b = nbr[a,n] and a source point (k', E'):
//   W_{q,w}[k',E'] = g[(k'+q) mod Nkz, E'+w, a] + g[(k'+q) mod Nkz, E'-w, a]   (0 outside the grid)
//   Y_ij[k',E']    = conj(alpha) sum_{q,w} conj(D[q,w-1,a,n,i,j]) W_{q,w}[k',E']
// (the adjoint of the (qz, w, +/-) stencil and of the D contraction; over
// signed frequencies the g at E'+w term takes conj(Dp) and the one at E'-w
// conj(Dm)), and with
// B = G[k',E',b,0], P_ij = grad_i H . B . grad_j H^H:
//   dG[k',E',b,0]   += sum_ij grad_i H^H . Y_ij . grad_j H
//   d gradH[a,n,m]  += sum_j Y_mj . (grad_j H . B^H) + sum_i Y_im^H . (grad_i H . B)
//   dD[q,w-1,a,n,ij] = conj(alpha) sum_{k',E'} sum_rc conj(P_ij[rc]) W_{q,w}[rc]
//   (over signed frequencies: dDp from the g at E'+w terms, dDm from E'-w)
// Shifted blocks are re-gathered from G and g, nothing of the forward is stored.
//
// Here dG and d gradH are formed by one workgroup per neighbour atom b, which walks
// the edges that point at b (a reverse adjacency built in the workspace, in
// edge order), so every output element has one owner: no atomics, bitwise
// reproducible; dD by one workgroup per edge.
#include <algorithm>

#include "kspace.h"
#include "sse_kernels.h"

namespace sse {

namespace {
constexpr int kBwdThreads = 256;
constexpr int kYHalf = kBwdThreads / 2;   // first thread of the second Y group
}

// ---------------------------------------------------------------- reverse adjacency
// ws layout (int32): count[na] | offset[na+1] | cursor[na] | edges[na*nb] | order[na]; once it is
// built, the first word holds what spread_kernel found
__global__ void rcsr_count_kernel(int64_t na, int64_t nb, const int32_t* __restrict__ nbr, int32_t* count) {
    for (int64_t x = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; x < na * nb; x += (int64_t)gridDim.x * blockDim.x) {
        const int32_t b = nbr[x];
        if (b >= 0 && b < na) atomicAdd(&count[b], 1);
    }
}

// single workgroup exclusive scan (na is at most a few hundred thousand)
__global__ void rcsr_scan_kernel(int64_t na, const int32_t* __restrict__ count, int32_t* offset, int32_t* cursor) {
    __shared__ int32_t part[1024];
    const int tid = threadIdx.x, nt = blockDim.x;
    const int64_t per = (na + nt - 1) / nt;
    const int64_t lo = tid * per, hi = (lo + per < na) ? lo + per : na;
    int32_t s = 0;
    for (int64_t i = lo; i < hi; ++i) s += count[i];
    part[tid] = s;
    __syncthreads();
    if (tid == 0) {
        int32_t run = 0;
        for (int t = 0; t < nt; ++t) {
            const int32_t v = part[t];
            part[t] = run;
            run += v;
        }
        offset[na] = run;
    }
    __syncthreads();
    int32_t run = part[tid];
    for (int64_t i = lo; i < hi; ++i) {
        offset[i] = run;
        cursor[i] = run;
        run += count[i];
    }
}

__global__ void rcsr_fill_kernel(int64_t na, int64_t nb, const int32_t* __restrict__ nbr, int32_t* cursor, int32_t* edges) {
    for (int64_t x = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; x < na * nb; x += (int64_t)gridDim.x * blockDim.x) {
        const int32_t b = nbr[x];
        if (b >= 0 && b < na) edges[atomicAdd(&cursor[b], 1)] = (int32_t)x;
    }
}

// the fill order is arbitrary: sort each (short) list so the walk is in edge order
__global__ void rcsr_sort_kernel(int64_t na, const int32_t* __restrict__ offset, int32_t* edges) {
    for (int64_t b = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; b < na; b += (int64_t)gridDim.x * blockDim.x) {
        const int32_t lo = offset[b], hi = offset[b + 1];
        for (int32_t i = lo + 1; i < hi; ++i) {
            const int32_t v = edges[i];
            int32_t j = i - 1;
            while (j >= lo && edges[j] > v) {
                edges[j + 1] = edges[j];
                --j;
            }
            edges[j + 1] = v;
        }
    }
}

// atoms in decreasing in-degree (the dispatch order of both dG / d gradH kernels:
// a workgroup's time grows with the in-degree of its atom, so the longest start
// first and the shortest fill the end).  One workgroup; degrees above 255
// share the first bucket; the order within a bucket is arbitrary, which changes
// no result (every workgroup of that kernel owns its outputs).
__global__ __launch_bounds__(1024) void rcsr_order_kernel(int64_t na, const int32_t* __restrict__ count,
                                                          int32_t* __restrict__ order) {
    __shared__ int32_t cursor[256];
    const int tid = threadIdx.x;
    if (tid < 256) cursor[tid] = 0;
    __syncthreads();
    auto bucket = [&](int64_t a) { return 255 - (count[a] < 255 ? count[a] : 255); };
    for (int64_t a = tid; a < na; a += 1024) atomicAdd(&cursor[bucket(a)], 1);
    __syncthreads();
    if (tid == 0) {
        int32_t run = 0;
        for (int k = 0; k < 256; ++k) {
            const int32_t c = cursor[k];
            cursor[k] = run;
            run += c;
        }
    }
    __syncthreads();
    for (int64_t a = tid; a < na; a += 1024) order[atomicAdd(&cursor[bucket(a)], 1)] = (int32_t)a;
}

// The whole adjacency and order in one launch for small tables: six launches of a few
// microseconds each, one of them a scan whose middle runs on one thread, were a tenth of the smallest
// adjoint.  One workgroup, the counts in LDS.
constexpr int kSmallAtoms = 4096, kSmallEdges = 1 << 16;

// exclusive prefix sums of v over the 1024 threads (part: 1024 entries)
__device__ __forceinline__ int32_t scan_1024(int32_t v, int32_t* part, int tid) {
    part[tid] = v;
    __syncthreads();
    for (int step = 1; step < 1024; step <<= 1) {
        const int32_t add = tid >= step ? part[tid - step] : 0;
        __syncthreads();
        part[tid] += add;
        __syncthreads();
    }
    const int32_t r = part[tid] - v;
    __syncthreads();
    return r;
}

__global__ __launch_bounds__(1024) void rcsr_small_kernel(int na, int nb, const int32_t* __restrict__ nbr,
                                                          int32_t* __restrict__ offset, int32_t* __restrict__ edges,
                                                          int32_t* __restrict__ order) {
    __shared__ int32_t cursor[kSmallAtoms];
    __shared__ int32_t part[1024];
    __shared__ int32_t bucket[256];
    const int tid = threadIdx.x, total = na * nb;
    for (int i = tid; i < na; i += 1024) cursor[i] = 0;
    __syncthreads();
    for (int x = tid; x < total; x += 1024) {
        const int32_t b = nbr[x];
        if (b >= 0 && b < na) atomicAdd(&cursor[b], 1);
    }
    __syncthreads();
    constexpr int kPer = kSmallAtoms / 1024;
    const int per = (na + 1023) / 1024, lo = tid * per;
    int32_t cnt[kPer], sum = 0;
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        cnt[u] = u < per && lo + u < na ? cursor[lo + u] : 0;
        sum += cnt[u];
    }
    int32_t run = scan_1024(sum, part, tid);
    if (tid < 256) bucket[tid] = 0;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        if (u >= per || lo + u >= na) continue;
        cursor[lo + u] = run;
        offset[lo + u] = run;
        run += cnt[u];
        if (lo + u == na - 1) offset[na] = run;
        atomicAdd(&bucket[255 - (cnt[u] < 255 ? cnt[u] : 255)], 1);
    }
    __syncthreads();
    const int32_t first = scan_1024(tid < 256 ? bucket[tid] : 0, part, tid);
    if (tid < 256) bucket[tid] = first;
    __syncthreads();
    for (int x = tid; x < total; x += 1024) {
        const int32_t b = nbr[x];
        if (b >= 0 && b < na) edges[atomicAdd(&cursor[b], 1)] = x;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        if (u >= per || lo + u >= na) continue;
        order[atomicAdd(&bucket[255 - (cnt[u] < 255 ? cnt[u] : 255)], 1)] = lo + u;
        // the fill order is arbitrary: sort the list so the walk is in edge order
        int32_t* e = edges + cursor[lo + u] - cnt[u];
        for (int i = 1; i < cnt[u]; ++i) {
            const int32_t v = e[i];
            int j = i - 1;
            for (; j >= 0 && e[j] > v; --j) e[j + 1] = e[j];
            e[j + 1] = v;
        }
    }
}

__global__ void zero_i32_kernel(int64_t n, int32_t* p) {
    for (int64_t x = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; x < n; x += (int64_t)gridDim.x * blockDim.x) p[x] = 0;
}

// ws layout after the reverse adjacency (256-byte aligned): the d gradH shares of
// every edge (complex [share][na*nb][3][norb][norb]), added in order by
// bwd_dh_reduce_kernel, if d gradH is asked for; then the momentum transforms of g
// and of G, as far as there is room
static size_t bwd_csr_bytes(const Dims& d) {  // count, offset, cursor, edges, order
    return (sizeof(int32_t) * (size_t)(4 * d.na + 1 + d.na * d.nb) + 255) / 256 * 256;
}
static bool bwd_use_kspace(const Dims& d) {
    return fwd_kspace_supported(d, true) && dh_kspace_supported(d) && corr_kspace_supported(d, true);
}
// one d gradH share per 32 energies on the shape of the matrix-core forward, whose Nkz
// shares would take more room, else one per momentum, as the kernels of this file always write
static bool bwd_by_energy(const Dims& d, bool signed_form) {
    return !signed_form && d.norb == 10 && d.nkz == 7 && d.nqz == 7 && d.nw == 10 && bwd_use_kspace(d) &&
           d.na * ((d.ne + 31) / 32) <= INT32_MAX;
}
static int64_t bwd_shares(const Dims& d, bool signed_form) {
    return bwd_by_energy(d, signed_form) ? (d.ne + 31) / 32 : d.nkz;
}
static size_t bwd_dh_bytes(const Dims& d, bool signed_form) {
    return (sizeof(cd) * (size_t)(bwd_shares(d, signed_form) * d.na * d.nb * 3 * d.norb * d.norb) + 255) / 256 * 256;
}
// the whole transform of g, or of slot 0 of G
static size_t bwd_hat_bytes(const Dims& d) {
    return (size_t)(16 * d.norb * d.norb * d.nkz * d.ne * d.na + 255) / 256 * 256;
}
size_t bwd_workspace_bytes_for(const Dims& d, bool signed_form, bool with_dh, bool with_hat) {
    const bool hat = with_hat && !signed_form && d.norb == 10 && d.nkz == 7 && d.nw == 10 && (d.nb == 3 || d.nb == 4) &&
                     d.ne < (int64_t(1) << 28);
    return bwd_csr_bytes(d) + (with_dh ? bwd_dh_bytes(d, signed_form) : 0) + (hat ? bwd_hat_bytes(d) : 0);
}
size_t bwd_workspace_bytes(const Dims& d) {
    return std::max(bwd_workspace_bytes_for(d, false, true, true), bwd_workspace_bytes_for(d, true, true, true));
}
size_t bwd_fast_workspace_bytes(const Dims& d) {
    constexpr size_t kHats = size_t(16) << 30;  // at most this for the transforms
    const size_t least = bwd_workspace_bytes(d), hat = bwd_hat_bytes(d);
    if (!bwd_use_kspace(d) || hat > kHats) return least;
    const size_t base = bwd_csr_bytes(d) + std::max(bwd_dh_bytes(d, false), bwd_dh_bytes(d, true));
    return std::max(least, base + (2 * hat <= kHats ? 2 * hat : hat));
}

// --------------------------------------------------------------- W and Y of one source point
// A zero row read in place of g blocks outside the energy grid, so the loads of
// a batch of frequencies can all be issued before their products (never written;
// not const, so it shares the global address space with g).
__device__ double bwd_zero_row[2] = {0.0, 0.0};

// Y_ij[x] for all nine (i,j), summed over every qz and the frequencies
// w in [w_lo, w_hi] of the 2*Nqz*Nw shifted g blocks (both energy branches);
// the loads of two qz and kBatch frequencies are in flight together.
// conj(alpha) is applied by the caller.  SIGNED: the g block at E'+w takes the
// table sDn (coefficients at +w), the one at E'-w the table sDm (at -w).
template <bool SIGNED>
__device__ __forceinline__ void compute_y(const Dims& d, const double* __restrict__ gS, int64_t a, int64_t kp,
                                          int64_t ep, const cd* sDn, const cd* sDm, int64_t w_lo, int64_t w_hi,
                                          int x, cd* y) {
    constexpr int kBatch = 5, kQ = 2;
#pragma unroll
    for (int ij = 0; ij < 9; ++ij) y[ij] = cd{0.0, 0.0};
    for (int64_t q0 = 0; q0 < d.nqz; q0 += kQ) {
        for (int64_t w0 = w_lo; w0 <= w_hi; w0 += kBatch) {
            cd hi[kQ][kBatch], lo[kQ][kBatch];
#pragma unroll
            for (int u = 0; u < kQ; ++u) {
                const bool q_in = q0 + u < d.nqz;
                const int64_t k = (kp + (q_in ? q0 + u : 0)) % d.nkz;
#pragma unroll
                for (int t = 0; t < kBatch; ++t) {
                    const int64_t w = w0 + t;
                    const bool in = q_in && w <= w_hi, h_ok = in && ep + w < d.ne, l_ok = in && ep - w >= 0;
                    // energies clamped to the source energy when out of the grid, so no pointer leaves g
                    const double* ph = h_ok ? gS + 2 * (off_S(d, k, h_ok ? ep + w : ep, a) + x) : bwd_zero_row;
                    const double* pl = l_ok ? gS + 2 * (off_S(d, k, l_ok ? ep - w : ep, a) + x) : bwd_zero_row;
                    hi[u][t] = cd{ph[0], ph[1]};
                    lo[u][t] = cd{pl[0], pl[1]};
                }
            }
#pragma unroll
            for (int u = 0; u < kQ; ++u) {
                if (q0 + u >= d.nqz) break;
#pragma unroll
                for (int t = 0; t < kBatch; ++t) {
                    const int64_t w = w0 + t;
                    if (w > w_hi) break;
                    const int64_t qw = ((q0 + u) * d.nw + (w - 1)) * 9;
                    if constexpr (SIGNED) {
#pragma unroll
                        for (int ij = 0; ij < 9; ++ij) {
                            cfma_conja(y[ij], sDn[qw + ij], hi[u][t]);
                            cfma_conja(y[ij], sDm[qw + ij], lo[u][t]);
                        }
                    } else {
                        const cd wv{hi[u][t].re + lo[u][t].re, hi[u][t].im + lo[u][t].im};
#pragma unroll
                        for (int ij = 0; ij < 9; ++ij) cfma_conja(y[ij], sDn[qw + ij], wv);
                    }
                }
            }
        }
    }
}

// --------------------------------------------------------------- dG and d gradH
template <bool SIGNED>
__global__ __launch_bounds__(kBwdThreads) void bwd_dg_dh_kernel(Dims d, const double* __restrict__ G,
                                                                const double* __restrict__ Dg,
                                                                const double* __restrict__ Dmg,
                                                                const double* __restrict__ Ag,
                                                                const double* __restrict__ gS, cd calpha,
                                                                const int32_t* __restrict__ offset,
                                                                const int32_t* __restrict__ edges,
                                                                const int32_t* __restrict__ order, int64_t first,
                                                                double* __restrict__ dG, double* __restrict__ dApart) {
    extern __shared__ double smem[];
    const int N = (int)d.norb, NN = N * N;
    const int nqw = (int)(d.nqz * d.nw);
    cd* sDn = reinterpret_cast<cd*>(smem);  // [q][w][ij]
    cd* sDm = sDn + nqw * 9;                // [q][w][ij]  (SIGNED: the coefficients at -w)
    cd* sA = sDm + (SIGNED ? nqw * 9 : 0);  // [3][N][N]   grad H of the edge
    cd* sY = sA + 3 * NN;                   // [9][N][N]
    cd* sB = sY + 9 * NN;                   // [N][N]
    cd* sT = sB + NN;                       // [3][N][N]   sum_i A_i^H Y_ij
    cd* sC = sT + 3 * NN;                   // [3][N][N]   A_j B^H
    cd* sE = sC + 3 * NN;                   // [3][N][N]   A_i B
    cd* sdA = sE + 3 * NN;                  // [3][N][N]   accumulated d gradH of the edge
    cd* sY1 = sT;                           // [9][N][N]   second half of the frequency sum of Y; shares
                                            // sT, sC, sE (9 N^2), which are written only after the merge
    const int tid = threadIdx.x;
    // One workgroup per (neighbour atom b, momentum k'): Nkz times as many
    // workgroups as atoms.  The Nkz workgroups of one atom get ids on the same
    // XCD (they read the same D, grad H and g blocks); the atoms come in
    // decreasing in-degree (a workgroup walks the edges into its atom), so the
    // longest workgroups start first.
    const int64_t bid = first + blockIdx.x, span = 8 * d.nkz;
    const int64_t pos = (bid / span) * 8 + bid % 8;
    const int64_t kp = (bid % span) / 8;
    if (pos >= d.na) return;  // uniform for the workgroup, before any barrier
    const int64_t b = order[pos];
    const int32_t e_lo = offset[b], e_hi = offset[b + 1];

    // slots >= 1 of dG are not read by the forward map: zero
    if (dG && (d.gs > 1 || e_lo == e_hi)) {
        for (int64_t ep = 0; ep < d.ne; ++ep) {
            const int64_t base = off_G(d, kp, ep, b);
            const int64_t from = (e_lo == e_hi) ? 0 : NN;
            for (int64_t x = from + tid; x < d.gs * NN; x += kBwdThreads) cstore(dG, base + x, cd{0.0, 0.0});
        }
    }
    for (int32_t ei = e_lo; ei < e_hi; ++ei) {
        const int32_t edge = edges[ei];
        const int64_t a = edge / d.nb, n = edge % d.nb;
        __syncthreads();
        for (int x = tid; x < nqw * 9; x += kBwdThreads) {
            const int ij = x % 9, qw = x / 9;
            sDn[x] = cload(Dg, off_D(d, qw / d.nw, qw % d.nw, a, n) + ij);
            if constexpr (SIGNED) sDm[x] = cload(Dmg, off_D(d, qw / d.nw, qw % d.nw, a, n) + ij);
        }
        for (int x = tid; x < 3 * NN; x += kBwdThreads) {
            sA[x] = cload(Ag, off_A(d, a, n, 0) + x);
            sdA[x] = cd{0.0, 0.0};
        }
        __syncthreads();
        for (int64_t ep = 0; ep < d.ne; ++ep) {
            // Y: threads [0, NN) sum the frequencies up to Nw/2, threads
            // [kYHalf, kYHalf + NN) the rest; the halves are then added
            const int yh = tid >= kYHalf ? 1 : 0;
            for (int yx = tid - yh * kYHalf; yx < NN; yx += kYHalf) {
                cd y[9];
                const int64_t w_mid = d.nw / 2;
                compute_y<SIGNED>(d, gS, a, kp, ep, sDn, sDm, yh ? w_mid + 1 : 1, yh ? d.nw : w_mid, yx, y);
                cd* dst = yh ? sY1 : sY;
#pragma unroll
                for (int ij = 0; ij < 9; ++ij) dst[ij * NN + yx] = y[ij];
                if (!yh) sB[yx] = cload(G, off_G(d, kp, ep, b) + yx);
            }
            __syncthreads();
            for (int x = tid; x < 9 * NN; x += kBwdThreads) {
                const cd u = sY[x], v = sY1[x];
                sY[x] = cmul(calpha, cd{u.re + v.re, u.im + v.im});
            }
            __syncthreads();
            // T_j = sum_i A_i^H Y_ij ; C_j = A_j B^H ; E_i = A_i B
            for (int x = tid; x < 9 * NN; x += kBwdThreads) {
                const int m = x / NN, rc = x % NN, r = rc / N, c = rc % N;
                cd s{0.0, 0.0};
                if (m < 3) {
                    const int j = m;
                    for (int i = 0; i < 3; ++i)
                        for (int t = 0; t < N; ++t) cfma_conja(s, sA[i * NN + t * N + r], sY[(i * 3 + j) * NN + t * N + c]);
                    sT[j * NN + rc] = s;
                } else if (m < 6) {
                    const int j = m - 3;
                    for (int t = 0; t < N; ++t) cfma_conj(s, sA[j * NN + r * N + t], sB[c * N + t]);
                    sC[j * NN + rc] = s;
                } else {
                    const int i = m - 6;
                    for (int t = 0; t < N; ++t) cfma(s, sA[i * NN + r * N + t], sB[t * N + c]);
                    sE[i * NN + rc] = s;
                }
            }
            __syncthreads();
            // dG[k',E',b] (+)= sum_j T_j A_j
            for (int x = tid; dG && x < NN; x += kBwdThreads) {
                const int t = x / N, u = x % N;
                cd s{0.0, 0.0};
                for (int j = 0; j < 3; ++j)
                    for (int c = 0; c < N; ++c) cfma(s, sT[j * NN + t * N + c], sA[j * NN + c * N + u]);
                const int64_t o = off_G(d, kp, ep, b) + x;
                if (ei != e_lo) {
                    const cd prev = cload(dG, o);
                    s.re += prev.re;
                    s.im += prev.im;
                }
                cstore(dG, o, s);
            }
            // d gradH_m += sum_j Y_mj C_j + sum_i Y_im^H E_i
            for (int x = tid; dApart && x < 3 * NN; x += kBwdThreads) {
                const int m = x / NN, rc = x % NN, r = rc / N, c = rc % N;
                cd s = sdA[x];
                for (int j = 0; j < 3; ++j)
                    for (int t = 0; t < N; ++t) cfma(s, sY[(m * 3 + j) * NN + r * N + t], sC[j * NN + t * N + c]);
                for (int i = 0; i < 3; ++i)
                    for (int t = 0; t < N; ++t) cfma_conja(s, sY[(i * 3 + m) * NN + t * N + r], sE[i * NN + t * N + c]);
                sdA[x] = s;
            }
            __syncthreads();
        }
        // this momentum's share of the edge's d gradH (edge index a * nb + n)
        for (int x = tid; dApart && x < 3 * NN; x += kBwdThreads)
            cstore(dApart, (kp * d.na * d.nb + edge) * 3 * NN + x, sdA[x]);
    }
}

// d gradH of every edge (a, n): its partial sums (one per momentum k', or per
// energy range on the matrix-core path) added in share order; an edge whose
// neighbour entry lies outside [0, na) has no terms and gets zero
__global__ void bwd_dh_reduce_kernel(Dims d, const int32_t* __restrict__ nbr, const double* __restrict__ dApart,
                                     int64_t shares, double* __restrict__ dA) {
    const int64_t NN3 = 3 * d.norb * d.norb, per_k = d.na * d.nb * NN3;
    for (int64_t x = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; x < per_k; x += (int64_t)gridDim.x * blockDim.x) {
        const int32_t b = nbr[x / NN3];
        cd s{0.0, 0.0};
        if (b >= 0 && b < d.na)
            for (int64_t kp = 0; kp < shares; ++kp) {
                const cd v = cload(dApart, kp * per_k + x);
                s.re += v.re;
                s.im += v.im;
            }
        cstore(dA, x, s);
    }
}

// --------------------------------------------------------------- dD
// branches: bit 0 the g blocks at E'+w (the terms with G at E - w), bit 1 those at E'-w
__global__ __launch_bounds__(kBwdThreads) void bwd_dd_kernel(Dims d, const double* __restrict__ G,
                                                             const double* __restrict__ Ag,
                                                             const int32_t* __restrict__ nbr,
                                                             const double* __restrict__ gS, cd calpha, int branches,
                                                             int64_t first, double* __restrict__ dD) {
    extern __shared__ double smem[];
    const int N = (int)d.norb, NN = N * N;
    const int nqw = (int)(d.nqz * d.nw);
    cd* sA = reinterpret_cast<cd*>(smem);  // [3][N][N]
    cd* sB = sA + 3 * NN;                  // [N][N]
    cd* sE = sB + NN;                      // [3][N][N]  A_i B
    cd* sP = sE + 3 * NN;                  // [9][N][N]  A_i B A_j^H
    const int tid = threadIdx.x;
    const int64_t edge = first + blockIdx.x;
    if (edge >= d.na * d.nb) return;
    const int64_t a = edge / d.nb, n = edge % d.nb;
    const int32_t b = nbr[edge];
    for (int x = tid; x < 3 * NN; x += kBwdThreads) sA[x] = cload(Ag, off_A(d, a, n, 0) + x);
    // each thread owns up to two (q, w) pairs and accumulates all nine (i,j)
    constexpr int kPer = 2;
    cd acc[kPer][9];
#pragma unroll
    for (int s = 0; s < kPer; ++s)
#pragma unroll
        for (int ij = 0; ij < 9; ++ij) acc[s][ij] = cd{0.0, 0.0};
    const bool valid_b = b >= 0 && b < d.na;
    for (int64_t kp = 0; kp < d.nkz; ++kp)
        for (int64_t ep = 0; ep < d.ne; ++ep) {
            __syncthreads();
            for (int x = tid; x < NN; x += kBwdThreads) sB[x] = valid_b ? cload(G, off_G(d, kp, ep, b) + x) : cd{0.0, 0.0};
            __syncthreads();
            for (int x = tid; x < 3 * NN; x += kBwdThreads) {
                const int i = x / NN, r = (x % NN) / N, c = x % N;
                cd s{0.0, 0.0};
                for (int t = 0; t < N; ++t) cfma(s, sA[i * NN + r * N + t], sB[t * N + c]);
                sE[x] = s;
            }
            __syncthreads();
            for (int x = tid; x < 9 * NN; x += kBwdThreads) {
                const int ij = x / NN, i = ij / 3, j = ij % 3, r = (x % NN) / N, c = x % N;
                cd s{0.0, 0.0};
                for (int u = 0; u < N; ++u) cfma_conj(s, sE[i * NN + r * N + u], sA[j * NN + c * N + u]);
                sP[x] = s;
            }
            __syncthreads();
#pragma unroll
            for (int s = 0; s < kPer; ++s) {
                const int qw = tid + s * kBwdThreads;
                if (qw < nqw) {
                    const int64_t q = qw / d.nw, w = qw % d.nw + 1;
                    const int64_t k = (kp + q) % d.nkz;
                    const bool hi = (branches & 1) && ep + w < d.ne, lo = (branches & 2) && ep - w >= 0;
                    const double* g1 = gS + 2 * off_S(d, k, hi ? ep + w : ep, a);
                    const double* g2 = gS + 2 * off_S(d, k, lo ? ep - w : ep, a);
                    for (int rc = 0; rc < NN; ++rc) {
                        cd wv{0.0, 0.0};
                        if (hi) {
                            const cd v = cload(g1, rc);
                            wv.re += v.re;
                            wv.im += v.im;
                        }
                        if (lo) {
                            const cd v = cload(g2, rc);
                            wv.re += v.re;
                            wv.im += v.im;
                        }
#pragma unroll
                        for (int ij = 0; ij < 9; ++ij) cfma_conja(acc[s][ij], sP[ij * NN + rc], wv);
                    }
                }
            }
        }
#pragma unroll
    for (int s = 0; s < kPer; ++s) {
        const int qw = tid + s * kBwdThreads;
        if (qw < nqw) {
            const int64_t q = qw / d.nw, w = qw % d.nw;
#pragma unroll
            for (int ij = 0; ij < 9; ++ij) cstore(dD, off_D(d, q, w, a, n) + ij, cmul(calpha, acc[s][ij]));
        }
    }
}

static size_t bwd_lds_dg(const Dims& d, bool signed_form = false) {
    const size_t NN = (size_t)(d.norb * d.norb);
    return sizeof(cd) * ((size_t)d.nqz * d.nw * 9 * (signed_form ? 2 : 1) + 3 * NN + 9 * NN + NN + 4 * 3 * NN);
}
static size_t bwd_lds_dd(const Dims& d) {
    const size_t NN = (size_t)(d.norb * d.norb);
    return sizeof(cd) * (3 * NN + NN + 3 * NN + 9 * NN);
}

bool bwd_supported(const Dims& d) {
    return d.nqz * d.nw <= 2 * kBwdThreads && d.norb * d.norb <= kBwdThreads && bwd_lds_dg(d, true) <= 160 * 1024 &&
           bwd_lds_dd(d) <= 160 * 1024 && d.na * d.nb <= INT32_MAX && (d.na + 7) / 8 * 8 * d.nkz <= INT32_MAX;
}

static bool bwd_small(const Dims& d) { return d.nkz == 1 || d.nkz * d.ne * d.na <= kDirectBlocks; }
// Direct sums on the matrix cores where they have an instance.  dG and d gradH: 2.2 against 3.5 ms
// with dD (13 energies of 5 atoms), 69 against 268 ms (128 energies of 512).  dD: its matrix-core
// kernel has a workgroup per atom that takes 12.6 us per source point, the other one per (edge, q)
// that takes about 0.53 ms for few energies: by their rounds on 256 compute units.
static bool bwd_direct_mfma(const Dims& d, bool signed_form) { return !signed_form && bwd_mfma_specialised(d); }
static bool dd_direct_mfma(const Dims& d) {
    const int64_t cus = 256, rounds = (d.na + cus - 1) / cus, other = (d.na * d.nb * d.nkz + cus - 1) / cus;
    return pse_mfma_specialised(d) && (!bwd_small(d) || d.nkz * d.ne * rounds < 42 * other);
}

// the kernels of kspace.h: every gradient from the transforms of g and G (room for
// them, or for that of g, permitting), or as the sum over the momenta stands
static hipError_t launch_bwd_kspace(const Dims& d, const double* G, const double* Dp, const double* Dm, const double* A,
                                    const int32_t* nbr, cd alpha, const double* gS, double* dG, double* dDp, double* dDm,
                                    double* dA, char* ws, size_t ws_bytes, int* word, const int32_t* offset,
                                    const int32_t* edges, const int32_t* order, hipStream_t stream, bool signed_form) {
    const cd calpha{alpha.re, -alpha.im};
    const int nkz = (int)d.nkz;
    const int64_t nn = d.norb * d.norb;
    const bool d_part = dDp || dDm;
    const size_t hat = bwd_hat_bytes(d), used = bwd_csr_bytes(d) + (dA ? bwd_dh_bytes(d, signed_form) : 0);
    double *g_hat = nullptr, *G_hat = nullptr;
    // the direct sum under the same line as the forward (the gate stays open for it), or where
    // the arrays under a gradient's sum ask for it: g and D for dG, G too for d gradH, g and G for dD
    const bool small = bwd_small(d);
    auto gate = [&](int mask) { return ks::Gate{small ? nullptr : word, mask | ks::kSpreadSigma}; };
    const bool mfma = bwd_direct_mfma(d, signed_form), dd_mfma = dd_direct_mfma(d);
    hipError_t e = hipSuccess;
    if (gate(0).word) {
        // Room for one transform: that of g if dG is wanted, whose array then holds that of G until
        // its own turn comes (d gradH and dD go first); else that of G, which they read more often
        // than that of g.  Without room, dG's array for that of G all the same.
        const size_t room = ws_bytes >= used ? (ws_bytes - used) / hat : 0;
        const bool want_G = dA || d_part;
        double* first = reinterpret_cast<double*>(ws + used);
        if (room >= 1 && (dG || room >= 2)) g_hat = first;
        if (want_G && room >= 2)
            G_hat = reinterpret_cast<double*>(ws + used + hat);
        else if (want_G && dG)
            G_hat = dG;
        else if (want_G && room >= 1)
            G_hat = first;
        if (g_hat) e = launch_transform(d, 0, d.ne, ks::array_blocks(gS, d, 1), g_hat, nullptr, stream);
        if (e == hipSuccess && G_hat) e = launch_transform(d, 0, d.ne, ks::array_blocks(G, d, d.gs), G_hat, nullptr, stream);
        if (e == hipSuccess) e = launch_clear_word(word, stream);
        if (e == hipSuccess)
            e = launch_spread(nkz, ks::Gate{}, d.ne * d.na, nn, nn, gS, nullptr, ks::kSpreadSigma, word, stream);
        if (e == hipSuccess && (dG || dA))
            e = launch_spread(nkz, gate(0), d.nw * d.na * d.nb, 9, 9, Dp, Dm != Dp ? Dm : nullptr, ks::kSpreadD, word, stream);
        if (e == hipSuccess && want_G)
            e = launch_spread(nkz, gate(0), d.ne * d.na, nn, d.gs * nn, G, nullptr, ks::kSpreadG, word, stream);
        if (e != hipSuccess) return e;
    }
    double* shares = dA ? reinterpret_cast<double*>(ws + bwd_csr_bytes(d)) : nullptr;
    const ks::Gate dg_gate = gate(ks::kSpreadD), dh_gate = gate(ks::kSpreadD | ks::kSpreadG), dd_gate = gate(ks::kSpreadG);
    if (dA)
        e = launch_dh_kspace(d, dh_gate, !mfma, gS, g_hat, G, G_hat, Dp, Dm, A, nbr, alpha, bwd_by_energy(d, signed_form), shares,
                             stream);
    for (int branch = 1; branch <= 2; ++branch) {
        double* dD = branch == 1 ? dDp : dDm;
        if (!dD || e != hipSuccess) continue;
        const int branches = signed_form ? branch : 3;
        e = launch_dd_kspace(d, dd_gate, !dd_mfma, branches, gS, g_hat, G, G_hat, A, nbr, calpha, dD, stream);
        if (e == hipSuccess && dd_mfma) e = launch_dd_mfma(d, dd_gate, branches, gS, G, A, nbr, calpha, dD, stream);
    }
    if (dG && e == hipSuccess)
        e = launch_dg_kspace(d, dg_gate, !mfma, gS, g_hat, Dp, Dm, A, offset, edges, order, calpha, dG, stream);
    if (mfma && (dG || dA) && e == hipSuccess)
        e = launch_bwd_mfma(d, dg_gate, dh_gate, G, Dp, A, gS, calpha, offset, edges, order, dG, shares, stream);
    if (dA && e == hipSuccess) {
        const int64_t n = d.na * d.nb * 3 * nn;
        hipLaunchKernelGGL(bwd_dh_reduce_kernel, dim3((unsigned)std::min<int64_t>((n + 255) / 256, 65536)), dim3(256), 0, stream,
                           d, nbr, shares, bwd_shares(d, signed_form), dA);
        e = hipGetLastError();
    }
    return e;
}

// dD (or dDp / dDm) for the given energy branches
static hipError_t launch_dd(const Dims& d, const double* G, const double* A, const int32_t* nbr, const double* gS, cd calpha,
                            double* dD, int branches, hipStream_t stream) {
    const int64_t all = d.na * d.nb, step = launch_groups(kBwdThreads);
    for (int64_t first = 0; first < all; first += step)
        hipLaunchKernelGGL(bwd_dd_kernel, dim3((unsigned)std::min(step, all - first)), dim3(kBwdThreads), bwd_lds_dd(d), stream, d,
                           G, A, nbr, gS, calpha, branches, first, dD);
    return hipGetLastError();
}

hipError_t launch_bwd(const Dims& d, const double* G, const double* Dp, const double* Dm, const double* A,
                      const int32_t* nbr, cd alpha, const double* gS, double* dG, double* dDp, double* dDm, double* dA,
                      void* ws, size_t ws_bytes, hipStream_t stream, bool signed_form) {
    const cd calpha{alpha.re, -alpha.im};
    const bool kspace = bwd_use_kspace(d);
    const size_t lds = bwd_lds_dg(d, signed_form);
    auto kern = signed_form ? bwd_dg_dh_kernel<true> : bwd_dg_dh_kernel<false>;
    if (!kspace) {
        // every attribute is set before the first launch, so a failure leaves all outputs untouched
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)lds);
        if (e == hipSuccess)
            e = hipFuncSetAttribute(reinterpret_cast<const void*>(bwd_dd_kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                    (int)bwd_lds_dd(d));
        if (e != hipSuccess) return e;
    }
    int32_t* count = reinterpret_cast<int32_t*>(ws);
    int32_t* offset = count + d.na;
    int32_t* cursor = offset + d.na + 1;
    int32_t* edges = cursor + d.na;
    int32_t* order = edges + d.na * d.nb;
    if (dG || (dA && (!kspace || bwd_direct_mfma(d, signed_form)))) {
        if (d.na <= kSmallAtoms && d.na * d.nb <= kSmallEdges) {
            hipLaunchKernelGGL(rcsr_small_kernel, dim3(1), dim3(1024), 0, stream, (int)d.na, (int)d.nb, nbr, offset, edges, order);
        } else {
            const unsigned g1 = (unsigned)((d.na * d.nb + 255) / 256 < 4096 ? (d.na * d.nb + 255) / 256 : 4096);
            hipLaunchKernelGGL(zero_i32_kernel, dim3(g1), dim3(256), 0, stream, d.na, count);
            hipLaunchKernelGGL(rcsr_count_kernel, dim3(g1), dim3(256), 0, stream, d.na, d.nb, nbr, count);
            hipLaunchKernelGGL(rcsr_scan_kernel, dim3(1), dim3(1024), 0, stream, d.na, count, offset, cursor);
            hipLaunchKernelGGL(rcsr_fill_kernel, dim3(g1), dim3(256), 0, stream, d.na, d.nb, nbr, cursor, edges);
            const unsigned g2 = (unsigned)((d.na + 255) / 256 < 4096 ? (d.na + 255) / 256 : 4096);
            hipLaunchKernelGGL(rcsr_sort_kernel, dim3(g2), dim3(256), 0, stream, d.na, offset, edges);
            hipLaunchKernelGGL(rcsr_order_kernel, dim3(1), dim3(1024), 0, stream, d.na, count, order);
        }
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (kspace)
        return launch_bwd_kspace(d, G, Dp, Dm, A, nbr, alpha, gS, dG, dDp, dDm, dA, static_cast<char*>(ws), ws_bytes, count,
                                 offset, edges, order, stream, signed_form);
    if (dG || dA) {
        double* shares = dA ? reinterpret_cast<double*>(reinterpret_cast<char*>(ws) + bwd_csr_bytes(d)) : nullptr;
        const int64_t groups = (d.na + 7) / 8 * 8 * d.nkz;
        const int64_t step = launch_groups(kBwdThreads) / 8 * 8;
        for (int64_t first = 0; first < groups; first += step)
            hipLaunchKernelGGL(kern, dim3((unsigned)std::min(step, groups - first)), dim3(kBwdThreads), lds, stream, d, G, Dp, Dm,
                               A, gS, calpha, offset, edges, order, first, dG, shares);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        if (dA) {
            const int64_t n = d.na * d.nb * 3 * d.norb * d.norb;
            const unsigned g3 = (unsigned)((n + 255) / 256 < 65536 ? (n + 255) / 256 : 65536);
            hipLaunchKernelGGL(bwd_dh_reduce_kernel, dim3(g3), dim3(256), 0, stream, d, nbr, shares, bwd_shares(d, signed_form), dA);
            e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
    }
    if (dDp) {
        hipError_t e = launch_dd(d, G, A, nbr, gS, calpha, dDp, signed_form ? 1 : 3, stream);
        if (e != hipSuccess) return e;
    }
    if (dDm) return launch_dd(d, G, A, nbr, gS, calpha, dDm, 2, stream);
    return hipGetLastError();
}

}  // namespace sse
