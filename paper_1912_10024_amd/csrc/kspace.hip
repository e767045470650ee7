// The momentum transforms around the kernels of kspace.h.  Both are bound by
// memory: one read and one write of the array.
#include <algorithm>

#include "kspace.h"
#include "sse_kernels.h"

namespace sse {

// ks::momentum_sum of NK values in registers
template <int NK, bool CONJ>
__device__ __forceinline__ cd momentum_sum(const cd (&v)[NK > 0 ? NK : 1], const cd* tw, int m) {
    cd s = v[0];
#pragma unroll
    for (int k = 1; 2 * k < NK; ++k) ks::pair_fma<CONJ>(s, v[k], v[NK - k], ks::ld(tw + 2 * (k * m % NK)), ks::ld(tw + 2 * (k * m % NK) + 1));
    if constexpr (NK % 2 == 0) ks::middle_add(s, v[NK / 2], m);
    return s;
}

// hat[m][x][e - first][nn] = sum_k src[k][e][x][nn] exp(-2 pi i k m / nkz) for e in
// [first, first + n_e), x < na: a block's entries stay together, its momenta and
// energies come next to each other.  The sum runs over pairs of k as in ks::load_rows,
// bit for bit.  NK = 0: any nkz, the thread's inputs in LDS.
template <int NK>
__global__ __launch_bounds__(256) void transform_kernel(int nkz, ks::Twiddles table, int64_t first, int64_t n_e, int64_t na,
                                                        int64_t nn, int64_t atom, int64_t est, int64_t kst,
                                                        const double* __restrict__ src, double* __restrict__ hat,
                                                        int* __restrict__ clear) {
    if (clear && blockIdx.x == 0 && threadIdx.x == 0) *clear = 0;  // the word of the checks that follow
    extern __shared__ __align__(16) double smem[];
    cd* tw = reinterpret_cast<cd*>(smem);
    const int tid = threadIdx.x, threads = blockDim.x;
    ks::stage_twiddles(tw, table, nkz, tid, threads);
    __syncthreads();
    cd* col = tw + 2 * nkz + tid;
    const int64_t total = n_e * na * nn, out_kst = na * n_e * nn;
    for (int64_t x = blockIdx.x * (int64_t)threads + tid; x < total; x += (int64_t)gridDim.x * threads) {
        const int64_t blk = x / nn, rc = x - blk * nn, e = blk / na, a = blk - e * na;
        const double* p = src + 2 * ((first + e) * est + a * atom + rc);
        double* o = hat + 2 * ((a * n_e + e) * nn + rc);
        if constexpr (NK > 0) {
            cd v[NK > 0 ? NK : 1];
#pragma unroll
            for (int k = 0; k < NK; ++k) v[k] = cload(p, k * kst);
#pragma unroll
            for (int m = 0; m < NK; ++m) cstore(o, m * out_kst, momentum_sum<NK, false>(v, tw, m));
        } else {
            for (int k = 0; k < nkz; ++k) ks::st(col + k * threads, cload(p, k * kst));
            for (int m = 0; m < nkz; ++m)
                cstore(o, m * out_kst, ks::momentum_sum(nkz, m, tw, [&](int k) { return ks::ld(col + k * threads); }));
        }
    }
}

// X[k] = scale / nkz * sum_m X[m] exp(+2 pi i k m / nkz), in place over the leading axis of
// [nkz][blocks][bs] (the first nn entries of every block of bs).  edges: of Pi, whose edge
// blk mod edges may be marked, 0: none is
template <int NK>
__global__ __launch_bounds__(256) void inverse_kernel(int nkz, ks::Twiddles table, ks::Gate gate, int64_t edges,
                                                      int64_t blocks, int64_t nn, int64_t bs, cd scale,
                                                      double* X) {
    if (ks::shut<false>(gate)) return;
    extern __shared__ __align__(16) double smem[];
    cd* tw = reinterpret_cast<cd*>(smem);
    const int tid = threadIdx.x, threads = blockDim.x;
    ks::stage_twiddles(tw, table, nkz, tid, threads);
    __syncthreads();
    cd* col = tw + 2 * nkz + tid;
    // 1 / nkz in two terms: the quotient of every sum is rounded like a division
    const double inv = 1.0 / (double)nkz, inv_low = fma(-inv, (double)nkz, 1.0) * inv;
    auto scaled = [&](cd s) {
        const cd v = cmul(scale, s);
        return cd{fma(v.re, inv, v.re * inv_low), fma(v.im, inv, v.im * inv_low)};
    };
    const int64_t total = blocks * nn, kst = blocks * bs;
    for (int64_t x = blockIdx.x * (int64_t)threads + tid; x < total; x += (int64_t)gridDim.x * threads) {
        const int64_t blk = x / nn;
        double* p = X + 2 * (blk * bs + x - blk * nn);
        // (a thread that is done may have written that entry, but never the marker)
        if (edges && ks::marked(X, blk % edges * bs)) continue;
        if constexpr (NK > 0) {
            cd v[NK > 0 ? NK : 1];
#pragma unroll
            for (int m = 0; m < NK; ++m) v[m] = cload(p, m * kst);
#pragma unroll
            for (int k = 0; k < NK; ++k) cstore(p, k * kst, scaled(momentum_sum<NK, true>(v, tw, k)));
        } else {
            for (int m = 0; m < nkz; ++m) ks::st(col + m * threads, cload(p, m * kst));
            for (int k = 0; k < nkz; ++k)
                cstore(p, k * kst,
                       scaled(ks::momentum_sum<true>(nkz, k, tw, [&](int m) { return ks::ld(col + m * threads); })));
        }
    }
}

template <class K, class... Args>
static hipError_t launch_transform_kernel(K kern, bool any, int nkz, int64_t total, hipStream_t stream, Args... args) {
    const int threads = any ? 64 : 256;
    const size_t lds = sizeof(cd) * (size_t)(2 * nkz + (any ? nkz * threads : 0));
    if (any) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)lds);
        if (e != hipSuccess) return e;
    }
    const int64_t want = (total + threads - 1) / threads;
    hipLaunchKernelGGL(kern, dim3((unsigned)(want < 65536 ? want : 65536)), dim3(threads), lds, stream, nkz,
                       ks::twiddles(nkz), args...);
    return hipGetLastError();
}

#define SSE_BY_NKZ(KERN, TOTAL, ...)                                                                  \
    switch (nkz) {                                                                                    \
        case 2: return launch_transform_kernel(KERN<2>, false, nkz, TOTAL, stream, __VA_ARGS__);      \
        case 3: return launch_transform_kernel(KERN<3>, false, nkz, TOTAL, stream, __VA_ARGS__);      \
        case 4: return launch_transform_kernel(KERN<4>, false, nkz, TOTAL, stream, __VA_ARGS__);      \
        case 5: return launch_transform_kernel(KERN<5>, false, nkz, TOTAL, stream, __VA_ARGS__);      \
        case 6: return launch_transform_kernel(KERN<6>, false, nkz, TOTAL, stream, __VA_ARGS__);      \
        case 7: return launch_transform_kernel(KERN<7>, false, nkz, TOTAL, stream, __VA_ARGS__);      \
        default: return launch_transform_kernel(KERN<0>, true, nkz, TOTAL, stream, __VA_ARGS__);      \
    }

hipError_t launch_transform(const Dims& d, int64_t first, int64_t n_e, const ks::Blocks& src, double* hat, int* clear,
                            hipStream_t stream) {
    const int nkz = (int)d.nkz;
    const int64_t na = d.na, nn = d.norb * d.norb;
    SSE_BY_NKZ(transform_kernel, n_e * na * nn, first, n_e, na, nn, src.atom, src.est, src.kst, src.p, hat, clear)
}

hipError_t launch_inverse(int nkz, ks::Gate gate, int64_t edges, int64_t blocks, int64_t nn, int64_t bs, cd scale, double* X,
                          hipStream_t stream) {
    SSE_BY_NKZ(inverse_kernel, blocks * nn, gate, edges, blocks, nn, bs, scale, X)
}

#undef SSE_BY_NKZ

// Sets `bit` of *word where the blocks of p or q are not of like size at all momenta (every
// block has bs entries, nn of them used).  Bound by memory: one read of the arrays (1.5 GB
// of Go, 100 entries a block, in 0.3 ms).
__global__ __launch_bounds__(256) void spread_kernel(int nkz, ks::Gate only, int64_t blocks, int nn, int64_t bs, int64_t kst,
                                                     int L, const double* __restrict__ p, const double* __restrict__ q,
                                                     int bit, int* word) {
    if (ks::shut<true>(only)) return;  // nobody asks
    const int l = threadIdx.x & (L - 1);
    const int64_t per = 256 / L;
    bool like = true;
    for (int64_t b0 = blockIdx.x * per; b0 < blocks; b0 += gridDim.x * per) {
        const int64_t b = b0 + threadIdx.x / L, blk = b < blocks ? b : b0;
        like = ks::like_blocks(p + 2 * blk * bs, kst, nkz, nn, l, L) && like;
        if (q) like = ks::like_blocks(q + 2 * blk * bs, kst, nkz, nn, l, L) && like;
    }
    if (__syncthreads_or(!like) && threadIdx.x == 0) atomicOr(word, bit);
}

hipError_t launch_spread(int nkz, ks::Gate only, int64_t blocks, int64_t nn, int64_t bs, const double* p, const double* q, int bit,
                         int* word, hipStream_t stream) {
    const int L = ks::block_lanes(nn);
    const int64_t groups = (blocks + 256 / L - 1) / (256 / L), most = only.word ? 512 : 8192;
    hipLaunchKernelGGL(spread_kernel, dim3((unsigned)std::min(groups, most)), dim3(256), 0, stream, nkz, only, blocks, (int)nn, bs,
                       blocks * bs, L, p, q, bit, word);
    return hipGetLastError();
}

__global__ void clear_word_kernel(int* word) { *word = 0; }
hipError_t launch_clear_word(int* word, hipStream_t stream) {
    hipLaunchKernelGGL(clear_word_kernel, dim3(1), dim3(1), 0, stream, word);
    return hipGetLastError();
}

// Without room for the word: marks the edges of Pi whose blocks of Gs and of Go both differ
// in size, in the first output of each of their workgroups (w = 0, step, 2 step, ... of
// every momentum); an edge without a neighbour is not marked.
__global__ __launch_bounds__(256) void mark_pi_kernel(Dims d, ks::Blocks y, ks::Blocks x, int L, int step,
                                                      const int32_t* __restrict__ nbr, double* __restrict__ Pi) {
    const int l = threadIdx.x & (L - 1), per = 256 / L, nn = (int)(d.norb * d.norb);
    const int64_t edges = d.na * d.nb;
    for (int64_t edge = blockIdx.x; edge < edges; edge += gridDim.x) {
        const int64_t a = edge / d.nb, b = nbr[edge];
        const bool valid = b >= 0 && b < d.na;
        bool like_x = true, like_y = true;
        for (int64_t e0 = 0; valid && e0 < d.ne; e0 += per) {
            const int64_t e = e0 + threadIdx.x / L < d.ne ? e0 + threadIdx.x / L : e0;
            like_x = ks::like_blocks(x.p + 2 * (b * x.atom + e * x.est), x.kst, (int)d.nkz, nn, l, L) && like_x;
            like_y = ks::like_blocks(y.p + 2 * (a * y.atom + e * y.est), y.kst, (int)d.nkz, nn, l, L) && like_y;
        }
        const bool mark = __syncthreads_or(!like_x) && __syncthreads_or(!like_y);
        const int64_t slots = d.nkz * ((d.nw + step - 1) / step);
        for (int64_t s = threadIdx.x; s < slots; s += 256) {
            const int64_t k = s % d.nkz, w = s / d.nkz * step;
            *reinterpret_cast<unsigned long long*>(Pi + 2 * (((k * d.nw + w) * edges + edge) * 9)) = mark ? ks::kMarker : 0;
        }
    }
}

hipError_t launch_mark_pi(const Dims& d, const ks::Blocks& y, const ks::Blocks& x, int step, const int32_t* nbr, double* Pi,
                          hipStream_t stream) {
    const int64_t groups = std::min<int64_t>(d.na * d.nb, 1 << 20);
    hipLaunchKernelGGL(mark_pi_kernel, dim3((unsigned)groups), dim3(256), 0, stream, d, y, x, ks::block_lanes(d.norb * d.norb), step,
                       nbr, Pi);
    return hipGetLastError();
}

}  // namespace sse
