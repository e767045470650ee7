// Sigma in the momentum transform (fwd_kspace.h), any shape.
#include <algorithm>

#include "fwd_kspace.h"

namespace sse {

using namespace fwd;

bool fwd_kspace_supported(const Dims& d, bool two) {
    if (d.norb > 32 || d.nkz > 128 || d.ne >= (int64_t(1) << 28) || d.nw >= (1 << 14) || d.nb >= (1 << 28)) return false;
    return make_tile(d, ks::kEBlk, 1, 5, two, true).lds <= kLdsMax;
}

// bytes of workspace that hold hat G: all of it, or a slab of energies of at most
// kSlabBytes (at least the energies one tile meets)
static int64_t hat_energy_bytes(const Dims& d) { return 16 * d.nkz * d.na * d.norb * d.norb; }
size_t fwd_kspace_workspace(const Dims& d) {
    constexpr int64_t kSlabBytes = int64_t(4) << 30;
    if (d.nkz == 1 || d.nkz * d.ne * d.na <= kDirectBlocks || !fwd_kspace_supported(d, true)) return 0;
    const int64_t per = hat_energy_bytes(d), want = std::max(kSlabBytes / per, 64 + 4 * d.nw);
    return (size_t)(per * std::min(d.ne, want)) + 2 * ks::kWordBytes;
}

hipError_t launch_fwd_kspace(const Dims& d, const double* G, const double* Dp, const double* Dm, const double* A,
                             const double* B, const int32_t* nbr, cd alpha, double* S, bool transform, void* ws,
                             size_t ws_bytes, hipStream_t stream) {
    const bool two = Dm != Dp;
    const int64_t nn = d.norb * d.norb, ne = d.ne;
    const int nkz = (int)d.nkz;
    int cb;
    Tile t{};
    hipError_t e = choose_tile(d, two, B != nullptr, &cb, &t);
    if (e != hipSuccess) return e;
    const InEdges none{};
    const ks::Blocks raw = ks::array_blocks(G, d, d.gs);
    ks::Gate gate{nullptr, ks::kSpreadD | ks::kSpreadG};
    auto launch = [&](auto src, auto direct, const ks::Blocks& blocks, int64_t lo, int64_t hi) {
        constexpr int kSrc = decltype(src)::value;
        constexpr bool kDir = decltype(direct)::value;
        return B ? launch_tables<kSrc, kDir, kStored>(two, cb, d, gate, blocks, Dp, Dm, A, B, nbr, none, alpha, t, (int)lo,
                                                      (int)hi, 1, S, stream)
                 : launch_tables<kSrc, kDir, kHermitian>(two, cb, d, gate, blocks, Dp, Dm, A, B, nbr, none, alpha, t, (int)lo,
                                                         (int)hi, 1, S, stream);
    };
    if (!transform) return launch(kFrom<ks::kDirect>{}, std::true_type{}, raw, 0, ne);
    // the word of the checks, then hat G, both aligned
    int* word = reinterpret_cast<int*>(ks::aligned(ws));
    double* hat = reinterpret_cast<double*>(reinterpret_cast<char*>(word) + ks::kWordBytes);
    const int64_t left = static_cast<char*>(ws) + ws_bytes - reinterpret_cast<char*>(hat);
    const int64_t room = left / hat_energy_bytes(d);  // energies
    const bool slabs = room >= std::min(ne, (int64_t)t.eb + 2 * d.nw);
    auto check = [&] {
        gate.word = word;
        hipError_t c = launch_spread(nkz, ks::Gate{}, d.nw * d.na * d.nb, 9, 9, Dp, two ? Dm : nullptr, ks::kSpreadD, word, stream);
        if (c != hipSuccess) return c;
        return launch_spread(nkz, ks::Gate{word, ks::kSpreadD}, ne * d.na, nn, d.gs * nn, G, nullptr, ks::kSpreadG, word, stream);
    };
    if (slabs) {
        // slabs of whole tiles; a slab's transform takes the 2 nw energies around it
        const int64_t step = room >= ne ? ne : (room - 2 * d.nw) / t.eb * t.eb;
        for (int64_t lo = 0; lo < ne; lo += step) {
            const int64_t hi = std::min(ne, lo + step);
            const int64_t first = std::max<int64_t>(0, lo - d.nw), n_e = std::min(ne, hi + d.nw) - first;
            e = launch_transform(d, first, n_e, raw, hat, lo == 0 ? word : nullptr, stream);
            if (e == hipSuccess && lo == 0) e = check();
            if (e == hipSuccess) e = launch(kFrom<ks::kDirect>{}, std::false_type{}, ks::hat_blocks(hat, d, first, n_e), lo, hi);
            if (e != hipSuccess) return e;
        }
    } else {
        e = launch_clear_word(word, stream);
        if (e == hipSuccess) e = check();
        if (e == hipSuccess) e = launch(kFrom<ks::kTrans>{}, std::false_type{}, raw, 0, ne);
        if (e != hipSuccess) return e;
    }
    e = launch_inverse(nkz, gate, 0, ne * d.na, nn, nn, alpha, S, stream);
    if (e != hipSuccess) return e;
    // the direct sum on the matrix cores where they have an instance: more than twice as fast
    // (10 orbitals, 1024 atoms, 256 energies: 88 against 186 ms)
    if (!fwd_mfma_supports(d, SSE_FP64, B != nullptr)) return launch(kFrom<ks::kDirect>{}, std::true_type{}, raw, 0, ne);
    if (!two) return launch_fwd_mfma(d, SSE_FP64, G, Dp, A, B, nbr, alpha, S, stream, kBranchMinus | kBranchPlus, &gate);
    e = launch_fwd_mfma(d, SSE_FP64, G, Dp, A, B, nbr, alpha, S, stream, kBranchMinus, &gate);
    if (e != hipSuccess) return e;
    return launch_fwd_mfma(d, SSE_FP64, G, Dm, A, B, nbr, alpha, S, stream, kBranchPlus | kAccumulate, &gate);
}

}  // namespace sse
