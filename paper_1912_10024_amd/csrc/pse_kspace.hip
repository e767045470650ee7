// Pi in the momentum transform (corr_kspace.h), any shape.
#include <algorithm>

#include "corr_kspace.h"

namespace sse {

using namespace corr;

bool corr_kspace_supported(const Dims& d, bool both) { return ks::corr_fits(d, true, both); }

template <int SRC, bool DIRECT, class... Args>
static hipError_t launch_pi_corr(int wb, Args... args) {
    return launch_corr_shape<SRC, SRC, DIRECT, true, false, true>(wb, args...);
}

hipError_t launch_pi_kspace(const Dims& d, const double* Gs, const double* Go, const double* A, const int32_t* nbr, cd beta,
                            double* Pi, bool transform, void* ws, size_t ws_bytes, hipStream_t stream) {
    CorrTile t;
    if (!corr_tile(d, true, false, &t)) return hipErrorInvalidValue;
    const int64_t ne = d.ne, nn = d.norb * d.norb, edges = d.na * d.nb;
    const int nkz = (int)d.nkz;
    const ks::Blocks y = ks::array_blocks(Gs, d, d.gs), x = ks::array_blocks(Go, d, d.gs);
    const CorrArgs raw{y, x, 0, (int)ne, false};
    ks::Gate gate{nullptr, ks::kSpreadG | ks::kSpreadSigma};
    bool marks = false;
    auto direct = [&] { return launch_pi_corr<ks::kDirect, true>(t.wb, d, gate, marks, raw, A, nbr, beta, t, Pi, stream); };
    if (!transform) return direct();
    // The word of the checks, then the transforms: both whole, or slabs of whole tiles of energies
    // of both, or neither.  A slab of Go meets the energies of Gs above its first, up to nw
    // more than its own: one fewer than the two arrays have, which leaves the word its room.
    int* word = reinterpret_cast<int*>(ks::aligned(ws));
    double* hy = reinterpret_cast<double*>(reinterpret_cast<char*>(word) + ks::kWordBytes);
    const int64_t left = static_cast<char*>(ws) + ws_bytes - reinterpret_cast<char*>(hy);
    const int64_t per = 16 * d.nkz * d.na * nn, room = left > 0 ? left / per : 0;  // energies
    const int64_t step = room >= 2 * ne - 1 ? ne : (room - d.nw + 1) / 2 / t.eb * t.eb;
    hipError_t e = hipSuccess;
    const bool slabs = ws && step >= std::min<int64_t>(ne, t.eb);
    // without room for transforms the matrix cores' direct sum is the faster one, and the more
    // exact (41 against 48 ms)
    if (!slabs && pse_mfma_specialised(d)) return launch_pse(d, Gs, Go, A, nbr, beta, Pi, stream);
    auto check = [&] {
        gate.word = word;
        hipError_t c = launch_spread(nkz, ks::Gate{}, ne * d.na, nn, d.gs * nn, Go, nullptr, ks::kSpreadG, word, stream);
        if (c != hipSuccess) return c;
        return launch_spread(nkz, ks::Gate{word, ks::kSpreadG}, ne * d.na, nn, d.gs * nn, Gs, nullptr, ks::kSpreadSigma, word, stream);
    };
    if (slabs) {
        for (int64_t lo = 0; lo < ne && e == hipSuccess; lo += step) {
            const int64_t hi = std::min(ne, lo + step), n_x = hi - lo, n_y = std::min(ne, hi + d.nw) - (lo + 1);
            double* hx = hy + per / 8 * n_y;
            e = launch_transform(d, lo, n_x, x, hx, lo == 0 ? word : nullptr, stream);
            if (e == hipSuccess && n_y > 0) e = launch_transform(d, lo + 1, n_y, y, hy, nullptr, stream);
            if (e == hipSuccess && lo == 0) e = check();
            if (e != hipSuccess) return e;
            const CorrArgs g{ks::hat_blocks(hy, d, lo + 1, n_y), ks::hat_blocks(hx, d, lo, n_x), (int)lo, (int)hi, lo > 0};
            e = launch_pi_corr<ks::kDirect, false>(t.wb, d, gate, marks, g, A, nbr, beta, t, Pi, stream);
        }
    } else {
        if (ws && left >= 0) {
            e = launch_clear_word(word, stream);
            if (e == hipSuccess) e = check();
        } else {
            marks = true;
            e = launch_mark_pi(d, y, x, t.nwb * t.wb, nbr, Pi, stream);
        }
        if (e == hipSuccess) e = launch_pi_corr<ks::kTrans, false>(t.wb, d, gate, marks, raw, A, nbr, beta, t, Pi, stream);
    }
    if (e == hipSuccess) e = launch_inverse(nkz, gate, marks ? edges : 0, d.nw * edges, 9, 9, beta, Pi, stream);
    if (e != hipSuccess) return e;
    // the direct sum on the matrix cores where they have an instance: 41 against 156 ms (512 atoms,
    // 256 energies)
    return pse_mfma_specialised(d) ? launch_pse(d, Gs, Go, A, nbr, beta, Pi, stream, &gate) : direct();
}

// both transforms, or slabs of at most 32 GiB of them (a slab costs a prologue and a
// reduction: at 4864 atoms and 1024 energies 16 slabs took 1603 ms)
size_t corr_kspace_workspace(const Dims& d) {
    constexpr int64_t kSlabBytes = int64_t(32) << 30;
    if (d.nkz == 1 || d.nkz * d.ne * d.na <= kDirectBlocks || !corr_kspace_supported(d, false)) return 0;
    const int64_t per = 16 * d.nkz * d.na * d.norb * d.norb;
    return (size_t)(per * std::min(2 * d.ne, std::max(kSlabBytes / per, 256 + 4 * d.nw)));
}

}  // namespace sse
