// dG of the adjoint in the momentum transform (fwd_kspace.h), any shape.
#include "fwd_kspace.h"

namespace sse {

using namespace fwd;

hipError_t launch_dg_kspace(const Dims& d, ks::Gate gate, bool with_direct, const double* g, const double* g_hat, const double* Dp,
                            const double* Dm, const double* A, const int32_t* offset, const int32_t* edges,
                            const int32_t* order, cd calpha, double* dG, hipStream_t stream) {
    if (!gate.word && !with_direct) return hipSuccess;
    const bool two = Dm != Dp;
    const int64_t nn = d.norb * d.norb, ne = d.ne;
    int cb;
    Tile t{};
    hipError_t e = choose_tile(d, two, false, &cb, &t);
    if (e != hipSuccess) return e;
    const InEdges in{offset, edges, order};
    const ks::Blocks raw = ks::array_blocks(g, d, 1), hat = ks::hat_blocks(g_hat, d, 0, ne);
    const int32_t* no_nbr = nullptr;
    const double* no_b = nullptr;
    // the E - w terms of this sum come from the table of the G at E + w
    auto launch = [&](auto src, auto direct, const ks::Blocks& blocks) {
        return launch_tables<decltype(src)::value, decltype(direct)::value, kAdjoint>(two, cb, d, gate, blocks, Dm, Dp, A, no_b,
                                                                            no_nbr, in, calpha, t, 0, (int)ne, (int)d.gs, dG,
                                                                            stream);
    };
    if (gate.word) {
        e = g_hat ? launch(kFrom<ks::kDirect>{}, std::false_type{}, hat) : launch(kFrom<ks::kTrans>{}, std::false_type{}, raw);
        if (e == hipSuccess) e = launch_inverse((int)d.nkz, gate, 0, ne * d.na, nn, d.gs * nn, calpha, dG, stream);
        if (e != hipSuccess) return e;
    }
    if (!with_direct) return hipSuccess;
    return launch(kFrom<ks::kDirect>{}, std::true_type{}, raw);
}

}  // namespace sse
