// The D gradient of the adjoint in the momentum transform (corr_kspace.h), any shape.
#include "corr_kspace.h"

namespace sse {

using namespace corr;

template <int YSRC, int XSRC, bool DIRECT, class... Args>
static hipError_t launch_dd(int branches, int wb, Args... args) {
    if (branches == 3) return launch_corr_shape<YSRC, XSRC, DIRECT, true, true, false>(wb, args...);
    if (branches == 1) return launch_corr_shape<YSRC, XSRC, DIRECT, true, false, false>(wb, args...);
    return launch_corr_shape<YSRC, XSRC, DIRECT, false, true, false>(wb, args...);
}

hipError_t launch_dd_kspace(const Dims& d, ks::Gate gate, bool with_direct, int branches, const double* g, const double* g_hat, const double* G,
                            const double* G_hat, const double* A, const int32_t* nbr, cd calpha, double* dD,
                            hipStream_t stream) {
    if (!gate.word && !with_direct) return hipSuccess;
    CorrTile t;
    if (!corr_tile(d, (branches & 1) != 0, (branches & 2) != 0, &t)) return hipErrorInvalidValue;
    const CorrArgs raw{ks::array_blocks(g, d, 1), ks::array_blocks(G, d, d.gs), 0, (int)d.ne, false};
    if (gate.word) {
        CorrArgs a = raw;
        if (G_hat && g_hat) a.y = ks::hat_blocks(g_hat, d, 0, d.ne);
        if (G_hat) a.x = ks::hat_blocks(G_hat, d, 0, d.ne);
        hipError_t e;
        if (G_hat && g_hat)
            e = launch_dd<ks::kDirect, ks::kDirect, false>(branches, t.wb, d, gate, false, a, A, nbr, calpha, t, dD, stream);
        else if (G_hat)
            e = launch_dd<ks::kTrans, ks::kDirect, false>(branches, t.wb, d, gate, false, a, A, nbr, calpha, t, dD, stream);
        else
            e = launch_dd<ks::kTrans, ks::kTrans, false>(branches, t.wb, d, gate, false, a, A, nbr, calpha, t, dD, stream);
        if (e == hipSuccess) e = launch_inverse((int)d.nkz, gate, 0, d.nw * d.na * d.nb, 9, 9, calpha, dD, stream);
        if (e != hipSuccess) return e;
    }
    if (!with_direct) return hipSuccess;
    return launch_dd<ks::kDirect, ks::kDirect, true>(branches, t.wb, d, gate, false, raw, A, nbr, calpha, t, dD, stream);
}

}  // namespace sse
