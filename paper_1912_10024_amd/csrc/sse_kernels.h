// Launch entry points of the kernels behind the C ABI.
#pragma once

#include "sse_common.h"

namespace sse {

// Energy branches of Eq. 3 on a grid of positive frequencies w: the terms with
// G at E - w (coefficient at +w) and those with G at E + w (coefficient at -w)
constexpr int kBranchMinus = 1;  // terms with G at E - w
constexpr int kBranchPlus = 2;   // terms with G at E + w
constexpr int kAccumulate = 4;   // Sigma += result instead of Sigma = result

// direct term-by-term fp64 forward (any shape with norb^2 <= 1024); the terms
// with G at E - w read Dp, those with G at E + w read Dm (Dm == Dp: the
// one-table form of sse_forward); B = stored grad_j H_ba blocks (layout of A),
// or nullptr for A^H
bool generic_supported(const Dims& d);
hipError_t launch_fwd_generic(const Dims& d, const double* G, const double* Dp, const double* Dm, const double* A,
                              const double* B, const int32_t* nbr, cd alpha, double* S, hipStream_t stream);

namespace ks {
struct Blocks;  // kspace.h
struct Gate;
}

// the momentum transform of a block array into hat[m][atom][energy][nn] for the
// energies [first, first + n_e) (clear: a word that is set to zero, or NULL), and its inverse in
// place over the leading axis of [nkz][blocks][bs] (the first nn entries of every block), times
// scale / nkz; edges: 0, or those of Pi (marked ones are left)
hipError_t launch_transform(const Dims& d, int64_t first, int64_t n_e, const ks::Blocks& src, double* hat, int* clear,
                            hipStream_t stream);
hipError_t launch_inverse(int nkz, ks::Gate gate, int64_t edges, int64_t blocks, int64_t nn, int64_t bs, cd scale, double* X,
                          hipStream_t stream);

// the choice between transform and direct sum (ks::Gate): sets a bit of *word where blocks of
// p (or q, unless NULL) differ in size over the momenta, if all bits of `only` are set; or
// marks edges of Pi
hipError_t launch_spread(int nkz, ks::Gate only, int64_t blocks, int64_t nn, int64_t bs, const double* p, const double* q, int bit,
                         int* word, hipStream_t stream);
hipError_t launch_clear_word(int* word, hipStream_t stream);
hipError_t launch_mark_pi(const Dims& d, const ks::Blocks& y, const ks::Blocks& x, int step, const int32_t* nbr, double* Pi,
                          hipStream_t stream);

// fp64 forward in the momentum transform (kspace.h), any shape whose tile fits the
// LDS; transform = false sums over the source momenta as they stand.  Problems of
// at most kDirectBlocks output blocks (four per compute unit) keep the direct sum:
// their time is latency, and sums of integer-valued inputs stay exact.  ws holds the
// transform of G, or a slab of it, where ws_bytes has room (fwd_kspace_workspace);
// otherwise every workgroup transforms what it loads
constexpr int64_t kDirectBlocks = 1024;
bool fwd_kspace_supported(const Dims& d, bool two);
size_t fwd_kspace_workspace(const Dims& d);
hipError_t launch_fwd_kspace(const Dims& d, const double* G, const double* Dp, const double* Dm, const double* A,
                             const double* B, const int32_t* nbr, cd alpha, double* S, bool transform, void* ws,
                             size_t ws_bytes, hipStream_t stream);

// Pi in the momentum transform, any shape.  transform as for launch_fwd_kspace; ws holds
// the transforms of Gs and Go, or slabs of energies of them, whose sums are added in
// order (their last bits then depend on the room)
bool corr_kspace_supported(const Dims& d, bool both);
size_t corr_kspace_workspace(const Dims& d);
hipError_t launch_pi_kspace(const Dims& d, const double* Gs, const double* Go, const double* A, const int32_t* nbr, cd beta,
                            double* Pi, bool transform, void* ws, size_t ws_bytes, hipStream_t stream);

// The adjoint in the momentum transform, any shape.  g_hat, G_hat: the whole transforms
// of g = dL/dSigma and G (launch_transform), or NULL: every workgroup transforms what
// it loads (the same sums, bit for bit).
// dG from the in-edges of every atom; the one-table form passes Dm = Dp
hipError_t launch_dg_kspace(const Dims& d, ks::Gate gate, bool with_direct, const double* g, const double* g_hat, const double* Dp,
                            const double* Dm, const double* A, const int32_t* offset, const int32_t* edges,
                            const int32_t* order, cd calpha, double* dG, hipStream_t stream);
// d gradH: one share per edge and part of the (momenta, energies), added by the caller;
// by_energy: a share holds all momenta of 32 energies, else all energies of a momentum
bool dh_kspace_supported(const Dims& d);
hipError_t launch_dh_kspace(const Dims& d, ks::Gate gate, bool with_direct, const double* g, const double* g_hat, const double* G,
                            const double* G_hat, const double* Dp, const double* Dm, const double* A, const int32_t* nbr,
                            cd alpha, bool by_energy, double* shares, hipStream_t stream);
// dD; branches: 1 the terms with G at E - w (coefficients at +w), 2 those with G at E + w, 3 both
hipError_t launch_dd_kspace(const Dims& d, ks::Gate gate, bool with_direct, int branches, const double* g, const double* g_hat, const double* G,
                            const double* G_hat, const double* A, const int32_t* nbr, cd calpha, double* dD,
                            hipStream_t stream);

// the direct sums of the adjoint on the matrix cores: dG and the d gradH shares of the one-table
// form (one per 32 energies), each behind its own check, and dD
bool bwd_mfma_specialised(const Dims& d);
hipError_t launch_bwd_mfma(const Dims& d, ks::Gate gate, ks::Gate gate_dh, const double* G, const double* D, const double* A,
                           const double* gS, cd calpha, const int32_t* offset, const int32_t* edges, const int32_t* order,
                           double* dG, double* shares, hipStream_t stream);
hipError_t launch_dd_mfma(const Dims& d, ks::Gate gate, int branches, const double* g, const double* G, const double* A,
                          const int32_t* nbr, cd calpha, double* dD, hipStream_t stream);

// matrix-core forward (fp64 or fp32 operands; the split 16-bit forms go to
// launch_fwd_h16) for the shapes it is
// instantiated for; flags selects the energy branches (kBranchMinus,
// kBranchPlus) and whether the result is added to Sigma (kAccumulate)
// B: stored grad_j H_ba blocks (layout of A) as the right factor, or nullptr for A^H; gate: of the
// fp64 form behind the check of the momenta
bool fwd_mfma_specialised(const Dims& d);
// whether the matrix-core forward takes this precision (and a stored grad H_ba) at these dims
bool fwd_mfma_supports(const Dims& d, int precision, bool hba);
hipError_t launch_fwd_mfma(const Dims& d, int precision, const double* G, const double* D, const double* A,
                           const double* B, const int32_t* nbr, cd alpha, double* S, hipStream_t stream,
                           int flags = kBranchMinus | kBranchPlus, const ks::Gate* gate = nullptr);

// matrix-core forward with split 16-bit operands (SSE_FP16X2, SSE_BF16X2, and the
// single-term SSE_FP16 and SSE_FP16_UNSCALED with the flags of the one-table form
// only) for the shapes of fwd_mfma_specialised; B and flags as for launch_fwd_mfma
hipError_t launch_fwd_h16(const Dims& d, int precision, const double* G, const double* D, const double* A,
                          const double* B, const int32_t* nbr, cd alpha, double* S, hipStream_t stream, int flags);

// adjoint (fp64): reverse adjacency in the workspace, then dG/d gradH per neighbour atom and dD.
// signed_form: the terms with G at E - w read Dp and feed dDp, those at E + w
// read Dm and feed dDm; otherwise Dp is the one table and dDp its gradient (Dm,
// dDm unused).
size_t bwd_workspace_bytes(const Dims& d);  // enough for either form, with every gradient
// what one call requires: the reverse adjacency, plus the d gradH shares if that
// gradient is asked for, plus (with_hat) the transform of g on the shapes of the
// matrix-core forward with 3 or 4 neighbours
size_t bwd_workspace_bytes_for(const Dims& d, bool signed_form, bool with_dh, bool with_hat);
size_t bwd_fast_workspace_bytes(const Dims& d);  // what a call is fastest with
bool bwd_supported(const Dims& d);
hipError_t launch_bwd(const Dims& d, const double* G, const double* Dp, const double* Dm, const double* A,
                      const int32_t* nbr, cd alpha, const double* gS, double* dG, double* dDp, double* dDm, double* dA,
                      void* ws, size_t ws_bytes, hipStream_t stream, bool signed_form);

// absorption-branch coefficients: Dm[q,w,a,n,i,j] = Dopp[(-q) mod nqz, w, a, n, j, i]
hipError_t launch_absorption_d(const Dims& d, const double* Dopp, double* Dm, hipStream_t stream);

// Eq. 3 bracket from the full phonon blocks (symmetric neighbour table)
size_t combine_workspace_bytes(const Dims& d);
hipError_t launch_reverse_slots(const Dims& d, const int32_t* nbr, void* ws, hipStream_t stream);
hipError_t launch_combine_d(const Dims& d, const double* Dfull, const int32_t* nbr, double* Dc, void* ws,
                            hipStream_t stream);

// phonon self-energy (Eq. 4, off-diagonal blocks): matrix-core kernel for the shape it is
// instantiated for, a vector-ALU kernel for every other shape that fits
bool pse_mfma_specialised(const Dims& d);
bool pse_generic_supported(const Dims& d);
hipError_t launch_pse(const Dims& d, const double* Gs, const double* Go, const double* A, const int32_t* nbr, cd beta,
                      double* Pi, hipStream_t stream, const ks::Gate* gate = nullptr);
// sse_backward; with_hat = false: a workspace without the transform of g will do
// (sse_backward_noalloc)
int backward_one_table(const sse_dims* dims, const double* G, const double* D, const double* dH, const int32_t* nbr,
                       double alpha_re, double alpha_im, const double* dSigma, double* dG, double* dD, double* ddH,
                       void* workspace, size_t workspace_bytes, void* stream, bool with_hat);

// sets the thread-local text that sse_last_error returns; returns code
int set_error(int code, const char* fmt, ...);

// neighbour-table range check: sets *flag (device int) to 1 if any entry is outside [0, na)
hipError_t launch_check_nbr(const Dims& d, const int32_t* nbr, int* flag, hipStream_t stream);

}  // namespace sse
