"""Rounding errors of the fp64 kernels in the momentum transform, against sums in 80 bits.

A rounded operation errs by e = 2^-53 / sqrt(3) of its result in the mean square, and a chain
of L additions of random terms by e sqrt(L / 2) of its sum.  The steps of an output add up in
squares."""
import numpy as np
import pytest
import torch

from paper_1912_10024_amd import sse
from paper_1912_10024_amd.inputs import Dims, anti_hermitian_blocks, make_nbr

pytestmark = pytest.mark.gpu

E = 2.0 ** -53 / 3.0 ** 0.5


def _cn(rng, shape, s=1.0):
    return (rng.standard_normal(shape) + 1j * rng.standard_normal(shape)) * s


def _inputs(d, seed):
    rng = np.random.default_rng(seed)
    return dict(G=anti_hermitian_blocks(_cn(rng, d.g_shape)), Go=anti_hermitian_blocks(_cn(rng, d.g_shape)),
                D=_cn(rng, d.d_shape), Dm=_cn(rng, d.d_shape), dH=_cn(rng, d.dh_shape, 0.1), gS=_cn(rng, d.sigma_shape),
                nbr=make_nbr(rng, d.na, d.nb))


def _gpu(x):
    return {k: torch.from_numpy(np.ascontiguousarray(v)).cuda() for k, v in x.items()}


def _dg_80_bit(d, x, b, alpha):
    """dL/dG of atom b: sum over the edges into it of conj(alpha D_ij) A_i^H W A_j."""
    L = np.clongdouble
    out = np.zeros((d.nkz, d.ne, d.norb, d.norb), L)
    for a, n in zip(*np.nonzero(x["nbr"] == b)):
        A, D, g = x["dH"][a, n].astype(L), x["D"][:, :, a, n].astype(L), x["gS"][:, :, a].astype(L)
        Y = np.zeros((d.nkz, d.ne, 3, 3, d.norb, d.norb), L)
        for q in range(d.nkz):
            gq = np.roll(g, -q, axis=0)
            for w in range(1, d.nw + 1):
                W = np.zeros_like(gq)
                W[:, :d.ne - w] += gq[:, w:]
                W[:, w:] += gq[:, :d.ne - w]
                Y += np.conj(D[q, w - 1])[None, None, :, :, None, None] * W[:, :, None, None]
        T = np.einsum("irt,keijrc->kejtc", np.conj(A), Y)
        out += np.einsum("kejtc,jcu->ketu", T, A)
    return np.conj(L(alpha)) * out


@pytest.mark.parametrize("d", [Dims(nkz=5, ne=40, nqz=5, nw=6, na=24, nb=4, norb=8, g_slots=1),
                               Dims(nkz=3, ne=48, nqz=3, nw=5, na=40, nb=3, norb=6, g_slots=1)], ids=["nkz5", "nkz3"])
def test_dg_rounds_as_its_terms_do(d):
    """Chains of dG: the two products of N complex terms, the filter over 3 directions and
    2 Nw energies (added in pairs), the three directions of every in-edge, and about twelve
    single roundings of the transforms."""
    print(f"[gpu] dG accuracy dims={d.as_tuple()}", flush=True)
    x = _inputs(d, 8)
    t = _gpu(x)
    dG = sse.backward(t["G"], t["D"], t["dH"], t["nbr"], t["gS"], need=(True, False, False))[0]
    b = int(x["nbr"][0, 0])
    ref = _dg_80_bit(d, x, b, 1j)
    indeg = int((x["nbr"] == b).sum())
    bound = E * ((2 * d.norb + 6 * d.nw + 2 * d.norb + 3 * indeg) / 2 + 6) ** 0.5
    got = dG[:, :, b, 0].cpu().numpy().astype(np.clongdouble)
    err = float(np.sqrt((abs(got - ref) ** 2).sum() / (abs(ref) ** 2).sum()))
    print(f"  error {err:.3e}, bound {bound:.3e}", flush=True)
    assert err <= bound
