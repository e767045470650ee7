"""The direct fp64 kernels (Sigma, Pi and the gradients term by term), which run where the
window of frequencies does not fit the LDS of the kernels in the momentum transform, against
the CPU oracle.

The tolerance is the repository's fp64 bar of 1e-12: an output sums at most
2 * nkz * nw * nb * 9 * norb^2 products, and a chain of that many rounded additions of
random terms stays below 1e-13 at these sizes."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import oracle
from paper_1912_10024_amd import _lib, sse
from paper_1912_10024_amd.inputs import Dims, anti_hermitian_blocks, make_nbr

pytestmark = pytest.mark.gpu

TOL = 1e-12
SIGMA = Dims(nkz=2, ne=24, nqz=2, nw=40, na=3, nb=1, norb=32, g_slots=2)
PI = Dims(nkz=2, ne=16, nqz=2, nw=120, na=3, nb=2, norb=25, g_slots=1)
ADJOINT = Dims(nkz=2, ne=20, nqz=2, nw=100, na=4, nb=2, norb=16, g_slots=2)


def _cn(rng, shape, s=1.0):
    return (rng.standard_normal(shape) + 1j * rng.standard_normal(shape)) * s


def _inputs(d, seed):
    rng = np.random.default_rng(seed)
    return dict(G=anti_hermitian_blocks(_cn(rng, d.g_shape)), Go=_cn(rng, d.g_shape), D=_cn(rng, d.d_shape),
                Dm=_cn(rng, d.d_shape), dH=_cn(rng, d.dh_shape, 0.1), B=_cn(rng, d.dh_shape, 0.1),
                gS=_cn(rng, d.sigma_shape), nbr=make_nbr(rng, d.na, d.nb))


def _gpu(x):
    return {k: torch.from_numpy(v).cuda() for k, v in x.items()}


def _rel(a, b):
    return np.linalg.norm(a.cpu().numpy() - b) / np.linalg.norm(b)


def _asks(name, d, *args):
    out = ctypes.c_size_t(0)
    assert getattr(_lib.load(), name)(ctypes.byref(_lib.SSEDims.of(d)), *args, ctypes.byref(out)) == _lib.SSE_OK
    return out.value


def test_the_shapes_have_no_transform_kernel():
    """Those kernels would ask for room for their transforms at a larger number of energies."""
    large = lambda d: d.replace(ne=2000)
    assert _asks("sse_workspace_bytes", large(SIGMA), 0, 0) == 256
    assert _asks("sse_fast_workspace_bytes", large(PI), 3) == 0
    assert _asks("sse_fast_workspace_bytes", large(ADJOINT), 1) == _asks("sse_workspace_bytes", large(ADJOINT), 0, 1)


@pytest.mark.parametrize("two", [False, True], ids=["one_table", "two_tables"])
@pytest.mark.parametrize("stored", [False, True], ids=["hermitian", "stored"])
def test_sigma(two, stored):
    print(f"[gpu] direct sigma two={two} stored={stored}", flush=True)
    d = SIGMA
    x = _inputs(d, 1)
    t = _gpu(x)
    S = sse.forward_ex(t["G"], t["D"], t["dH"], t["nbr"], Dm=t["Dm"] if two else None, dHba=t["B"] if stored else None)
    right = x["B"] if stored else np.conj(np.swapaxes(x["dH"], -1, -2))
    ref = oracle.sse_forward_ex(d, x["G"], x["D"], x["Dm"] if two else x["D"], x["dH"], np.ascontiguousarray(right), x["nbr"])
    assert _rel(S, ref) <= TOL


def test_pi():
    print("[gpu] direct pi", flush=True)
    d = PI
    x = _inputs(d, 2)
    t = _gpu(x)
    P = sse.phonon_forward(t["G"], t["Go"], t["dH"], t["nbr"], d.nqz, d.nw)
    assert _rel(P, oracle.pse_forward(d, x["G"], x["Go"], x["dH"], x["nbr"])) <= TOL


@pytest.mark.parametrize("signed", [False, True], ids=["one_table", "two_tables"])
def test_gradients(signed):
    print(f"[gpu] direct adjoint signed={signed}", flush=True)
    d = ADJOINT
    x = _inputs(d, 3)
    t = _gpu(x)
    if signed:
        got = sse.backward_signed(t["G"], t["D"], t["Dm"], t["dH"], t["nbr"], t["gS"])
        ref = oracle.sse_backward_signed(d, x["G"], x["D"], x["Dm"], x["dH"], x["nbr"], x["gS"])
    else:
        got = sse.backward(t["G"], t["D"], t["dH"], t["nbr"], t["gS"])
        ref = oracle.sse_backward(d, x["G"], x["D"], x["dH"], x["nbr"], x["gS"])
    for g, r in zip(got, ref):
        if np.linalg.norm(r):
            assert _rel(g, r) <= TOL


def test_gradients_alone():
    """Each gradient by itself: what a call needs of the workspace differs."""
    print("[gpu] direct adjoint, one gradient at a time", flush=True)
    d = ADJOINT
    t = _gpu(_inputs(d, 4))
    full = sse.backward(t["G"], t["D"], t["dH"], t["nbr"], t["gS"])
    for i in range(3):
        got = sse.backward(t["G"], t["D"], t["dH"], t["nbr"], t["gS"], need=tuple(j == i for j in range(3)))
        assert torch.equal(got[i], full[i])
