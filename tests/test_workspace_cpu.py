"""Workspace sizes of the C entries against what the kernels write (runs without a GPU)."""
import ctypes

import pytest

from paper_1912_10024_amd import _lib
from paper_1912_10024_amd.inputs import Dims


def _bytes(d, op):
    out = ctypes.c_size_t(0)
    assert _lib.load().sse_workspace_bytes(ctypes.byref(_lib.SSEDims.of(d)), 0, op, ctypes.byref(out)) == _lib.SSE_OK
    return out.value


def _backward_rejects(d, nbytes):
    """Whether sse_backward (ddH alone) refuses a workspace of nbytes; it looks at no pointer before."""
    P = ctypes.c_void_p
    rc = _lib.load().sse_backward(ctypes.byref(_lib.SSEDims.of(d)), *([P(256)] * 4), 0.0, 1.0, P(256), None, None, P(256),
                                  P(256), nbytes, None)
    return rc == _lib.SSE_ERR_WORKSPACE


@pytest.mark.parametrize("ne", [1, 32, 192])
def test_shares_of_a_neighbour_count_beyond_the_transform_kernels(ne):
    """2^20 neighbours are more than the kernels in the momentum transform index, so the
    adjoint runs its direct kernels, which write one share of dL/d(dH) per momentum."""
    d = Dims(nkz=7, ne=ne, nqz=7, nw=10, na=1, nb=1 << 20, norb=10, g_slots=1)
    shares = 16 * d.nkz * d.na * d.nb * 3 * d.norb ** 2
    assert _bytes(d, 1) >= shares + 4 * (4 * d.na + 1 + d.na * d.nb)
    assert _backward_rejects(d, shares)


def _fast(d, op):
    out = ctypes.c_size_t(0)
    assert _lib.load().sse_fast_workspace_bytes(ctypes.byref(_lib.SSEDims.of(d)), op, ctypes.byref(out)) == _lib.SSE_OK
    return out.value


@pytest.mark.parametrize("norb,nw", [(25, 60), (12, 140)])
def test_pi_asks_for_a_workspace_wherever_its_one_window_fits(norb, nw):
    """Pi reads the energies above only; shapes where a window to both sides would not fit
    the LDS still run in the transform."""
    d = Dims(nkz=2, ne=130, nqz=2, nw=nw, na=5, nb=2, norb=norb, g_slots=1)
    assert _fast(d, 3) >= 16 * d.nkz * d.na * norb ** 2 * (2 * d.ne - 1)


@pytest.mark.parametrize("room", [1 << 40, 3 << 30, 100 << 20, 1000])
def test_a_forward_call_takes_the_room_there_is(monkeypatch, room):
    """Out of memory, the forward asks for half as much until it fits instead of falling to the
    least at once."""
    import torch

    from paper_1912_10024_amd import sse
    d = Dims(nkz=7, ne=256, nqz=7, nw=10, na=1024, nb=4, norb=10, g_slots=1)
    real, asked = torch.empty, []

    def empty(n, **kw):
        asked.append(n)
        if n > room:
            raise torch.OutOfMemoryError("no room")
        return real(min(n, 256), dtype=torch.uint8)

    monkeypatch.setattr(torch, "empty", empty)
    sse._forward_workspace(d, "fp64", "cpu")
    want = _bytes(d, 0)
    if room < 1 << 20:
        assert asked[-1] == 256
    else:
        assert asked[-1] <= room and (asked[-1] == want or 2 * asked[-1] > room // 2)
        assert asked[-1] > 256


def test_the_interface_of_the_workspaces_has_its_own_version():
    """sse_fast_workspace_bytes and sse_phonon_forward_ws, and the size that
    sse_workspace_bytes gives for the forward, came after version 6."""
    lib = _lib.load()
    assert {"sse_fast_workspace_bytes", "sse_phonon_forward_ws"} <= set(_lib.EXPORTS)
    assert lib.sse_abi_version() >= 7
