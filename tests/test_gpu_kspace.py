"""fp64 kernels in the momentum transform: Sigma at shapes where tiles, chunks of
rows, passes of columns and the transform itself have remainders, against the CPU
oracle; the same bits from every workspace size; non-finite coefficients.

The tolerance is the repository's fp64 bar of 1e-12.  It is wide for this route:
an output sums at most 2 * 3 * Nw * Nb * (Norb + 9) products through two products with
grad H, a filter and two transforms, whose relative rounding error is below
(number of terms in a chain) * 2^-53, under 1e-13 at these sizes."""
import numpy as np
import pytest
import torch

from oracle import oracle
from paper_1912_10024_amd import sse
from paper_1912_10024_amd.inputs import Dims, anti_hermitian_blocks, make_nbr

pytestmark = pytest.mark.gpu

TOL = 1e-12
# (dims, seed); all above 1024 output blocks, so the transform route runs for nkz > 1
SHAPES = [
    (Dims(nkz=7, ne=45, nqz=7, nw=10, na=5, nb=4, norb=10, g_slots=2), 1),   # the mid grids, ragged tile of energies
    (Dims(nkz=2, ne=150, nqz=2, nw=3, na=5, nb=3, norb=7, g_slots=1), 2),    # chunk of rows with a remainder
    (Dims(nkz=3, ne=131, nqz=3, nw=1, na=4, nb=1, norb=4, g_slots=1), 3),    # one frequency, one neighbour
    (Dims(nkz=5, ne=70, nqz=5, nw=6, na=4, nb=2, norb=11, g_slots=1), 4),    # odd norb, passes of 4 over 11
    (Dims(nkz=1, ne=350, nqz=1, nw=4, na=3, nb=2, norb=5, g_slots=1), 5),    # one momentum: the direct sum
    (Dims(nkz=9, ne=40, nqz=9, nw=5, na=4, nb=2, norb=3, g_slots=2), 6),     # any-nkz transform, norb below a pass
    (Dims(nkz=2, ne=180, nqz=2, nw=2, na=3, nb=2, norb=32, g_slots=1), 7),   # largest norb
    (Dims(nkz=3, ne=90, nqz=3, nw=33, na=4, nb=2, norb=6, g_slots=1), 8),    # a wide window of frequencies
    (Dims(nkz=4, ne=6, nqz=4, nw=9, na=45, nb=2, norb=8, g_slots=1), 9),     # fewer energies than frequencies
    (Dims(nkz=2, ne=600, nqz=2, nw=2, na=2, nb=1, norb=1, g_slots=1), 10),   # single entries
]
IDS = ["x".join(map(str, d.as_tuple())) for d, _ in SHAPES]


def _cn(rng, shape, s=1.0):
    return (rng.standard_normal(shape) + 1j * rng.standard_normal(shape)) * s


def _inputs(d, seed):
    rng = np.random.default_rng(seed)
    return dict(G=anti_hermitian_blocks(_cn(rng, d.g_shape)), D=_cn(rng, d.d_shape), Dm=_cn(rng, d.d_shape),
                dH=_cn(rng, d.dh_shape, 0.1), B=_cn(rng, d.dh_shape, 0.1), nbr=make_nbr(rng, d.na, d.nb))


def _gpu(x):
    return {k: torch.from_numpy(v).cuda() for k, v in x.items()}


def _rel(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


@pytest.mark.parametrize("d,seed", SHAPES, ids=IDS)
def test_sigma_matches_the_oracle(d, seed):
    print(f"[gpu] kspace sigma dims={d.as_tuple()}", flush=True)
    x = _inputs(d, seed)
    t = _gpu(x)
    S = sse.forward(t["G"], t["D"], t["dH"], t["nbr"], alpha=0.3 + 0.7j).cpu().numpy()
    assert _rel(S, oracle.sse_forward(d, x["G"], x["D"], x["dH"], x["nbr"], alpha=0.3 + 0.7j)) <= TOL
    S = sse.forward_signed(t["G"], t["D"], t["Dm"], t["dH"], t["nbr"]).cpu().numpy()
    assert _rel(S, oracle.sse_forward_signed(d, x["G"], x["D"], x["Dm"], x["dH"], x["nbr"])) <= TOL


@pytest.mark.parametrize("two", [False, True], ids=["one_table", "two_tables"])
@pytest.mark.parametrize("d,seed", [SHAPES[1], SHAPES[4]], ids=[IDS[1], IDS[4]])
def test_sigma_with_a_stored_right_factor(d, seed, two):
    print(f"[gpu] kspace stored factor dims={d.as_tuple()} two={two}", flush=True)
    x = _inputs(d, seed)
    t = _gpu(x)
    S = sse.forward_ex(t["G"], t["D"], t["dH"], t["nbr"], Dm=t["Dm"] if two else None, dHba=t["B"]).cpu().numpy()
    ref = oracle.sse_forward_ex(d, x["G"], x["D"], x["Dm"] if two else x["D"], x["dH"], x["B"], x["nbr"])
    assert _rel(S, ref) <= TOL


def test_every_workspace_gives_the_same_bits():
    """Room for the whole transform, for a slab of energies (a ragged last one), and
    for nothing: the same sums in the same order."""
    d, seed = SHAPES[0]
    d = d.replace(ne=150)
    print(f"[gpu] kspace workspaces dims={d.as_tuple()}", flush=True)
    t = _gpu(_inputs(d, seed))
    args = (t["G"], t["D"], t["dH"], t["nbr"])
    full = sse.forward(*args)
    per = 16 * d.nkz * d.na * d.norb ** 2
    for energies in (150, 101, 80, 2):
        ws = torch.empty(max(256, per * energies), dtype=torch.uint8, device="cuda")
        assert torch.equal(sse.forward(*args, ws=ws), full), energies


def test_atoms_without_valid_neighbours_and_a_bad_entry():
    d, seed = SHAPES[1]
    print(f"[gpu] kspace bad neighbours dims={d.as_tuple()}", flush=True)
    x = _inputs(d, seed)
    x["nbr"][2] = -1
    x["nbr"][3, 1] = d.na
    t = _gpu(x)
    x["D"][:, :, 2] = 0
    x["D"][:, :, 3, 1] = 0
    t["D"][:, :, 2] = float("nan")      # coefficients of an edge without a neighbour are not read
    x["nbr"] = np.where((x["nbr"] < 0) | (x["nbr"] >= d.na), 0, x["nbr"])   # the oracle's own entries stay in range
    S = sse.forward(t["G"], t["D"], t["dH"], t["nbr"]).cpu().numpy()
    ref = oracle.sse_forward(d, x["G"], x["D"], x["dH"], x["nbr"].astype(np.int32))
    assert np.array_equal(S[:, :, 2], np.zeros_like(S[:, :, 2]))
    assert _rel(S, ref) <= TOL


@pytest.mark.parametrize("two", [False, True], ids=["one_table", "two_tables"])
def test_a_coefficient_that_is_not_finite_stays_with_its_terms(two):
    """An infinite coefficient at frequency w reaches the energies that have a term
    with it and no others."""
    d = Dims(nkz=3, ne=90, nqz=3, nw=60, na=4, nb=2, norb=2, g_slots=1)
    print(f"[gpu] kspace non-finite coefficient dims={d.as_tuple()} two={two}", flush=True)
    t = _gpu(_inputs(d, 12))
    w = 55
    if two:
        t["Dm"][1, w - 1, 1, 0, 2, 0] = float("inf")   # terms with G at E + w
        S = sse.forward_signed(t["G"], t["D"], t["Dm"], t["dH"], t["nbr"])
        hit = [e for e in range(d.ne) if e + w < d.ne]
    else:
        t["D"][1, w - 1, 1, 0, 2, 0] = float("inf")
        S = sse.forward(t["G"], t["D"], t["dH"], t["nbr"])
        hit = [e for e in range(d.ne) if e + w < d.ne or e - w >= 0]
    ok = torch.isfinite(torch.view_as_real(S)).all(-1).all(-1).all(-1).all(0)   # [ne, na]
    want = torch.ones_like(ok)
    want[hit, 1] = False
    assert torch.equal(ok, want)


def test_problems_of_a_thousand_blocks_keep_exact_sums():
    """At most 1024 output blocks: integer-valued inputs give integers exactly (the sum
    over momenta as it stands), on a shape without a matrix-core instance."""
    d = Dims(nkz=4, ne=32, nqz=4, nw=3, na=8, nb=2, norb=6, g_slots=1)
    print(f"[gpu] kspace exact sums dims={d.as_tuple()}", flush=True)
    rng = np.random.default_rng(3)
    ints = lambda shape: (rng.integers(-3, 4, shape) + 1j * rng.integers(-3, 4, shape)).astype(np.complex128)
    x = dict(G=ints(d.g_shape), D=ints(d.d_shape), dH=ints(d.dh_shape), nbr=make_nbr(rng, d.na, d.nb))
    t = _gpu(x)
    S = sse.forward(t["G"], t["D"], t["dH"], t["nbr"], alpha=1.0).cpu().numpy()
    assert np.array_equal(S, oracle.sse_forward(d, x["G"], x["D"], x["dH"], x["nbr"], alpha=1.0))


# ------------------------------------------------------------------ Pi
PI_SHAPES = [s for i, s in enumerate(SHAPES) if i not in (6,)] + [
    (Dims(nkz=2, ne=180, nqz=2, nw=3, na=3, nb=2, norb=25, g_slots=1), 7),   # the largest norb Pi takes
    (Dims(nkz=7, ne=61, nqz=7, nw=10, na=4, nb=3, norb=10, g_slots=2), 13),
    (Dims(nkz=3, ne=100, nqz=3, nw=7, na=4, nb=2, norb=9, g_slots=1), 14),   # blocks of 4 over 7 frequencies
]


@pytest.mark.parametrize("d,seed", PI_SHAPES, ids=["x".join(map(str, d.as_tuple())) for d, _ in PI_SHAPES])
def test_pi_matches_the_oracle(d, seed):
    print(f"[gpu] kspace pi dims={d.as_tuple()}", flush=True)
    rng = np.random.default_rng(seed + 100)
    x = _inputs(d, seed)
    x["Go"] = _cn(rng, d.g_shape)
    x["nbr"][1, 0] = d.na + 2
    t = _gpu(x)
    P = sse.phonon_forward(t["G"], t["Go"], t["dH"], t["nbr"], d.nqz, d.nw, beta=0.2 - 0.9j).cpu().numpy()
    x["nbr"][1, 0] = 0
    ref = oracle.pse_forward(d, x["G"], x["Go"], x["dH"], x["nbr"], beta=0.2 - 0.9j)
    assert np.array_equal(P[:, :, 1, 0], np.zeros_like(P[:, :, 1, 0]))
    ref[:, :, 1, 0] = 0
    assert _rel(P, ref) <= TOL


def _pi_ws(t, d, nbytes):
    """Pi through the C entry with a workspace of nbytes."""
    import ctypes

    from paper_1912_10024_amd import _lib
    out = torch.full(d.d_shape, complex(float("nan"), float("nan")), dtype=torch.complex128, device="cuda")
    ws = torch.empty(max(nbytes, 1), dtype=torch.uint8, device="cuda")
    P = lambda v: ctypes.c_void_p(v.data_ptr())
    rc = _lib.load().sse_phonon_forward_ws(ctypes.byref(_lib.SSEDims.of(d)), P(t["G"]), P(t["Go"]), P(t["dH"]), P(t["nbr"]),
                                           0.0, -1.0, P(out), P(ws), nbytes, ctypes.c_void_p(0))
    torch.cuda.synchronize()
    assert rc == 0
    return out.cpu().numpy()


def test_pi_workspaces():
    d = Dims(nkz=3, ne=140, nqz=3, nw=6, na=5, nb=2, norb=6, g_slots=1)
    print(f"[gpu] kspace pi workspaces dims={d.as_tuple()}", flush=True)
    x = _inputs(d, 3)
    x["Go"] = _cn(np.random.default_rng(4), d.g_shape)
    t = _gpu(x)
    ref = oracle.pse_forward(d, x["G"], x["Go"], x["dH"], x["nbr"])
    per = 16 * d.nkz * d.na * d.norb ** 2
    whole = _pi_ws(t, d, per * 2 * d.ne)
    assert _rel(whole, ref) <= TOL
    assert np.array_equal(_pi_ws(t, d, 0), whole)
    for energies in (279, 200, 120):
        assert _rel(_pi_ws(t, d, per * energies), ref) <= TOL, energies


def test_pi_block_that_is_not_finite_stays_with_its_terms():
    """A non-finite block of Go at energy E reaches the frequencies with E + w on the grid."""
    d = Dims(nkz=2, ne=150, nqz=2, nw=12, na=4, nb=1, norb=3, g_slots=1)
    print(f"[gpu] kspace pi non-finite dims={d.as_tuple()}", flush=True)
    x = _inputs(d, 5)
    x["Go"] = _cn(np.random.default_rng(6), d.g_shape)
    b = int(x["nbr"][2, 0])
    x["Go"][1, d.ne - 4, b, 0, 1, 1] = np.inf
    t = _gpu(x)
    P = sse.phonon_forward(t["G"], t["Go"], t["dH"], t["nbr"], d.nqz, d.nw)
    ok = torch.isfinite(torch.view_as_real(P)).all(-1).all(-1).all(-1).all(0).cpu()   # [nw, na, nb]
    for a in range(d.na):
        hit = int(x["nbr"][a, 0]) == b
        assert ok[3:, a].all()
        assert bool(ok[:3, a].any()) != hit


# ------------------------------------------------------------------ the adjoint
ADJ_SHAPES = [s for i, s in enumerate(SHAPES) if i not in (6,)] + [
    (Dims(nkz=2, ne=130, nqz=2, nw=3, na=5, nb=2, norb=16, g_slots=2), 15),  # the largest norb the adjoint takes
]


def _grads(d, seed):
    x = _inputs(d, seed)
    x["gS"] = _cn(np.random.default_rng(seed + 77), d.sigma_shape)
    return x


@pytest.mark.parametrize("d,seed", ADJ_SHAPES, ids=["x".join(map(str, d.as_tuple())) for d, _ in ADJ_SHAPES])
def test_adjoint_matches_the_oracle(d, seed):
    print(f"[gpu] kspace adjoint dims={d.as_tuple()}", flush=True)
    x = _grads(d, seed)
    t = _gpu(x)
    alpha = -0.4 + 0.8j
    got = sse.backward(t["G"], t["D"], t["dH"], t["nbr"], t["gS"], alpha=alpha)
    ref = oracle.sse_backward(d, x["G"], x["D"], x["dH"], x["nbr"], x["gS"], alpha=alpha)
    for name, g, r in zip(("dG", "dD", "ddH"), got, ref):
        assert _rel(g.cpu().numpy(), r) <= TOL, name
    got = sse.backward_signed(t["G"], t["D"], t["Dm"], t["dH"], t["nbr"], t["gS"], alpha=alpha)
    ref = oracle.sse_backward_signed(d, x["G"], x["D"], x["Dm"], x["dH"], x["nbr"], x["gS"], alpha=alpha)
    for name, g, r in zip(("dG", "dDp", "dDm", "ddH"), got, ref):
        assert _rel(g.cpu().numpy(), r) <= TOL, name


@pytest.mark.parametrize("d,seed", [SHAPES[0], SHAPES[1]], ids=IDS[:2])
def test_adjoint_with_every_workspace_gives_the_same_bits(d, seed):
    """Both transforms in the workspace, that of dSigma alone, or neither."""
    import ctypes

    from paper_1912_10024_amd import _lib
    print(f"[gpu] kspace adjoint workspaces dims={d.as_tuple()}", flush=True)
    t = _gpu(_grads(d, seed))
    full = sse.backward(t["G"], t["D"], t["dH"], t["nbr"], t["gS"])
    need = ctypes.c_size_t(0)
    assert _lib.load().sse_workspace_bytes(ctypes.byref(_lib.SSEDims.of(d)), 0, 1, ctypes.byref(need)) == 0
    hat = 16 * d.nkz * d.ne * d.na * d.norb ** 2 + 256
    for nbytes in (need.value, need.value + hat, need.value + 2 * hat):
        ws = torch.full((nbytes,), 255, dtype=torch.uint8, device="cuda")
        for a, b in zip(sse.backward(t["G"], t["D"], t["dH"], t["nbr"], t["gS"], ws=ws), full):
            assert torch.equal(a, b), nbytes
    got = sse.backward_noalloc(t["G"], t["D"], t["dH"], t["nbr"], t["gS"], dG=torch.empty_like(full[0]),
                               dD=torch.empty_like(full[1]), ddH=torch.empty_like(full[2]))
    for a, b in zip(got, full):
        assert torch.equal(a, b)


@pytest.mark.parametrize("na,nb", [(2, 1), (1025, 3), (4096, 16), (4097, 2)], ids=["two", "odd", "largest_small", "large"])
def test_adjoint_adjacency_at_the_edges_of_its_kernels(na, nb):
    """The reverse adjacency in one launch (up to 4096 atoms and 65536 edges) and in
    several, with atoms that no edge points at and one that many point at."""
    d = Dims(nkz=2, ne=2, nqz=2, nw=1, na=na, nb=nb, norb=1, g_slots=1)
    print(f"[gpu] kspace adjacency dims={d.as_tuple()}", flush=True)
    x = _grads(d, 21)
    if na > 2:
        x["nbr"][: na // 4, 0] = na - 1
    t = _gpu(x)
    got = sse.backward(t["G"], t["D"], t["dH"], t["nbr"], t["gS"])
    ref = oracle.sse_backward(d, x["G"], x["D"], x["dH"], x["nbr"], x["gS"])
    for name, g, r in zip(("dG", "dD", "ddH"), got, ref):
        assert _rel(g.cpu().numpy(), r) <= TOL, name


def test_pi_and_dd_with_a_ragged_last_group_of_frequencies():
    """More frequency blocks than the lanes of a workgroup hold: several workgroups per
    (edge, momentum), the last of them with fewer blocks."""
    d = Dims(nkz=2, ne=44, nqz=2, nw=31, na=12, nb=2, norb=25, g_slots=1)
    print(f"[gpu] kspace pi groups dims={d.as_tuple()}", flush=True)
    x = _inputs(d, 31)
    x["Go"] = _cn(np.random.default_rng(32), d.g_shape)
    t = _gpu(x)
    P = sse.phonon_forward(t["G"], t["Go"], t["dH"], t["nbr"], d.nqz, d.nw).cpu().numpy()
    assert _rel(P, oracle.pse_forward(d, x["G"], x["Go"], x["dH"], x["nbr"])) <= TOL
    d = Dims(nkz=2, ne=60, nqz=2, nw=41, na=9, nb=2, norb=16, g_slots=1)
    print(f"[gpu] kspace adjoint groups dims={d.as_tuple()}", flush=True)
    x = _grads(d, 33)
    t = _gpu(x)
    got = sse.backward(t["G"], t["D"], t["dH"], t["nbr"], t["gS"])
    ref = oracle.sse_backward(d, x["G"], x["D"], x["dH"], x["nbr"], x["gS"])
    for name, g, r in zip(("dG", "dD", "ddH"), got, ref):
        assert _rel(g.cpu().numpy(), r) <= TOL, name


def test_pi_where_only_one_window_fits():
    """A shape whose window to both sides does not fit the LDS: Pi, with the workspace it
    asks for and without one."""
    d = Dims(nkz=2, ne=130, nqz=2, nw=60, na=5, nb=1, norb=25, g_slots=1)
    print(f"[gpu] kspace pi wide dims={d.as_tuple()}", flush=True)
    x = _inputs(d, 41)
    x["Go"] = _cn(np.random.default_rng(42), d.g_shape)
    t = _gpu(x)
    ref = oracle.pse_forward(d, x["G"], x["Go"], x["dH"], x["nbr"])
    assert _rel(sse.phonon_forward(t["G"], t["Go"], t["dH"], t["nbr"], d.nqz, d.nw).cpu().numpy(), ref) <= TOL
    assert _rel(_pi_ws(t, d, 0), ref) <= TOL


def test_more_workgroups_than_one_launch_takes():
    """A launch holds at most 2^32 work-items.  Over a million atoms with four neighbours
    need more for Pi and dD (2^23 workgroups of 512) and for d gradH (2^24 of 256); sampled
    atoms against the oracle on their own neighbourhood."""
    d = Dims(nkz=2, ne=2, nqz=2, nw=1, na=1100000, nb=8, norb=1, g_slots=1)
    print(f"[gpu] kspace many atoms dims={d.as_tuple()}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    cn = lambda shape: torch.view_as_complex(torch.randn((*shape, 2), generator=gen, dtype=torch.float64, device="cuda"))
    t = dict(G=cn(d.g_shape), Go=cn(d.g_shape), D=cn(d.d_shape), dH=cn(d.dh_shape), gS=cn(d.sigma_shape))
    step = torch.tensor([1, 2, 5, 17, 1000, 40001, 333333, 700001], device="cuda")
    t["nbr"] = ((torch.arange(d.na, device="cuda")[:, None] + step[None]) % d.na).to(torch.int32).contiguous()
    P = sse.phonon_forward(t["G"], t["Go"], t["dH"], t["nbr"], d.nqz, d.nw)
    grads = sse.backward(t["G"], t["D"], t["dH"], t["nbr"], t["gS"])
    for a in (0, 7, d.na // 2, d.na - 1):
        # the atom and its neighbours as a structure of their own: its edges alone have terms
        atoms = [a] + t["nbr"][a].tolist()
        own = {k: t[k][:, :, atoms].cpu().numpy().copy() for k in ("G", "Go", "D", "gS")}
        own["dH"] = t["dH"][atoms].cpu().numpy().copy()
        own["gS"][:, :, 1:] = 0
        e = d.replace(na=len(atoms))
        nbr = np.tile(np.arange(1, d.nb + 1, dtype=np.int32), (len(atoms), 1))
        ref = oracle.pse_forward(e, own["G"], own["Go"], own["dH"], nbr)
        assert _rel(P[:, :, a].cpu().numpy(), ref[:, :, 0]) <= TOL
        _, rD, rH = oracle.sse_backward(e, own["G"], own["D"], own["dH"], nbr, own["gS"])
        assert _rel(grads[1][:, :, a].cpu().numpy(), rD[:, :, 0]) <= TOL
        assert _rel(grads[2][a].cpu().numpy(), rH[0]) <= TOL


def test_more_workgroups_than_one_launch_takes_in_half_precision():
    """The same for the 16-bit forward, whose workgroups (norb per atom, of 512) pass 2^32
    work-items at two million atoms of four orbitals; against the fp64 form there."""
    d = Dims(nkz=3, ne=3, nqz=3, nw=2, na=2110000, nb=4, norb=4, g_slots=1)
    print(f"[gpu] 16-bit many atoms dims={d.as_tuple()}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(6)

    def cn(shape):
        x = torch.empty(shape, dtype=torch.complex128, device="cuda")
        torch.view_as_real(x).normal_(generator=gen)
        return x

    G, D, dH = cn(d.g_shape), cn(d.d_shape), cn(d.dh_shape)
    step = torch.tensor([1, 2, 1000, 700001], device="cuda")
    nbr = ((torch.arange(d.na, device="cuda")[:, None] + step[None]) % d.na).to(torch.int32).contiguous()
    out = torch.full(d.sigma_shape, complex(float("nan"), float("nan")), dtype=torch.complex128, device="cuda")
    S = sse.forward(G, D, dH, nbr, precision="fp16x2", out=out)
    ref = sse.forward(G, D, dH, nbr)
    for a in (0, 1055000, 2097151, 2097152, d.na - 1):
        err = (S[:, :, a] - ref[:, :, a]).abs().norm() / ref[:, :, a].abs().norm()
        assert float(err) <= 1e-5, (a, float(err))   # fp16x2 carries about 22 bits; unwritten is NaN


@pytest.mark.parametrize("dims", [(4, 32, 3, 8, 2, 6), (3, 16, 2, 16, 4, 4), (1, 200, 4, 7, 3, 5), (7, 13, 10, 5, 4, 10),
                                  (7, 4, 10, 36, 4, 10)],
                         ids=lambda v: "x".join(map(str, v)))
def test_gradients_of_a_thousand_blocks_keep_exact_sums(dims):
    """At most 1024 blocks: integer-valued inputs give integer gradients exactly, for one
    coefficient table and for two."""
    nkz, ne, nw, na, nb, norb = dims
    d = Dims(nkz=nkz, ne=ne, nqz=nkz, nw=nw, na=na, nb=nb, norb=norb, g_slots=2)
    print(f"[gpu] kspace exact gradients dims={d.as_tuple()}", flush=True)
    rng = np.random.default_rng(9)
    ints = lambda shape: (rng.integers(-3, 4, shape) + 1j * rng.integers(-3, 4, shape)).astype(np.complex128)
    x = dict(G=ints(d.g_shape), D=ints(d.d_shape), Dm=ints(d.d_shape), dH=ints(d.dh_shape), gS=ints(d.sigma_shape),
             nbr=make_nbr(rng, d.na, d.nb))
    t = _gpu(x)
    got = sse.backward(t["G"], t["D"], t["dH"], t["nbr"], t["gS"], alpha=1.0)
    ref = oracle.sse_backward(d, x["G"], x["D"], x["dH"], x["nbr"], x["gS"], alpha=1.0)
    for name, g, r in zip(("dG", "dD", "ddH"), got, ref):
        assert np.array_equal(g.cpu().numpy(), r), name
    got = sse.backward_signed(t["G"], t["D"], t["Dm"], t["dH"], t["nbr"], t["gS"], alpha=1.0)
    ref = oracle.sse_backward_signed(d, x["G"], x["D"], x["Dm"], x["dH"], x["nbr"], x["gS"], alpha=1.0)
    for name, g, r in zip(("dG", "dDp", "dDm", "ddH"), got, ref):
        assert np.array_equal(g.cpu().numpy(), r), name
