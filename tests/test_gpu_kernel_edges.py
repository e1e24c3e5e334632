"""The sweep kernels at the edges of their tiles and of the rules that choose
between them: one-workgroup sweeps against level sweeps (bitwise), reverse
against forward mode (the adjoint identity), complex64 against complex128, the
b = 0 decision inside a kernel, register-resident undetected-block rows, and the
state-vector reverse mode's items.

Tolerances: a result passes at most smax levels (<= 56 here) of sums over 2 M + 1
<= 17 terms, and the A of `contracting` has norm about 1/2, so errors do not grow along
the levels: 56 * 17 * 4 eps = 8.5e-13 in double precision (bound used: 1e-11 of
the sum of the absolute products), 4.5e-4 at worst and, as roundings are
independent, about its square root's share, 1e-5, in single precision."""
import numpy as np
import pytest
import torch

import oracle as O
from parity import assert_close, assert_grad_close
from paper_2303_08879_amd import fockdiag as F

pytestmark = pytest.mark.gpu


def contracting(rng, D, b_zero):
    X = rng.standard_normal((D, D)) + 1j * rng.standard_normal((D, D))
    X = (X + X.T) * (0.25 / np.sqrt(2 * D))
    b = np.zeros(D, complex) if b_zero else 0.3 * (rng.standard_normal(D) + 1j * rng.standard_normal(D))
    return X, b, 0.8 + 0.1j


def dev(x, dtype):
    return torch.tensor(np.asarray(x), dtype=dtype, device="cuda")


def grad(cut, mask, dtype, A, b, c, g, b_mode, every=0):
    """rho and (dA, db, dc) of a plan, checkpointed every `every` levels."""
    print(f"[gpu edges] cut={cut} mask={bin(mask)} dtype={dtype} b_mode={b_mode} every={every}", flush=True)
    plan = F.Plan(cut, mask, dtype, b_mode)
    F.fd_plan_set_checkpoint(plan, every)
    At, bt, ct = dev(A, dtype), dev(b, dtype), dev([c], dtype)
    wsb, svb = plan.workspace(True)
    ws = torch.empty(wsb, dtype=torch.uint8, device="cuda")
    saved = torch.empty(svb, dtype=torch.uint8, device="cuda")
    rho = torch.empty(plan.out_shape, dtype=dtype, device="cuda")
    dA, db, dc = torch.empty_like(At), torch.empty_like(bt), torch.empty_like(ct)
    F.fock_diag_fwd(plan, At, bt, ct, rho, ws, saved)
    F.fock_diag_vjp(plan, At, bt, ct, saved, dev(g, dtype), dA, db, dc, ws)
    torch.cuda.synchronize()
    F.fd_device_status(plan)
    return rho.cpu().numpy(), dA.cpu().numpy(), db.cpu().numpy(), dc.cpu().numpy()


# every detected-mode count, levels that end inside a tile of 16 points, plans
# on both sides of the one-workgroup limits, levels with and without a workgroup
# per tile, the largest levels in tiles of 64 points (six of cutoff 8: not; eight of cutoff 6)
POINTS = [[64], [2], [10, 10], [33, 16], [9, 8, 7], [17, 16, 15], [7, 6, 7, 5], [12, 11, 13, 12], [5, 4, 5, 3, 6],
          [8, 7, 8, 7, 6], [4, 4, 3, 4, 5, 4], [8, 8, 8, 8, 8, 8], [4, 3, 3, 4, 3, 4, 3], [5] * 7, [4] * 8, [6] * 8]
# blocks of undetected modes: row counts around the 16-row tiles, ragged chunks
BLOCKS = [([3, 4, 3], 0b110), ([9, 5, 4], 0b110), ([12, 3, 4, 3, 2], 0b11110), ([17, 4, 3, 3], 0b1110),
          ([23, 3, 2, 3, 2, 2], 0b111110), ([33, 7], 0b10), ([3, 4, 5, 4], 0b1100), ([4, 5, 3, 2, 3], 0b11100)]
SHAPES = [(cut, (1 << len(cut)) - 1) for cut in POINTS] + BLOCKS


@pytest.mark.parametrize("b_zero", [True, False])
@pytest.mark.parametrize("cut,mask", SHAPES)
def test_sweeps_agree(cut, mask, b_zero):
    M = len(cut)
    rng = np.random.default_rng(900 + 31 * M + sum(cut) + b_zero)
    A, b, c = contracting(rng, 2 * M, b_zero)
    mode = "zero" if b_zero else "general"
    c128, c64 = torch.complex128, torch.complex64
    shape = F.Plan(cut, mask, c128, mode).out_shape
    g = rng.standard_normal(shape) + 1j * rng.standard_normal(shape)
    rho, *d = grad(cut, mask, c128, A, b, c, g, mode)
    # level sweeps (every checkpointed forward): the same values and gradients
    for x, r in zip(grad(cut, mask, c128, A, b, c, g, mode, every=3), (rho, *d)):
        assert np.array_equal(x, r)
    # <g, J t> = <J^T g, t>; with b = 0 the gradient of b at even outputs is zero
    tA = rng.standard_normal((2 * M, 2 * M)) + 1j * rng.standard_normal((2 * M, 2 * M))
    tb = np.zeros(2 * M) if b_zero else rng.standard_normal(2 * M) + 1j * rng.standard_normal(2 * M)
    tc = complex(rng.standard_normal(), rng.standard_normal())
    plan = F.Plan(cut, mask, c128, "general")
    ws = torch.empty(plan.jvp_workspace(), dtype=torch.uint8, device="cuda")
    r2, t2 = (torch.empty(plan.out_shape, dtype=c128, device="cuda") for _ in range(2))
    F.fock_diag_jvp(plan, dev(A, c128), dev(b, c128), dev([c], c128), dev(tA, c128), dev(tb, c128), dev([tc], c128), r2,
                    t2, ws)
    t2 = t2.cpu().numpy()
    lhs = np.sum(np.conj(g) * t2)
    rhs = np.sum(tA * np.conj(d[0])) + np.sum(tb * np.conj(d[1])) + tc * np.conj(d[2][0])
    assert abs(lhs - rhs) <= 1e-11 * np.sum(np.abs(g) * np.abs(t2))
    # complex64
    low = grad(cut, mask, c64, A, b, c, g, mode)
    flat = lambda v: np.concatenate([np.asarray(x).ravel() for x in v]).astype(np.complex128)
    assert np.linalg.norm(low[0] - rho) <= 1e-5 * np.linalg.norm(rho)
    assert np.linalg.norm(flat(low[1:]) - flat(d)) <= 1e-5 * np.linalg.norm(flat(d))


# one-workgroup sweeps decide on b in the kernel, level sweeps on the host
@pytest.mark.parametrize("cut,mask", [([5, 4], 0b11), ([12, 11, 13, 12], 0b1111), ([5, 4], 0b10)])
@pytest.mark.parametrize("last", [0.0, -0.0, 1e-200])
def test_auto_decides_on_b(cut, mask, last):
    D = 2 * len(cut)
    rng = np.random.default_rng(77)
    A, b, c = contracting(rng, D, True)
    b[-1] = last
    shape = F.Plan(cut, mask, torch.complex128, "auto").out_shape
    g = rng.standard_normal(shape) + 1j * rng.standard_normal(shape)
    got = grad(cut, mask, torch.complex128, A, b, c, g, "auto")
    # a plan with undetected modes sweeps every level either way
    ref = grad(cut, mask, torch.complex128, A, b, c, g, "zero" if last == 0 and mask == (1 << len(cut)) - 1 else "general")
    for x, r in zip(got, ref):
        assert np.array_equal(x, r)


@pytest.mark.parametrize("cut", [[2, 3], [3, 3], [16, 2], [33, 2], [64, 2]])
def test_undetected_rows(cut):
    # the block of one undetected mode, its rows in registers
    rng = np.random.default_rng(sum(cut))
    A, b, c = contracting(rng, 4, False)
    shape = F.Plan(cut, 0b10, torch.complex128, "general").out_shape
    g = rng.standard_normal(shape) + 1j * rng.standard_normal(shape)
    rho, dA, db, dc = grad(cut, 0b10, torch.complex128, A, b, c, g, "general")
    assert_close(rho, O.fock_diag(A, b, c, cut, 0b10), label=f"rows {cut}")
    ref = O.fock_diag_vjp(A, b, c, cut, 0b10, g)
    assert_grad_close((dA, db, complex(dc[0])), ref, label=f"rows {cut}")


# sums in one wavefront and split over two (six and more modes), tiles that are
# not whole wavefronts, a last chunk that is short
STATES = [[1, 1], [64], [64, 33], [40, 37], [13, 9, 8], [5, 4, 3, 6, 2], [4, 3, 5, 2, 3, 4], [3, 4, 2, 3, 2, 3, 3], [4] * 8]


def state_vjp(cut, c, psi, g, dtype):
    print(f"[gpu edges] state vjp cut={cut} dtype={dtype}", flush=True)
    M = len(cut)
    plan = F.StatePlan(cut, dtype, "general")
    ws = torch.empty(plan.vjp_workspace(), dtype=torch.uint8, device="cuda")
    dA = torch.empty((M, M), dtype=dtype, device="cuda")
    db, dc = torch.empty(M, dtype=dtype, device="cuda"), torch.empty(1, dtype=dtype, device="cuda")
    F.fock_state_vjp(plan, dev([c], dtype), dev(psi, dtype), dev(g, dtype), dA, db, dc, ws)
    torch.cuda.synchronize()
    return dA.cpu().numpy(), db.cpu().numpy(), dc.cpu().numpy()


@pytest.mark.parametrize("cut", STATES)
@pytest.mark.parametrize("dtype,tol", [(torch.complex128, 1e-10), (torch.complex64, 1e-5)])
def test_state_reverse_items(cut, dtype, tol):
    M = len(cut)
    rng = np.random.default_rng(sum(cut))
    A, b, c = contracting(rng, M, False)
    psi = O.state_vector(A, b, c, cut)
    g = rng.standard_normal(cut) + 1j * rng.standard_normal(cut)
    rA, rb, rc = O.adjoint_closed_form(A, b, c, psi, g)
    flat = lambda v: np.concatenate([np.asarray(x).ravel() for x in v]).astype(np.complex128)
    got, ref = flat(state_vjp(cut, c, psi, g, dtype)), flat((rA, rb, [rc]))
    assert np.linalg.norm(got - ref) <= tol * np.linalg.norm(ref)


@pytest.mark.parametrize("cut", [[5], [6, 5, 4], [3, 4, 2, 3, 2, 3, 3]])
def test_state_reverse_leaves_out_absent_products(cut):
    # the last amplitude has no entry above it and the first none below: neither
    # an infinite amplitude there nor an infinite cotangent here reaches dA and db
    rng = np.random.default_rng(len(cut))
    psi = rng.standard_normal(cut) + 1j * rng.standard_normal(cut)
    g = rng.standard_normal(cut) + 1j * rng.standard_normal(cut)
    psi.flat[-1] = g.flat[0] = 0
    dA, db, _ = state_vjp(cut, 0.7 - 0.2j, psi, g, torch.complex128)
    psi.flat[-1] = np.inf
    g.flat[0] = complex(np.inf, np.nan)
    iA, ib, ic = state_vjp(cut, 0.7 - 0.2j, psi, g, torch.complex128)
    for x, r in ((iA, dA), (ib, db)):   # (two compilations of the same sums)
        assert np.linalg.norm(x - r) <= 1e-12 * np.linalg.norm(r)
    assert not np.isfinite(ic[0])
