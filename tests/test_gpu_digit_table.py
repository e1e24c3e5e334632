"""Plans with and without the digit table of their lattice points: the level
kernels take a point's digits from the table or derive them from its rank, and
the results are the same bit for bit (plans whose sweeps would run in one
workgroup fold the gradient's sums in another order without it: equal to
rounding).  Also who holds a table and when it goes."""
import numpy as np
import pytest
import torch

from paper_2303_08879_amd import fockdiag as F

pytestmark = pytest.mark.gpu
C128, C64 = torch.complex128, torch.complex64


def dev(x, dtype):
    return torch.tensor(np.asarray(x), dtype=dtype, device="cuda")


def triple(M, b_zero):
    rng = np.random.default_rng(40 + M + b_zero)
    X = rng.standard_normal((2 * M, 2 * M)) + 1j * rng.standard_normal((2 * M, 2 * M))
    b = np.zeros(2 * M) if b_zero else 0.3 * (rng.standard_normal(2 * M) + 1j * rng.standard_normal(2 * M))
    return (X + X.T) * (0.25 / np.sqrt(4 * M)), b, 0.8 + 0.1j


def results(cut, dtype, b_zero, table, total=None):
    """rho, gradients, tangent, and rho of a batch of two."""
    print(f"[gpu digits] cut={cut} dtype={dtype} b_zero={b_zero} table={table} total={total}", flush=True)
    M = len(cut)
    mask, mode = (1 << M) - 1, "zero" if b_zero else "general"
    make = lambda m: F.Plan(cut, mask, dtype, m) if total is None else F.Plan(cut, mask, dtype, m, total_cutoff=total)
    A, b, c = triple(M, b_zero)
    A, b, c = dev(A, dtype), dev(b, dtype), dev([c], dtype)
    plan = make(mode)
    F.fd_plan_use_digit_table(plan, table)
    assert (plan.query(F.FD_Q_TABLE_BYTES) > 0) == table
    rng = np.random.default_rng(3)
    g = dev(rng.standard_normal(plan.out_shape) + 1j * rng.standard_normal(plan.out_shape), dtype)
    w, s = plan.workspace(True)
    ws, saved = (torch.empty(n, dtype=torch.uint8, device="cuda") for n in (w, s))
    rho = torch.empty(plan.out_shape, dtype=dtype, device="cuda")
    dA, db, dc = torch.empty_like(A), torch.empty_like(b), torch.empty_like(c)
    F.fock_diag_fwd(plan, A, b, c, rho, ws, saved)
    F.fock_diag_vjp(plan, A, b, c, saved, g, dA, db, dc, ws)
    out = [rho, dA, db, dc]
    if not b_zero:
        wj = torch.empty(plan.jvp_workspace(), dtype=torch.uint8, device="cuda")
        r, t = torch.empty_like(rho), torch.empty_like(rho)
        F.fock_diag_jvp(plan, A, b, c, A, b, c, r, t, wj)
        out += [r, t]
    if total is None:
        w0 = plan.workspace(False)[0]
        wss = [torch.empty(w0, dtype=torch.uint8, device="cuda") for _ in range(2)]
        rs = [torch.empty_like(rho) for _ in range(2)]
        F.fock_diag_fwd_batch([plan, plan], [A, A], [b, b], [c, c], rs, wss)
        out += rs
    torch.cuda.synchronize()
    F.fd_device_status(plan)
    return [x.cpu().numpy() for x in out]


# levels of more than 32 (bridge, 16-point tile) items: level sweeps either way, in
# tiles of 16 and of 64 points
@pytest.mark.parametrize("cut", [[33, 32, 31], [12, 11, 13, 12], [8, 7, 8, 7, 6], [7, 6, 7, 6, 5, 6], [5] * 7, [4] * 8,
                                 [20] * 5, [6] * 8])
@pytest.mark.parametrize("dtype,b_zero", [(C128, False), (C64, True)])
def test_level_sweeps_without_the_table(cut, dtype, b_zero):
    for x, r in zip(results(cut, dtype, b_zero, False), results(cut, dtype, b_zero, True)):
        assert np.array_equal(x, r)


@pytest.mark.parametrize("cut", [[64], [10, 10], [64, 64], [17, 16, 15], [5, 4, 3], [3] * 7])
@pytest.mark.parametrize("b_zero", [True, False])
def test_small_plans_without_the_table(cut, b_zero):
    got, ref = results(cut, C128, b_zero, False), results(cut, C128, b_zero, True)
    for x, r in zip(got[:1] + got[4:], ref[:1] + ref[4:]):
        assert np.array_equal(x, r)
    # gradients: at most 2^12 terms a sum in either order
    flat = lambda v: np.concatenate([y.ravel() for y in v])
    assert np.linalg.norm(flat(got[1:4]) - flat(ref[1:4])) <= 2 ** 12 * 2.0 ** -52 * np.linalg.norm(flat(ref[1:4]))


def test_plans_of_one_lattice_share_a_table():
    cut, mask = [8] * 7, (1 << 7) - 1                     # 2^21 points, 16 MiB
    A, b, c = triple(7, True)

    def first_call(dtype, mode, enable=True):
        plan = F.Plan(cut, mask, dtype, mode)
        F.fd_plan_use_digit_table(plan, enable)
        ws = torch.empty(plan.workspace(False)[0], dtype=torch.uint8, device="cuda")
        rho = torch.empty(plan.out_shape, dtype=dtype, device="cuda")
        F.fock_diag_fwd(plan, dev(A, dtype), dev(b, dtype), dev([c], dtype), rho, ws)
        torch.cuda.synchronize()
        return plan, rho.cpu().numpy()

    def free():
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        return torch.cuda.mem_get_info()[0]

    table = 8 * 8 ** 7
    first_call(C128, "zero")[0].close()                   # kernels loaded
    none, _ = first_call(C128, "zero", False)
    f0 = free()
    a, rho = first_call(C128, "zero")
    f1 = free()
    others = [first_call(C64, "zero")[0], first_call(C128, "auto")[0], first_call(C128, "general")[0]]
    f2 = free()
    assert a.query(F.FD_Q_TABLE_BYTES) == table and f0 - f1 >= table
    assert f1 - f2 < table
    a.close()                                             # the others still read it
    late, again = first_call(C128, "auto")
    assert np.array_equal(again, rho)
    for p in others + [late]:
        F.fd_plan_use_digit_table(p, False)
    assert free() >= f0 - table // 2


def test_level_sweeps_without_the_table_total_cutoff():
    for x, r in zip(results([15] * 5, C128, False, False, 14), results([15] * 5, C128, False, True, 14)):
        assert np.array_equal(x, r)


def test_batch_budget_counts_tables():
    from paper_2303_08879_amd.batching import BatchRunner
    shapes = [([6] * 5, 31), ([6] * 5, 31), ([4, 3, 3], 0b110)]
    trip = [triple(len(cut), True) for cut, _ in shapes]
    table = 8 * 6 ** 5
    r = BatchRunner(shapes, trip)
    assert r.table_bytes == table
    need = r.arena.numel()
    assert len(r.groups) == 1
    assert len(BatchRunner(shapes, trip, budget_bytes=need + table).groups) == 1
    assert len(BatchRunner(shapes, trip, budget_bytes=need + table - 1).groups) == 2
