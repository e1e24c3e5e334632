"""Length of the summation chains of the state-vector reverse mode.

With psi = 1 and g = x everywhere and c = 1, cbar is N x exactly (N = 2^25 entries),
and every term and partial sum is positive, so the relative error is at most n u,
u = 2^-53, for n additions between a term and the result.  The kernel adds 16
entries in a lane, 6 steps over the lanes, the compensated sum of these folds (2
u whatever their number), 4 wavefronts, 2 slots of a final thread and 8 steps of its
tree: n = 38.  x is chosen against a longer chain: 1 + 2^-45 less half an ulp loses its
last bits in each of the additions to a partial sum of 256 to 512, 2^-46 of the result =
128 u."""
import numpy as np
import pytest
import torch

from paper_2303_08879_amd import fockdiag as F

pytestmark = pytest.mark.gpu


def test_state_reverse_chain_length():
    cut, dtype = [8] * 7 + [16], torch.complex128
    M, N = len(cut), 8 ** 7 * 16
    x = 1.0 + 2.0 ** -45 - 2.0 ** -52
    plan = F.StatePlan(cut, dtype, "general")
    ws = torch.empty(plan.vjp_workspace(), dtype=torch.uint8, device="cuda")
    psi = torch.ones(cut, dtype=dtype, device="cuda")
    g = torch.full(cut, x, dtype=dtype, device="cuda")
    c = torch.ones(1, dtype=dtype, device="cuda")
    dA = torch.empty((M, M), dtype=dtype, device="cuda")
    db, dc = torch.empty(M, dtype=dtype, device="cuda"), torch.empty(1, dtype=dtype, device="cuda")
    F.fock_state_vjp(plan, c, psi, g, dA, db, dc, ws)
    got = np.longdouble(dc.cpu().numpy()[0].real)
    err = abs(got - np.longdouble(x) * N) / (np.longdouble(x) * N)
    print(f"[state sums] relative error {float(err):.2e} = {float(err) * 2 ** 53:.1f} u", flush=True)
    assert err <= 38 * 2.0 ** -53
