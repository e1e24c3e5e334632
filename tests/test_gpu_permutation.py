"""The permutations between output and node order where a thread starts to take
several elements (2^20): outputs of a box plan against those of a plan with a
total photon cutoff that keeps every level, which come in node order without a
permutation; gradients with the cotangent permuted on the host."""
import numpy as np
import pytest
import torch

import test_gpu_kernel_edges as E
from paper_2303_08879_amd import fockdiag as F

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cut", [[32, 32, 32, 32], [33, 32, 32, 31], [7, 5, 6], [4]])
def test_permutations_against_node_order(cut):
    M, dtype = len(cut), torch.complex128
    print(f"[gpu permutation] cut={cut}", flush=True)
    rng = np.random.default_rng(sum(cut))
    A, b, c = (E.dev(x, dtype) for x in (lambda t: (t[0], t[1], [t[2]]))(E.contracting(rng, 2 * M, True)))
    order = np.argsort(np.indices(cut).sum(0).ravel(), kind="stable")   # level by level, C order within
    g = rng.standard_normal(cut) + 1j * rng.standard_normal(cut)
    out = []
    for total, cot in ((None, g), (sum(cut) - M, g.ravel()[order])):
        plan = F.Plan(cut, (1 << M) - 1, dtype, "zero", total_cutoff=total)
        w, s = plan.workspace(True)
        ws, saved = (torch.empty(n, dtype=torch.uint8, device="cuda") for n in (w, s))
        rho = torch.empty(plan.out_shape, dtype=dtype, device="cuda")
        dA, db, dc = torch.empty_like(A), torch.empty_like(b), torch.empty_like(c)
        F.fock_diag_fwd(plan, A, b, c, rho, ws, saved)
        F.fock_diag_vjp(plan, A, b, c, saved, E.dev(cot, dtype), dA, db, dc, ws)
        torch.cuda.synchronize()
        out.append([x.cpu().numpy().ravel() for x in (rho, dA, dc)])
    assert np.array_equal(out[0][0][order], out[1][0])
    for x, r in zip(out[0][1:], out[1][1:]):
        assert np.linalg.norm(x - r) <= 1e-12 * np.linalg.norm(r)
