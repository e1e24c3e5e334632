"""The reverse mode's limit on the undetected block belongs to the interface: no
plan with a detected mode is refused (rows that do not fit the LDS are streamed),
and without one the limit does not move with the LDS of a kernel that such plans
never launch."""
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2303_08879_amd", "csrc")

# (c64, undetected cutoffs): the largest of their kind that are taken, and the next one
TAKEN = [(0, [7, 10]), (0, [14, 7]), (0, [19, 6]), (1, [7, 14]), (1, [14, 10]), (1, [17, 9]), (1, [22, 8]),
         (1, [3, 3, 6]), (1, [3, 6, 3]), (1, [5, 2, 7]), (1, [5, 7, 2]), (0, [64]), (1, [64]), (0, [2, 2]),
         (0, [4, 3, 3])]
REFUSED = [(0, [7, 11]), (0, [14, 8]), (0, [19, 7]), (1, [7, 15]), (1, [14, 11]), (1, [17, 10]), (1, [22, 9]),
           (1, [3, 3, 7]), (1, [5, 2, 8]), (0, [4, 3, 4]), (1, [4, 4, 5])]


@pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir("/opt/rocm/include"),
                    reason="needs g++ and the ROCm headers")
def test_blocks_taken_and_refused(tmp_path):
    exe = str(tmp_path / "limits")
    cmd = ["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
           "-I" + os.path.join(ROOT, "include"), "-I" + CSRC, os.path.join(CSRC, "planner.cpp"),
           os.path.join(ROOT, "tests", "host_sanitize", "block_limits.cpp"), "-o", exe,
           "-L/opt/rocm/lib", "-lamdhip64", "-Wl,-rpath,/opt/rocm/lib"]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-3000:]
    cases, want = [], []
    for dt, cu in TAKEN + REFUSED:
        cases.append((dt, cu, []))
        want.append(int((dt, cu) in TAKEN))
        for cd in ([2], [3, 2], [2] * 6):
            cases.append((dt, cu, cd))
            want.append(1)
    text = "".join(" ".join(map(str, [dt, len(cu), len(cd), *cu, *cd])) + "\n" for dt, cu, cd in cases)
    r = subprocess.run([exe], input=text, capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, (r.returncode, r.stderr[-2000:])
    got = [int(x) for x in r.stdout.split()]
    assert [(c, g) for c, g, w in zip(cases, got, want) if g != w] == [] and len(got) == len(want)


@pytest.mark.gpu
@pytest.mark.parametrize("cutoffs,name", [([7, 10], "complex128"), ([19, 6], "complex128"), ([22, 8], "complex64"),
                                          ([3, 3, 6], "complex64")])
def test_largest_blocks_without_detected_modes(cutoffs, name):
    """Gradients against the oracle's closed-form adjoint.  A cotangent passes through
    at most sum(2 (C - 1)) steps of the fill, each a rounding of a few eps of terms that
    decay, then one sum over the block: 1e-10 in complex128 as for every gradient here,
    2e-5 in complex64 (168 eps: four for each of the at most 42 steps of [22, 8] or 22 of
    [3, 3, 6])."""
    import torch
    import oracle as O
    from paper_2303_08879_amd import fockdiag as F
    dt = getattr(torch, name)
    rng = np.random.default_rng(11)
    M = len(cutoffs)
    X = rng.standard_normal((2 * M, 2 * M)) + 1j * rng.standard_normal((2 * M, 2 * M))
    A = (X + X.T) * (0.3 / np.sqrt(8 * M))
    b = 0.3 * (rng.standard_normal(2 * M) + 1j * rng.standard_normal(2 * M))
    plan = F.Plan(cutoffs, 0, dt, "general")
    g = rng.standard_normal(plan.out_shape) + 1j * rng.standard_normal(plan.out_shape)
    t = [torch.tensor(x, dtype=dt, device="cuda") for x in (A, b, np.array([0.8 + 0.1j]), g)]
    ref = O.fock_diag_vjp(*[x.cpu().numpy().astype(complex) for x in t[:2]], complex(t[2].item()), cutoffs, 0,
                          t[3].cpu().numpy().astype(complex))
    w, s = plan.workspace(True)
    ws = torch.empty(max(w, 256), dtype=torch.uint8, device="cuda")
    sv = torch.empty(max(s, 256), dtype=torch.uint8, device="cuda")
    rho = torch.empty(plan.out_shape, dtype=dt, device="cuda")
    d = [torch.empty_like(x) for x in t[:3]]
    F.fock_diag_fwd(plan, *t[:3], rho, ws, sv)
    F.fock_diag_vjp(plan, *t[:3], sv, t[3], *d, ws)
    torch.cuda.synchronize()
    tol = 1e-10 if dt == torch.complex128 else 2e-5
    for x, y in zip(d, ref):
        assert O.rel_err(x.cpu().numpy().ravel(), np.ravel(y)) <= tol
