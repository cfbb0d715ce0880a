"""Every specialised size in both precisions, 16 to 512: the kernels of each plan launched
once in each role (single and chained evaluations, full and compact outputs, first stages
kept, the step adjoint) on a state with every mode non-zero.

Against the size-generic passes, tolerances as in test_gpu_size_passes.py (relative L2: FP64
1e-12; FP32 1e-5 for the nonlinear term and the step adjoint, 3e-6 after two steps), but 4e-8
n for the FP32 term beyond 250: the terms of a white state cancel, each side is 1.5e-8 n
from the FP64 one.  Bit for bit: steps of one call and calls of one step, a step that keeps its first stage, and
the adjoint with that stage and without.
"""

import pytest

from test_size_plans import SIZES

STAGE_SIZES = [64, 128, 144, 160, 192, 216, 240, 256, 270, 324, 360, 384, 512]
CASES = sorted([(n, "fp32") for n in STAGE_SIZES]
               + [(n, "fp32" if t == "float" else "fp64") for t, n, _, _, _ in SIZES])


def test_every_size_is_here():
    smooth = [n for n in range(16, 513, 2) if 2 ** 9 * 3 ** 6 * 5 ** 4 % n == 0]
    assert CASES == sorted((n, p) for n in smooth for p in ("fp32", "fp64"))


def _fields(n, prec, count):
    """White states (not solenoidal), Hermitian on the k_z = 0 plane."""
    import torch
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(n)
    out = []
    for _ in range(count):
        u = torch.randn(3, n, n, n // 2 + 1, device="cuda:0", generator=gen,
                        dtype=torch.complex64 if prec == "fp32" else torch.complex128)
        u *= n ** -1.5
        p = u[..., 0]
        u[..., 0] = 0.5 * (p + torch.roll(torch.flip(p, (1, 2)), (1, 1), (1, 2)).conj())
        out.append(u)
    return out


def _rel(a, b):
    import torch
    return float(torch.linalg.vector_norm(torch.view_as_real(a - b)) / torch.linalg.vector_norm(torch.view_as_real(b)))


@pytest.mark.gpu
@pytest.mark.parametrize("n,prec", CASES)
def test_size(n, prec):
    import torch
    from paper_2603_08892_amd import ns
    print(f"[every size] n={n} {prec}", flush=True)
    tol_nl, tol_step = (max(1e-5, 4e-8 * n), 3e-6) if prec == "fp32" else (1e-12, 1e-12)
    fast = ns.Solver(n, 0.01, 0.95, precision=prec)
    gen = ns.Solver(n, 0.01, 0.95, precision=prec, generic=True)
    u, lam = _fields(n, prec, 2)
    dt = 0.25 / n
    al = [[0.4, 0.15, 0.9], [0.7, 0.3, 0.05]]
    assert _rel(fast.nonlinear(u, shift=al[0]), gen.nonlinear(u, shift=al[0])) <= tol_nl
    # two steps of a call: against the generic passes, and bit for bit against two calls
    for scheme in ("rk4", "random", "exact"):
        both, single, other = u.clone(), u.clone(), u.clone()
        if scheme == "rk4":
            fast.step_rk4(both, dt, 2)
            gen.step_rk4(other, dt, 2)
            for i in range(2):
                fast.step_rk4(single, dt, 1, step0=i)
        else:
            sh = al if scheme == "random" else None
            fast.step_ps(both, dt, 2, scheme, alphas=sh)
            gen.step_ps(other, dt, 2, scheme, alphas=sh)
            for i in range(2):
                fast.step_ps(single, dt, 1, scheme, alphas=sh and [sh[i]], step0=i)
        assert torch.equal(both, single), scheme
        assert _rel(both, other) <= tol_step, scheme
        del both, single, other
    # a step that keeps its first stage, and the adjoint with it
    plain, kept, s1 = u.clone(), u.clone(), fast.empty()
    fast.step_ps(plain, dt, 1, "random", alphas=al[:1])
    fast.step_ps(kept, dt, 1, "random", alphas=al[:1], stage1=s1)
    assert torch.equal(plain, kept)
    del plain, kept
    a = fast.vjp_ps(u, lam.clone(), dt, "random", alpha=al[0])
    b = fast.vjp_ps(u, lam.clone(), dt, "random", alpha=al[0], stage1=s1)
    assert torch.equal(a, b)
    assert _rel(a, gen.vjp_ps(u, lam.clone(), dt, "random", alpha=al[0])) <= tol_nl
    a = fast.vjp_ps(u, lam.clone(), dt, "exact")
    assert _rel(a, gen.vjp_ps(u, lam.clone(), dt, "exact")) <= tol_nl
