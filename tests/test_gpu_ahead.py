"""Solves of few columns, whose iterations are enqueued ahead of the convergence test: orders around the borders of the
step's register forms (512 to 4096 per block), columns that stop at different steps, step limits that cut a group short.

Tolerance: diagonally dominant matrices of condition number below 4 (Gershgorin), so a residual of 1e-10 leaves at most
4e-10 of the solution.
"""
import numpy as np
import pytest

from .gpu_common import flush

torch = pytest.importorskip("torch")
P = pytest.importorskip("paper_2310_15644_amd")

pytestmark = pytest.mark.gpu


def system(n, m, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    A = torch.randn((n, n), dtype=torch.complex128, device="cuda", generator=g)
    A = (A + A.T) * (0.25 / (2.0 * n ** 0.5))      # spectral radius about 0.35
    Z = (A + torch.eye(n, device="cuda")).contiguous()
    V = torch.randn((m, n), dtype=torch.complex128, device="cuda", generator=g)
    V[0] = 0.0
    if m > 1:
        V[1] = 0.0
        V[1, 3] = 1.0
    return Z, V


@pytest.mark.parametrize("n", [5, 511, 512, 513, 1025, 2048, 2049, 4096, 4097])
@pytest.mark.parametrize("solver", ["cocg", "cgs"])
def test_ahead_orders(n, solver):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    flush(f"ahead n={n} {solver}")
    s = P.COCG if solver == "cocg" else P.CGS
    Z, V = system(n, 4, n)
    J, st = P.solve(Z, V, solver=s, tol=1e-10, maxit=400)
    assert st.code == 0 and np.all(st.status == 0) and np.all(st.relres_true <= 2e-10)
    assert st.iters[0] == 0 and not bool(J[0].any())
    ref = torch.linalg.solve(Z, V[1:].T.contiguous()).T
    assert float((J[1:] - ref).norm() / ref.norm()) <= 4e-10
    # a column's steps do not depend on its neighbours (one at a time, and cut short)
    for c in (1, 3):
        J1, s1 = P.solve(Z, V[c:c + 1].contiguous(), solver=s, tol=1e-10, maxit=400)
        assert abs(int(s1.iters[0]) - int(st.iters[c])) <= 1
    for maxit in (1, 16, 17):
        _, sc = P.solve(Z, V, solver=s, tol=1e-300, maxit=maxit)
        assert sc.code == 1 and int(sc.iters[3]) == maxit


@pytest.mark.parametrize("solver,n", [("cocg", 9001), ("cgs", 9001), ("cgs", 25001)])
def test_ahead_large_orders(solver, n):
    """Orders whose groups are shorter (13, 6 and one iteration: n^2 x 16 bytes once or twice an iteration against
    16 GiB), columns that stop at different steps, and limits on both sides of a group."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    flush(f"ahead n={n} {solver}")
    s = P.COCG if solver == "cocg" else P.CGS
    Z, V = system(n, 3, n)
    J, st = P.solve(Z, V, solver=s, tol=1e-10, maxit=400)
    assert st.code == 0 and np.all(st.status == 0) and np.all(st.relres_true <= 2e-10) and st.iters[0] == 0
    R = V - J @ Z      # Z is symmetric
    assert float((R.norm(dim=1) / V.norm(dim=1).clamp(min=1.0)).max()) <= 4e-10
    J1, s1 = P.solve(Z, V[2:].contiguous(), solver=s, tol=1e-10, maxit=400)
    assert abs(int(s1.iters[0]) - int(st.iters[2])) <= 1
    for maxit in (1, 6, 7, 13, 14):
        _, sc = P.solve(Z, V, solver=s, tol=1e-300, maxit=maxit)
        assert sc.code == 1 and int(sc.iters[2]) == maxit
