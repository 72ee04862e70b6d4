"""The fp16 split product: every tile of its rule at ragged rows, unknowns and K, badly scaled and special values.

Tolerance: both operands are within 2^-23 of the stored values in each part and l l' is below 2^-22 of a product, so that
sum |z| |x| 2^-21 bounds the error of a complex output before the FP32 sums of at most 64 terms, whose roundings (three
products of sixteen terms each, 12 per 64 terms and part) add less than 2^-20 of it: 3e-6 of sum |z| |x|.
"""
import ctypes

import numpy as np
import pytest

from .gpu_common import flush

torch = pytest.importorskip("torch")
P = pytest.importorskip("paper_2310_15644_amd")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def split():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    v = [t[2] for t in P.gemm_variants()].index(64)
    prev = P.gemm_select(False, v), P.gemm_select(True, v)
    yield v
    P.gemm_select(False, prev[0])
    P.gemm_select(True, prev[1])


def operands(n, m, seed, spread):
    rng = np.random.default_rng(seed)
    Z = rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n))
    X = rng.standard_normal((m, n)) + 1j * rng.standard_normal((m, n))
    # rows (and parts of rows) of very different magnitude
    Z *= 10.0 ** rng.uniform(-spread, spread, (n, 1)) * 10.0 ** rng.uniform(-2, 2, (n, n))
    X *= 10.0 ** rng.uniform(-spread, spread, (m, 1)) * 10.0 ** rng.uniform(-2, 2, (m, n))
    return (torch.as_tensor(Z, device="cuda").to(torch.complex64), torch.as_tensor(X, device="cuda").to(torch.complex64))


# one block of 32 x 32 and its neighbours, K tails of 16, 32 and 64 terms, the four tiles of the rule
@pytest.mark.parametrize("n,m", [(1, 2), (15, 9), (31, 33), (33, 32), (63, 31), (64, 64), (65, 65), (129, 2), (1025, 97),
                                 (8230, 20), (4097, 40), (4130, 130)])
def test_split_tiles(split, n, m):
    flush(f"split product n={n} nrhs={m}")
    Z, X = operands(n, m, 31 * n + m, 8.0)
    Zd, Xd = Z.to(torch.complex128), X.to(torch.complex128)
    ref = Xd @ Zd.T.contiguous()
    bound = Xd.abs() @ Zd.abs().T.contiguous()
    for Y in (P.zx(Z, X).to(torch.complex128), P.zx_flush64(Z, Xd)):
        assert float(((Y - ref).abs() / bound).max()) <= 3e-6


# ranges of K: one chunk more than one, tails of a chunk, the three tiles on both sides of their lines (32 right-hand
# sides, order 2048), rows of Y past 64 and 128
@pytest.mark.parametrize("n,m", [(65, 33), (129, 2), (129, 64), (191, 129), (2048, 32), (2049, 32), (2050, 33), (4317, 45)])
def test_split_ranges(split, n, m):
    flush(f"split product over ranges of K n={n} nrhs={m}")
    nb = ctypes.c_size_t()
    assert P.lib().efie_zx_workspace_size(n, m, P.C64, ctypes.byref(nb)) == 0 and nb.value > 0
    Z, X = operands(n, m, 17 * n + m, 8.0)
    Zd, Xd = Z.to(torch.complex128), X.to(torch.complex128)
    bound = Xd.abs() @ Zd.abs().T.contiguous()
    Y = P.zx(Z, X)
    assert float(((Y.to(torch.complex128) - Xd @ Zd.T.contiguous()).abs() / bound).max()) <= 3e-6
    assert torch.equal(torch.view_as_real(Y), torch.view_as_real(P.zx(Z, X)))   # a fixed order of the sums
    # a workspace one byte short: the product of the call without one
    ptr = [ctypes.c_void_p(t.data_ptr()) for t in (Z, X)]
    ws, outs = torch.empty(nb.value, dtype=torch.uint8, device="cuda"), []
    for w, b in ((None, 0), (ctypes.c_void_p(ws.data_ptr()), nb.value - 1)):
        outs.append(torch.empty_like(X))
        assert P.lib().efie_zx_ws(ptr[0], P.C64, n, ptr[1], ctypes.c_void_p(outs[-1].data_ptr()), m, w, b, None) == 0
    outs.append(torch.empty_like(X))
    assert P.lib().efie_zx(ptr[0], P.C64, n, ptr[1], ctypes.c_void_p(outs[-1].data_ptr()), m, None) == 0
    torch.cuda.synchronize()
    assert all(torch.equal(torch.view_as_real(o), torch.view_as_real(outs[0])) for o in outs[1:])


def test_split_special_values(split):
    n, m = 200, 40
    Z, X = operands(n, m, 5, 0.0)
    X[3] = 0.0                       # a zero row
    X[5, 64:128] = 0.0               # a zero chunk
    X[7, 150] = float("inf")
    X[9, 10] = float("nan")
    Z[:, 17] *= 1e-30
    Z[11] = 1e-38 * Z[11]            # near the smallest normal numbers
    Y = P.zx(Z, X)
    assert bool((Y[3] == 0).all())
    for r in (7, 9):
        assert not bool(torch.isfinite(Y[r].abs()).any())
    keep = [r for r in range(m) if r not in (7, 9)]
    Xd, Zd = X[keep].to(torch.complex128), Z.to(torch.complex128)
    bound = Xd.abs() @ Zd.abs().T.contiguous() + 1e-36
    assert float(((Y[keep].to(torch.complex128) - Xd @ Zd.T.contiguous()).abs() / bound).max()) <= 3e-6


def wide_operands(n, m, kind, seed):
    """Rows whose chunks hold values of very different size, the large ones against zeros: errors of the large ones' size
    would stand out.  zero_x / zero_z: values over 24 decades against a matrix of mostly zeros; one: a single 1e9 in every
    chunk of Z against zeros of X; noise: 1e-17 where X would be zero; parts: Z with real parts ten decades below, X real."""
    rng = np.random.default_rng(seed)
    Z = rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n))
    X = rng.standard_normal((m, n)) + 1j * rng.standard_normal((m, n))
    if kind == "zero_x":
        Z *= 10.0 ** rng.uniform(-12, 12, (n, n))
        X *= rng.random((m, n)) < 0.1
    elif kind == "zero_z":
        X *= 10.0 ** rng.uniform(-12, 12, (m, n))
        Z *= rng.random((n, n)) < 0.1
    elif kind == "one":
        Z[:, 7::32] *= 1e9
        X[:, 7::32] = 0.0
    elif kind == "noise":
        Z[:, 7::32] *= 1e9
        Z[:, 9::32] *= 1e-9
        X[:, 7::32] *= 1e-17
    else:
        Z = 1e-10 * Z.real + 1j * Z.imag
        X = X.real + 0j
    return (torch.as_tensor(Z, device="cuda").to(torch.complex64), torch.as_tensor(X, device="cuda").to(torch.complex64))


# the four tiles in the block and the three over ranges of K, ragged rows, unknowns and K.  A chunk that the two parts do
# not hold takes FP32 products: 128 terms of a part, 2^-24 each of the partial sum at most, 8e-6 of sum |z| |x| (of each
# part's own terms for "parts"), and the split bound above elsewhere.
@pytest.mark.parametrize("kind", ["zero_x", "zero_z", "one", "noise", "parts"])
@pytest.mark.parametrize("n,m", [(33, 32), (65, 65), (129, 2), (1025, 97), (2050, 33), (4097, 40), (8230, 20)])
def test_split_wide_range(split, n, m, kind):
    Z, X = wide_operands(n, m, kind, 13 * n + m)
    Zd, Xd = Z.to(torch.complex128), X.to(torch.complex128)
    ref = Xd @ Zd.T.contiguous()
    if kind == "parts":
        bound = torch.complex(Xd.real.abs() @ Zd.real.abs().T.contiguous(), Xd.real.abs() @ Zd.imag.abs().T.contiguous())
        ratio = lambda e: max(float((e.real.abs() / bound.real).max()), float((e.imag.abs() / bound.imag).max()))
    else:
        bound = Xd.abs() @ Zd.abs().T.contiguous()
        ratio = lambda e: float((e.abs() / bound.clamp(min=1e-300)).max())
    for Y in (P.zx(Z, X).to(torch.complex128), P.zx_flush64(Z, Xd)):
        err = ratio(Y - ref)
        flush(f"split product of wide rows {kind} n={n} nrhs={m}: {err:.1e}")
        assert err <= 8e-6
