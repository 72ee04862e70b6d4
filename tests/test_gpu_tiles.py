"""The tile edges of the assembly: orders on both sides of each rule, ragged last tiles, real and complex k.

Tolerances as for every assembly: max |dZ| <= 1e-11 max |Z| in FP64 (rounding order), 2e-5 in complex64 (FP32 phase and
distance).
"""
import ctypes

import numpy as np
import pytest

import synth
from oracle import calderon as ocal
from oracle import efie as oefie
from oracle import rwg

from .gpu_common import flush

torch = pytest.importorskip("torch")
P = pytest.importorskip("paper_2310_15644_amd")

pytestmark = pytest.mark.gpu


# N = 30 f^2: 30, 270 and 750 take 16-wide tiles, 1080 and 3000 32-wide ones, 3630 the 64-wide ones
@pytest.mark.parametrize("f", [1, 3, 5, 6, 10, 11])
@pytest.mark.parametrize("dt,tol", [("c128", 1e-11), ("c64", 2e-5)])
def test_tile_edges_sampled_rows(f, dt, tol):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    v, t = synth.ellipsoid(f, (1.0, 0.9, 1.15))
    m = rwg.build(v, t)
    mesh = P.Mesh(v, t).upload("cuda")
    rows = sorted({0, 15, 16, 31, min(32, m.n - 1), m.n // 2, m.n - 1} & set(range(m.n)))
    for k in (0.7, ocal.ktilde(1.4)):
        flush(f"tiles N={m.n} {dt} k={k}")
        Z = P.assemble(mesh, k, dtype=dt)
        assert bool((Z == Z.T).all())
        Zo = oefie.z_rows(m, k, rows)
        assert np.abs(Z[rows].cpu().numpy() - Zo).max() <= tol * np.abs(Zo).max()


# The complex128 assembly by pair rows (P.assemble) against the tiles (the workspace of the near blocks only): T = 20, 80
# and 500 triangles (parts of a block of 256 sources, one test triangle per block), 2000 and 2880 (four per block), every
# tile edge; triangles in random order (stored transposed), the far rule, complex k.  The same values are added in the same
# order, so the matrices are equal bit for bit.
@pytest.mark.parametrize("f,shuffle,far,k", [(1, False, 0.0, 0.7), (2, True, 0.0, 0.7 - 0.1j), (5, True, 4.0, 2.0),
                                             (5, False, 0.0, 0.1), (10, True, 0.0, 1.5), (12, False, 3.0, 1.0 - 0.2j)])
def test_pair_rows_equal_tiles(f, shuffle, far, k):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    v, t = synth.ellipsoid(f, (1.0, 0.9, 1.15))
    if shuffle:
        t = t[np.random.default_rng(f).permutation(len(t))]
    mesh = P.Mesh(v, t).upload("cuda")
    mesh.set_far_rule(far)
    flush(f"pair rows against tiles N={mesh.n} shuffle={shuffle} far={far} k={k}")
    lo, full, rows = ctypes.c_size_t(), ctypes.c_size_t(), ctypes.c_size_t()
    L = P.lib()
    assert L.efie_assemble_workspace_size(mesh._h, P.C128, ctypes.byref(lo), ctypes.byref(full)) == 0
    assert L.efie_assemble_pairs_workspace_size(mesh._h, P.C128, ctypes.byref(rows)) == 0
    assert rows.value == 64 * mesh.n**2
    out = []
    k = complex(k)
    for nb in (full.value, rows.value):
        ws = torch.full((nb,), 0xFF, dtype=torch.uint8, device="cuda")   # NaN where nothing is written
        Z = torch.empty((mesh.n, mesh.n), dtype=torch.complex128, device="cuda")
        assert L.efie_assemble_ws(mesh._h, k.real, k.imag, P.ETA0, P.C128, ctypes.c_void_p(Z.data_ptr()),
                                  ctypes.c_void_p(ws.data_ptr()), nb, None) == 0
        torch.cuda.synchronize()
        out.append(Z)
    assert torch.equal(torch.view_as_real(out[0]), torch.view_as_real(out[1]))
    assert torch.equal(out[1], out[1].T)
    assert torch.equal(out[1], P.assemble(mesh, k))
