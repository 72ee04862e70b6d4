"""The tile edges of the assembly: orders on both sides of each rule, ragged last tiles, real and complex k.

Tolerances as for every assembly: max |dZ| <= 1e-11 max |Z| in FP64 (rounding order), 2e-5 in complex64 (FP32 phase and
distance).
"""
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
