"""Excitation and radiation matrix with eight directions per block (many directions, a ragged last group, orders on both
sides of a block of 256 RWGs) against one direction per block (few directions per call).

Tolerance: both evaluate the same values; a phase of at most 2 k max |r| rounds by 2^-52 of itself, and a value sums 14
points: 1e-13 of the largest value for k max |r| = 10.
"""
import numpy as np
import pytest

import synth

from .gpu_common import flush

torch = pytest.importorskip("torch")
P = pytest.importorskip("paper_2310_15644_amd")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("f,ndir", [(2, 4099), (3, 2050), (4, 2055)])
def test_direction_groups(f, ndir):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    v, t = synth.ellipsoid(f, (1.0, 0.8, 1.25))
    mesh = P.Mesh(v, t).upload("cuda")
    k = 8.0
    flush(f"plane waves N={mesh.n} directions={ndir}")
    dirs = synth.uniform_directions(ndir, seed=f)
    pol = np.cross(dirs, [0.3, -0.5, 0.8])
    V = P.excite_planewave(mesh, k, dirs, pol)
    rng = np.random.default_rng(f)
    J = torch.as_tensor(rng.standard_normal((2, mesh.n)) + 1j * rng.standard_normal((2, mesh.n)), device="cuda")
    F = P.farfield(mesh, k, J, dirs)
    for a in range(0, ndir, 500):
        b = min(ndir, a + 500)
        W = P.excite_planewave(mesh, k, dirs[a:b], pol[a:b])
        assert float((W - V[a:b]).abs().max()) <= 1e-13 * float(V.abs().max())
        E = P.farfield(mesh, k, J, dirs[a:b])
        assert float((E - F[:, a:b]).abs().max()) <= 1e-13 * mesh.n * float(F.abs().max())
