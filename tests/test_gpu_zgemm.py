"""The FP64 matrix-core product: its tiles at ragged rows, columns and K, and the far field's rectangular form.

Tolerance: FP64 sums of K <= 17000 terms in another order, K * 2^-53 of sum |a| |b| at most; 1e-13 covers the rounding of
sums of this length many times over.
"""
import numpy as np
import pytest

import synth
from oracle import efie as oefie
from oracle import rwg

from .gpu_common import flush

torch = pytest.importorskip("torch")
P = pytest.importorskip("paper_2310_15644_amd")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


# 32 x 32 tiles of four K groups (fewer chunks than groups, K tails of 8), the 16 x 64 and the 64 x 64 tile
@pytest.mark.parametrize("n,m", [(1, 9), (7, 9), (9, 33), (33, 31), (65, 64), (1025, 33), (2113, 65), (4099, 1025), (16411, 13)])
def test_zgemm_tiles(n, m):
    flush(f"zgemm n={n} nrhs={m}")
    g = torch.Generator(device="cuda").manual_seed(n + m)
    Z = torch.randn((n, n), dtype=torch.complex128, device="cuda", generator=g)
    X = torch.randn((m, n), dtype=torch.complex128, device="cuda", generator=g)
    Y = P.zx(Z, X)
    ref = X @ Z.T.contiguous()
    bound = X.abs() @ Z.abs().T.contiguous()
    assert float(((Y - ref).abs() / bound).max()) <= 1e-13


# nrhs below nine takes the vector kernel, from nine the matrix cores
@pytest.mark.parametrize("nrhs,ndir", [(8, 5), (9, 1), (33, 16), (40, 17)])
def test_farfield_rectangular(nrhs, ndir):
    v, t = synth.ellipsoid(3, (1.0, 0.9, 1.1))
    m = rwg.build(v, t)
    dirs = synth.uniform_directions(ndir, seed=4)
    rng = np.random.default_rng(nrhs)
    J = rng.standard_normal((nrhs, m.n)) + 1j * rng.standard_normal((nrhs, m.n))
    F = P.farfield(P.Mesh(v, t).upload("cuda"), 1.7, torch.as_tensor(J, device="cuda"), dirs).cpu().numpy()
    Fo = oefie.farfield(m, 1.7, J, dirs)
    assert np.abs(F - Fo).max() <= 1e-12 * np.abs(Fo).max()
