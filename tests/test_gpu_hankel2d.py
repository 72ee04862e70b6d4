"""The 2-D kernel's ranges of |kappa| R and every Gauss rule: few nodes (segments longer than a wavelength, wrapped
tiles), tiny and large wavenumbers, real and complex, against the oracle.

Tolerance as for the other operator tests: 1e-11 of the largest entry (the oracle's Hankel functions are good to 1e-13).
"""
import numpy as np
import pytest

import synth
from oracle import bie2d as ob

from .gpu_common import flush, rel_max

torch = pytest.importorskip("torch")
P = pytest.importorskip("paper_2310_15644_amd")

pytestmark = pytest.mark.gpu


# |kappa| R from 1e-5 to about 160: the power series, the four polynomial ranges and their borders
@pytest.mark.parametrize("n,q", [(8, 4), (9, 2), (16, 3), (17, 5), (31, 8), (46, 6)])
@pytest.mark.parametrize("k", [1e-3, 0.9, 3.7, 16.0, 75.0])
def test_contour_ranges(n, q, k):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    nodes, circ = synth.contour_ellipse(n), synth.contour_circle(n)
    h = P.Bie2d(nodes, circ, q=q, device="cuda")
    c = ob.Contour(nodes)
    for kap in (complex(k), complex(k, -0.4 * k), complex(k, -3.0 * k)):
        flush(f"contour n={n} q={q} kappa={kap}")
        got = [t.cpu().numpy() for t in h.assemble(kap)]
        for a, b in zip(got, ob.assemble(c, kap, q)):
            assert rel_max(a, b) <= 1e-11


# Square windows of more than 512 tiles (the triangle of tiles, mirrored): the whole curve (first and last nodes are
# neighbours), ragged last tiles, a window inside the curve, every Gauss rule; against the window one column short, which
# evaluates every tile.  Tolerance: 64 products of a pair in another order, cancelling by at most 1e2 in N: 64 x 1e2 x 2^-53.
@pytest.mark.parametrize("n,q,r0,r1", [(345, 2, 0, 345), (361, 3, 0, 361), (360, 4, 0, 360), (347, 5, 0, 347),
                                       (350, 6, 0, 350), (353, 8, 0, 353), (500, 4, 77, 433)])
@pytest.mark.parametrize("kap", [7.3 + 0.0j, 7.3 - 2.0j])
def test_mirrored_tiles(n, q, r0, r1, kap):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    flush(f"contour window n={n} q={q} rows {r0}..{r1} kappa={kap}")
    h = P.Bie2d(synth.contour_joukowsky(n), synth.contour_circle(n), q=q, device="cuda")
    full = h.assemble(kap, rows=slice(r0, r1), cols=slice(r0, r1))
    part = h.assemble(kap, rows=slice(r0, r1), cols=slice(r0, r1 - 1))
    for a, b in zip(full, part):
        assert float((a[:, :-1] - b).abs().max()) <= 1e-12 * float(b.abs().max())
        assert bool(torch.isfinite(torch.view_as_real(a)).all())
    for a in (full[0], full[2]):   # symmetric kernels
        assert float((a - a.T).abs().max()) <= 1e-12 * float(a.abs().max())
