"""The closed-form faces against the oracle where a field's largest magnitude
says little: opacities without bound."""
import numpy as np
import pytest

from paper_1312_6127_amd import inputs as I
from test_gpu_parity import dev, field_err, host, say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def G():
    from paper_1312_6127_amd import grrmhd

    grrmhd.lib()
    assert torch.cuda.is_available()
    return grrmhd


@pytest.mark.parametrize("flux", ["llf", "hll"])
@pytest.mark.parametrize("n", [(14, 9, 8), (16, 9, 1)], ids=lambda n: "x".join(map(str, n)))
def test_faces_of_unbounded_opacity(G, orc, n, flux):
    """Infinite and nearly infinite opacities leave the radiation the gas's own
    speed, as any large one does (1e-12 of a field, as the parity tests)."""
    say("case faces, unbounded opacity", n, flux)
    pd, P, ca, ce = I.accretion_disk(n=n, seed=4, flux=flux)
    P = orc.bc(pd, P)
    r = np.random.default_rng(8)
    kind = r.integers(0, 5, ca.shape)
    ca = np.choose(kind, [ca, np.full_like(ca, np.inf), np.full_like(ca, 1.7e308),
                          np.full_like(ca, 1e290), np.zeros_like(ca)])
    g = G.Grid(pd)
    F, emf, vch = (host(x) for x in g.fluxes(dev(P), dev(ca), dev(ce)))
    Fr, emfr, vchr = orc.fluxes(pd, P, ca, ce)
    assert np.isfinite(Fr).all() and np.isfinite(F).all()
    for d in range(3):
        assert field_err(F[d], Fr[d]).max() < 1e-12, d
    assert field_err(vch, vchr).max() < 1e-12
    g.close()
