"""The closed-form faces against the oracle where a field's largest magnitude
says little: opacities without bound; faces far from where a field is large."""
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


def _window(x, pd, d):
    """The largest of x over the four cells of each face's stencil along d."""
    a = x.reshape(I.nalloc(pd)[::-1])
    out = a.copy()
    for s in (-1, 1, 2):
        out = np.maximum(out, np.roll(a, s, axis=2 - d))
    return out.reshape(-1)


@pytest.mark.parametrize("flux", ["llf", "hll"])
@pytest.mark.parametrize("n", [(61, 30, 1), (31, 14, 4), (40, 24, 4)],
                         ids=lambda n: "x".join(map(str, n)))
def test_faces_at_their_own_scale(G, orc, n, flux):
    """Every face against the energy-momentum (gas with its rest mass,
    radiation) and field of its own stencil, components in the normal
    observer's units, times the coordinate speed of light: 1e-12, as a field's
    largest magnitude in the parity tests (40 terms, each at most 100 times the
    sum's scale).  From the disk's inner edge to its outer one the gas falls by
    1e2, the radiation by 1e5."""
    say("case faces, own scale", n, flux)
    pd, P, ca, ce = I.accretion_disk(n=n, seed=n[0], flux=flux)
    f = 10.0 ** (4.0 * np.random.default_rng(n[0]).random(ca.shape) - 2.0)
    ce = f * max(n) / P[0]
    P = orc.bc(pd, P)
    g = G.Grid(pd)
    F = host(g.fluxes(dev(P), dev(ca), dev(ce))[0])
    Fr = orc.fluxes(pd, P, ca, ce)[0]
    U = np.abs(orc.prim_to_cons(pd, P))
    x1, x2, _ = I.cell_coords(pd)
    N1, N2, _ = I.nalloc(pd)
    up, lo = np.zeros((3, N2, N1)), np.zeros((3, N2, N1))
    for j in range(N2):
        for i in range(N1):
            gl, gu, _, _ = orc.geom_arrays(orc.geom(pd, x1[0, j, i], x2[0, j, i]))
            for a in range(3):
                up[a, j, i] = np.sqrt(gu[1 + a, 1 + a] - gu[0, 1 + a] ** 2 / gu[0, 0])
                lo[a, j, i] = np.sqrt(gl[1 + a, 1 + a])
    rep = [np.broadcast_to(w[:, None], (3,) + x1.shape).reshape(3, -1) for w in (up, lo)]
    up, lo = rep
    one = np.ones_like(up[0])
    groups = {"gas": ([0, 1, 2, 3, 4], [one, one, *up]), "field": ([5, 6, 7], list(lo)),
              "radiation": ([8, 9, 10, 11], [one, *up])}
    worst = 0.0
    spread = []
    for d in range(3):
        if n[d] == 1:
            continue
        on = np.abs(Fr[d]).max(0) > 0.0
        for name, (qs, ws) in groups.items():
            own = np.max([w * U[q] for q, w in zip(qs, ws)], axis=0)
            scale = _window(own * up[d], pd, d)
            err = np.max([w * np.abs(F[d, q] - Fr[d, q]) for q, w in zip(qs, ws)], axis=0)
            ok = on & (scale > 0.0)
            e = (err[ok] / scale[ok]).max() if ok.any() else 0.0
            spread.append(scale[ok].max() / scale[ok].min())
            say(f"  d {d} {name}: {e:.2e}, scales over {spread[-1]:.1e}")
            worst = max(worst, e)
    assert max(spread) > 1e3
    assert worst < 1e-12
    g.close()
