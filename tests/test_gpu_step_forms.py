"""What a step at a given dt has in common with the step that computed that dt
(rounding), with the adjoint's forward sweep (every bit) and, on a staggered
field, with the former (every bit)."""
import numpy as np
import pytest

from paper_1312_6127_amd import inputs as I
from test_gpu_parity import dev, field_err, host, interior_mask, say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def G():
    from paper_1312_6127_amd import grrmhd

    grrmhd.lib()
    assert torch.cuda.is_available()
    return grrmhd


def _step(g, P, U, ca, ce, dt, fixed, faces=None):
    Pt, Ut, Bt = P.clone(), U.clone(), None if faces is None else faces.clone()
    if faces is None:
        g.step(Pt, Ut, ca, ce, dt, dt_fixed=fixed)
    else:
        g.step_staggered(Pt, Ut, Bt, ca, ce, dt, dt_fixed=fixed)
    return [x for x in (Pt, Ut, Bt) if x is not None]


@pytest.mark.parametrize("opt", ["rk3", "imex3", "ppm", "full", "staggered"])
@pytest.mark.parametrize("n", [(40, 20, 8), (33, 17, 1)], ids=lambda n: "x".join(map(str, n)))
def test_fixed_dt_and_courant_dt(G, orc, n, opt):
    """Each of the two agrees with the oracle to 1e-11 (the parity tests'
    bound of a step), hence with the other to 2e-11."""
    say("case step forms", n, opt)
    kw = {"imex3": dict(scheme="imex3"), "ppm": dict(ng=4, recon="ppm"), "full": dict(cascade=1),
          "staggered": dict(ct="staggered")}.get(opt, {})
    stag = opt == "staggered"
    pd, P, ca, ce, *faces = I.accretion_disk(n=n, seed=3, faces=stag, **kw)
    g = G.Grid(pd)
    P, ca, ce = dev(P), dev(ca), dev(ce)
    B = dev(faces[0]) if stag else None
    U = g.prim_to_cons(P)
    dt = dev(np.zeros(1))
    m = interior_mask(pd)
    own = _step(g, P, U, ca, ce, dt, False, B)
    assert float(host(dt)[0]) > 0.0
    given = _step(g, P, U, ca, ce, dt, True, B)
    for out, fixed in ((own, False), (given, True)):   # each repeats itself
        for a, b in zip(out, _step(g, P, U, ca, ce, dt, fixed, B)):
            assert np.array_equal(host(a)[:, m], host(b)[:, m]), fixed
    if stag:
        for a, b in zip(own, given):
            assert np.array_equal(host(a)[:, m], host(b)[:, m])
        g.close()
        return
    for a, b in zip(own, given):
        err = field_err(host(a), host(b), m).max()
        say("  own dt against the same dt given:", err)
        assert err < 2e-11
    Pn, Un, ws = g.step_checkpointed(P, ca, ce, dt)
    assert np.array_equal(host(Pn)[:, m], host(given[0])[:, m])
    assert np.array_equal(host(Un)[:, m], host(given[1])[:, m])
    g.close()
