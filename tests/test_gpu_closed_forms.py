"""The closed forms of the FP64 step (faces, geometric source, implicit solve)
and the order in which their launches take a grid, against the oracle at the
sizes and states where they could go wrong: pieces of 64 faces and 128 cells
and their remainders, one cell along an axis, tiles that no grid line fills,
faces on either side of the optically thick limiter, cells whose radiation
the limiters act on.

Tolerance: that of the parity tests, 1e-12 of a field's largest magnitude; a
flux or source is a sum of at most 40 rounded terms, none larger than 100
times the sum's scale: 40 * 100 * 2^-53 = 4e-13.  For the solved cells see
_tolerance.
"""
import numpy as np
import pytest

from paper_1312_6127_amd import inputs as I
from test_oracle_pins import _periodic_box
from test_gpu_parity import _batch_cons, dev, field_err, host, interior_mask, say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def G():
    from paper_1312_6127_amd import grrmhd

    grrmhd.lib()
    assert torch.cuda.is_available()
    return grrmhd


SHAPES = [(61, 1, 1), (63, 1, 1), (64, 1, 1), (129, 1, 1), (7, 4, 1), (62, 2, 1), (16, 8, 1),
          (9, 6, 2), (31, 4, 4), (14, 9, 8), "box"]


def _name(n):
    return n if n == "box" else "x".join(map(str, n))


def _state(n, flux):
    if n == "box":   # flat space, field and motion in every direction
        n = (13, 10, 5)
        pd, P, ca, ce = _periodic_box(n, seed=7)
        pd["flux"] = flux
    elif n[1] == 1:
        pd, P, ca, ce = I.shock_tube_1d(n[0], flux=flux)
    else:
        pd, P, ca, ce = I.accretion_disk(n=n, seed=n[0], flux=flux)
    # cell optical depths from 1e-2 to 1e2 on both sides of the limiter's 4/3
    f = 10.0 ** (4.0 * np.random.default_rng(n[0]).random(ca.shape) - 2.0)
    return pd, P, ca, f * max(n) / P[0]


@pytest.mark.parametrize("flux", ["llf", "hll"])
@pytest.mark.parametrize("n", SHAPES, ids=_name)
def test_faces_and_update(G, orc, n, flux):
    say("case", n, flux, "closed-form faces and update")
    pd, P, ca, ce = _state(n, flux)
    P = orc.bc(pd, P)
    g = G.Grid(pd)
    F, emf, vch = (host(x) for x in g.fluxes(dev(P), dev(ca), dev(ce)))
    Fr, emfr, vchr = orc.fluxes(pd, P, ca, ce)
    for d in range(3):
        assert field_err(F[d], Fr[d]).max() < 1e-12, d
    assert field_err(emf, emfr).max() < 1e-12
    assert field_err(vch, vchr).max() < 1e-12
    dt = orc.timestep(pd, vchr)
    U = orc.prim_to_cons(pd, P)
    Up = U * (1 + 1e-3 * np.sin(np.arange(U.size)).reshape(U.shape))
    m = interior_mask(pd)
    for a, b, c in [(1.0, 0.0, 1.0), (1 / 3, 2 / 3, 2 / 3)]:
        Ue = host(g.explicit_update(a, b, c, dev(np.array([dt])), dev(P), dev(U), dev(Up), dev(Fr),
                                    dev(emfr)))
        Uer = orc.explicit_update(pd, a, b, c, dt, P, U, Up, Fr, emfr)
        assert field_err(Ue, Uer, m).max() < 1e-12, (a, field_err(Ue, Uer, m))
    g.close()


def _explicit(orc, pd, P, ca, kind):
    U = orc.prim_to_cons(pd, P)
    odd = np.arange(P.shape[1]) % 3 == 1
    if kind == "weak":        # radiation energy of either sign near nothing
        U[8:, odd] *= 1e-3
        U[8, odd] *= np.where(np.arange(odd.sum()) % 2, 1.0, -1.0)
    elif kind == "beamed":    # flux beyond what the energy carries
        U[9, odd] += 1.2 * np.abs(U[8, odd])
    elif kind == "thick":
        ca = ca + 1e4
    return U, ca, 1e-3


LIMITERS = 1 << 2 | 1 << 3   # ST_TYPE2_NEG, ST_BASIC


def _tolerance(orc, pd, U, P, dt, ca, ce, Pr, Ur, good):
    """1e-12, or 100 times (the rounded operations of a residual) what one ulp
    of the inputs moves the oracle's own solution by, if that is more."""
    own = np.zeros(2)
    for s in range(3):
        r = np.random.default_rng(s)
        f, h = (1.0 + 2.0 ** -52 * r.standard_normal(U.shape) for _ in range(2))
        P2, U2, _, st = orc.implicit_grid(pd, U * f, P * h, dt, ca, ce)
        same = good & ((st & orc.ST_FAIL) == 0)
        own = np.maximum(own, [field_err(P2, Pr, same).max(), field_err(U2, Ur, same).max()])
    return np.maximum(1e-12, 100.0 * own)


@pytest.mark.parametrize("kind", ["plain", "weak", "beamed", "thick"])
@pytest.mark.parametrize("n", [(65, 1, 1), (7, 4, 1), (31, 6, 2), "box"], ids=_name)
def test_implicit(G, orc, n, kind):
    say("case", n, kind, "closed-form implicit solve")
    pd, P, ca, ce = _state(n, "llf")
    P = orc.bc(pd, P)
    ce = np.zeros_like(ce)
    U, ca, dt = _explicit(orc, pd, P, ca, kind)
    g = G.Grid(pd)
    Pg, Ug, it, st, err = (host(x) for x in g.implicit(dev(U), dev(P), 1.0, dev(np.array([dt])),
                                                       dev(ca), dev(ce)))
    Pr, Ur, itr, str_ = orc.implicit_grid(pd, U, P, dt, ca, ce)
    m = interior_mask(pd)
    fail, failr = (st & orc.ST_FAIL) != 0, (str_ & orc.ST_FAIL) != 0
    assert (fail != failr)[m].mean() < 0.02
    # the same limiters acted, and the residual is solved
    good = m & ~fail & ~failr & (err < 1e-12) & (((st ^ str_) & LIMITERS) == 0)
    assert good.sum() > 0.9 * (m & ~failr).sum()
    tol = _tolerance(orc, pd, U, P, dt, ca, ce, Pr, Ur, good)
    assert field_err(Pg, Pr, good).max() < tol[0], (field_err(Pg, Pr, good), tol)
    assert field_err(Ug, Ur, good).max() < tol[1], (field_err(Ug, Ur, good), tol)
    g.close()


@pytest.mark.parametrize("n", [(7, 4, 1), (97, 13, 6)], ids=_name)
def test_lane_statistics(G, orc, n):
    """Launches of fewer and of more tiles than the statistics have slots: the
    totals are the cells' own trip counts."""
    say("case", n, "lane statistics")
    pd, P, ca, ce = I.accretion_disk(n=n, seed=3)
    P = orc.bc(pd, P)
    g = G.Grid(pd)
    U = g.prim_to_cons(dev(P))
    for launches in (1, 2):
        _, _, it, st, _ = g.implicit(U, dev(P), 1.0, dev(np.array([1e-3])), dev(ca), dev(ce))
        trips, slots, rest = g.implicit_stats()
        m = interior_mask(pd)
        assert rest == 0 and np.all(host(st)[m] == G.ST_PMHD)
        assert trips == launches * (host(it)[m] + 1).sum()
        assert trips <= slots <= launches * 64 * (host(it)[m] + 1).sum() and slots % 64 == 0
    g.close()


def test_batch_cascade_in_parts(G, orc):
    """A batch whose cascade list is longer than the lanes of the grid (lanes
    take their inversions in parts, bisections wait for company), against the
    same cells in batches down to a single cell, whose lists are spread over
    the wavefronts: the same bits, cell by cell."""
    k, reps = 5000, 30
    n = k * reps + 1
    say("case batch cascade", n)
    pd, P, dt, ca, ce = I.implicit_batch(k, seed=11)
    U = _batch_cons(orc, pd, P)
    tile = np.arange(n) % k
    dt = dt[tile] * (1.0 + 0.02 * (np.arange(n) // k))
    args = [dev(x) for x in (U[:, tile], P[:, tile], dt, ca[tile], ce[tile])]
    ws = G.batch_workspace(n)
    whole = G.implicit_source_ex(pd, *args, G.PER_CELL, ws=ws)
    assert G.batch_stats(ws)[2] > 64 * 1024
    evals = G.batch_cascade_stats(ws)[0]
    at = parts = 0
    for size in (1, 63, 64, 65, 1023, 4099, 20000, n):
        end = min(at + size, n)
        sub = [x[..., at:end].contiguous() for x in args]
        ws = G.batch_workspace(end - at)
        part = G.implicit_source_ex(pd, *sub, G.PER_CELL, ws=ws)
        parts += G.batch_cascade_stats(ws)[0]
        for a, b in zip(whole, part):
            a, b = host(a[..., at:end].contiguous()), host(b)
            assert np.array_equal(a.view(np.uint8), b.view(np.uint8)), (at, end)
        at = end
    assert at == n and parts == evals
