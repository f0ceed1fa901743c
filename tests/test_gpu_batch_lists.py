"""The lists of a batch's cascade at the edges of their shared storage: no
extreme cell, some, all; a workspace of exactly the stated size."""
import numpy as np
import pytest

from paper_1312_6127_amd import inputs as I
from test_gpu_parity import _batch_cons, dev, host, say

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def G():
    from paper_1312_6127_amd import grrmhd

    grrmhd.lib()
    assert torch.cuda.is_available()
    return grrmhd


@pytest.mark.parametrize("cascade", [0, 1])
@pytest.mark.parametrize("share", [0.0, 0.3, 1.0])
@pytest.mark.parametrize("n", [1, 65, 3001])
def test_extreme_cells_share_the_list(G, orc, n, share, cascade):
    """The same bits in every form, and cell by cell in batches of 64; nothing
    written beyond the workspace."""
    say("case batch lists", n, share, cascade)
    pd, P, dt, ca, ce = I.implicit_batch(n, seed=12)
    pd["cascade"] = cascade
    ext = np.random.default_rng(n).random(n) < share
    P[8, ext] *= 1e-20
    U = _batch_cons(orc, pd, P)
    args = [dev(x) for x in (U, P, dt, ca, ce)]
    outs = []
    for mode, block, wpc in ((G.PER_CELL, 64, 1), (G.PER_ITERATION, 64, 0), (G.PERSISTENT, 64, 8),
                             (G.PERSISTENT, 256, 16)):
        ws, wsb = G.batch_workspace(n, mode)
        raw = torch.full((wsb + 512,), 0xA5, dtype=torch.uint8, device="cuda")
        off = (-raw.data_ptr()) % 256
        ws = raw[off:off + wsb]
        outs.append([host(x) for x in G.implicit_source_ex(pd, *args, mode, block, wpc,
                                                           ws=(ws, wsb))])
        assert (host(raw[off + wsb:]) == 0xA5).all() and (host(raw[:off]) == 0xA5).all()
        listed = G.batch_stats((ws, wsb))[2]
        assert listed >= ext.sum()
    st = outs[0][3]
    assert ((st & G.ST_EXTREME) != 0)[ext].all()   # the recipe has a few of its own
    for o in outs[1:]:
        for a, b in zip(o, outs[0]):
            assert np.array_equal(a.view(np.uint8), b.view(np.uint8))
    for at in range(0, n, 64):
        part = G.implicit_source(pd, *(x[..., at:at + 64].contiguous() for x in args))
        for a, b in zip(part, outs[0]):
            b = np.ascontiguousarray(b[..., at:at + 64])
            assert np.array_equal(host(a).view(np.uint8), b.view(np.uint8)), at
