"""The records that a listed cell's attempts are kept in between kernels, on
the CPU: the device solver headers compiled for the host (hipcc; no GPU
needed).  A cascade resumed from a record must give the same bits as the one
that keeps its attempts in registers."""
import os
import shutil
import subprocess

import numpy as np
import pytest

from paper_1312_6127_amd import inputs as I

HERE = os.path.dirname(os.path.abspath(__file__))
HIPCC = shutil.which("hipcc")
pytestmark = pytest.mark.skipif(HIPCC is None, reason="hipcc not found")


def _run(tmp_path, source, *args):
    exe = tmp_path / "check"
    subprocess.run([HIPCC, "-O2", "-std=c++17", "-x", "hip", "--offload-arch=gfx950",
                    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                    "-o", str(exe), os.path.join(HERE, "host", source)],
                   check=True, capture_output=True)
    out = subprocess.run([str(exe), *args], check=True, capture_output=True, text=True).stdout
    return dict(zip(out.split()[0::2], map(int, out.split()[1::2])))


def _batch_file(orc, path, n, **change):
    pd, P, dt, ca, ce = I.implicit_batch(n, seed=9)
    pd.update(change)
    g0 = orc.geom(pd, 0.0, 0.0)
    U = np.stack([orc.p2u(pd, g0, P[:, c]) for c in range(n)], axis=1)
    U[1] -= 0.3 * U[8]
    U[8] *= 1.3
    with open(path, "wb") as f:
        np.array([n], dtype=np.int64).tofile(f)
        np.array([pd["gam"], pd["arad"], pd["gamma_max"], pd["tol_pmhd"], pd["tol_urad"],
                  pd["tol_accept"], pd["tol_fail"], pd["max_iter"], pd["roundoff"], 0.0]).tofile(f)
        for a in (U, P, dt, ca, ce):
            np.ascontiguousarray(a, dtype=np.float64).tofile(f)


@pytest.mark.parametrize("accept", [1e-9, 1e-14])
def test_full_cascade_resumes_from_the_record(orc, tmp_path, accept):
    """accept 1e-14: most solutions stay unaccepted, so the cascade runs on
    after the URAD attempt and often returns to it."""
    _batch_file(orc, tmp_path / "batch.bin", 1500, tol_accept=accept, roundoff=0)
    vals = _run(tmp_path, "cascade_records_check.cpp", str(tmp_path / "batch.bin"))
    assert vals["resumed"] > 300 and vals["urad"] > 50, vals
    assert vals["differing"] == 0, vals


def test_regime_is_decided_once(orc, tmp_path):
    """Fast gas on a Kerr-Schild grid, its radiation a few ulp about 10 eps of
    the gas energy; attempts of one step, so that the cells on the other side
    are listed too."""
    n = 4000
    pd, *_ = I.accretion_disk(n=(16, 8, 1))
    r = np.random.default_rng(3)
    sym = [(a, b) for a in range(4) for b in range(a, 4)]
    rows = []
    for c in range(n):
        g = orc.geom(pd, r.uniform(0.3, 3.0), r.uniform(0.4, 1.2))
        lo, up, gdet, alpha = orc.geom_arrays(g)
        P = np.zeros(12)
        P[0], P[1] = 1.0, 10.0 ** r.uniform(-4, 0)
        s = 1.0 / np.sqrt(np.diag(lo)[1:])
        P[2:5] = 10.0 ** r.uniform(0, 1.5) * r.standard_normal(3) * s
        P[9:12] = P[2:5] + r.standard_normal(3) * s

        def vel(ut):
            gm = np.sqrt(1.0 + ut @ lo[1:, 1:] @ ut)
            u = np.concatenate([[0.0], ut]) - gm * alpha * up[0]
            u[0] = gm / alpha
            return u

        w = vel(P[2:5]) @ lo @ vel(P[9:12])
        k = (4.0 * w * w - 1.0) / 3.0
        eps = 10.0 * np.finfo(float).eps
        P[8] = eps * P[1] / (1.0 - eps) / k * (1.0 + r.integers(-8, 9) * 2.0 ** -52)
        U = orc.p2u(pd, g, P)
        U[8:] *= 1e16   # the explicit state's radiation is not negligible
        rows.append(np.concatenate([[lo[a, b] for a, b in sym], [up[a, b] for a, b in sym],
                                    [gdet, alpha], U, P, [1e-3]]))
    with open(tmp_path / "cells.bin", "wb") as f:
        np.array([n], dtype=np.int64).tofile(f)
        np.array([pd["gam"], pd["arad"], pd["gamma_max"], pd["tol_pmhd"], pd["tol_urad"],
                  pd["tol_accept"], pd["tol_fail"], 1, pd["roundoff"]],
                 dtype=np.float64).tofile(f)
        np.array(rows).tofile(f)
    vals = _run(tmp_path, "cascade_extreme_check.cpp", str(tmp_path / "cells.bin"))
    assert vals["extreme"] > 500 and vals["cells"] - vals["extreme"] > 100, vals
    assert vals["split"] > 100, vals
    assert vals["differing"] == 0, vals


@pytest.mark.parametrize("steps", [1, 4, 60])
def test_urad_attempt_in_parts(orc, tmp_path, steps):
    """1, the long lists' 4 and, as on short lists, all Newton steps of an
    evaluation's gas inversion a trip."""
    _batch_file(orc, tmp_path / "batch.bin", 6000)
    vals = _run(tmp_path, "urad_parts_check.cpp", str(tmp_path / "batch.bin"), str(steps))
    assert vals["cells"] > 1000 and vals["bisected"] > 50 and vals["rootless"] > 50, vals
    assert (vals["parts"] > 0) == (steps < 60), vals
    assert vals["differing"] == 0, vals
