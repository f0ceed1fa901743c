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
