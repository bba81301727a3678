"""EAM passes with 16, 4 and 2 threads per atom (up to 8192 atoms, up to
131,072, beyond): copies of one periodic 250-atom cell, just below and above the
two boundaries, with fully EAM, mixed and EAM-free atoms; every copy against the
oracle on the single cell, orthorhombic and sheared, tables and closed form.

Tolerance 1e-10, as in the other FP64 parity tests (the same FP64 sums in
another order; the bonds' terms are those of the serial sum to a few ulp)."""
import dataclasses

import numpy as np
import pytest

from gpu_helpers import run_force
from oracle.ap import APOracle
from oracle.eam_analytic import AnalyticWEam
from oracle.geometry import Systems
from paper_2505_12958_amd import ap
from paper_2505_12958_amd import workloads as w

pytestmark = pytest.mark.gpu

PARAMS = dict(w.W_EAM, zbl=w.ZBL_C)
TOL = 1e-10


@pytest.fixture(scope="module")
def cells():
    """Per (shear, closed form): the cell and the oracle's result for it."""
    out = {}
    base = w.make_bulk("cell", 5, 3.165, 4, n_max=3, l_max=2, nu_max=3, jitter=0.08)
    lam = np.random.default_rng(3).choice([0.0, 0.25, 1.0], base.n_atoms)
    for sheared in (False, True):
        m = np.eye(3) + (np.array([[0, 0.02, 0], [0, 0, 0], [-0.01, 0, 0]]) if sheared else 0.0)
        wl = dataclasses.replace(base, pos=base.pos @ m, box=base.box @ m)
        for closed in (False, True):
            model = AnalyticWEam(PARAMS) if closed else None
            ref = APOracle(None if closed else wl.eam, None, eam_model=model)
            out[sheared, closed] = wl, lam, ref.evaluate(Systems.from_workload(wl), lam)
    return out


@pytest.mark.parametrize("copies", [1, 32, 33, 524, 525])
@pytest.mark.parametrize("sheared", [False, True])
@pytest.mark.parametrize("closed", [False, True])
def test_every_copy_matches_the_oracle(cells, copies, sheared, closed):
    wl, lam, ref = cells[sheared, closed]
    n = wl.n_atoms
    many = dataclasses.replace(
        wl, pos=np.tile(wl.pos, (copies, 1)), box=np.tile(wl.box, (copies, 1, 1)),
        sys_offset=np.arange(copies + 1, dtype=np.int64) * n, masses=np.tile(wl.masses, copies),
        fixed=np.tile(wl.fixed, copies), vel=np.tile(wl.vel, (copies, 1)))
    g = run_force(many, lam=np.tile(lam, copies), with_ace=False, with_rev=False, capacity=96,
                  eam_analytic=PARAMS if closed else None)
    F, E = g["forces"].reshape(copies, n, 3), g["e_atom"].reshape(copies, n)
    assert np.abs(F - ref["forces"]).max() <= TOL * np.sqrt((ref["forces"] ** 2).mean())
    assert np.abs(E - ref["e_atom"]).max() <= TOL * np.abs(ref["e_atom"]).max()
    assert np.abs(g["virial"] - ref["virial"]).max() <= TOL * np.abs(ref["virial"]).max()
