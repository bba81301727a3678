"""ACE bond kernels beyond 524,288 atoms, where a bounded number of workgroups
takes the listed atoms in turn: copies of one periodic 250-atom cell, few and
many listed atoms (below and above one turn of 32,768), every copy against the
oracle on the single cell.

Tolerances as in the other parity tests: 1e-10 in FP64, 1e-5 (relative norm) in
mixed precision."""
import dataclasses

import numpy as np
import pytest

from gpu_helpers import run_force
from oracle.ap import APOracle
from oracle.geometry import Systems
from paper_2505_12958_amd import ap
from paper_2505_12958_amd import workloads as w

pytestmark = pytest.mark.gpu

COPIES = 2098


@pytest.mark.parametrize("n_ace", [3, 21])
@pytest.mark.parametrize("precision", [ap.AP_PREC_FP64, ap.AP_PREC_MIXED])
def test_every_copy_matches_the_oracle(n_ace, precision):
    wl = w.make_bulk("cell", 5, 3.165, 4, n_max=3, l_max=2, nu_max=3, jitter=0.08)
    n = wl.n_atoms
    lam = np.zeros(n)
    lam[np.random.default_rng(5).permutation(n)[:n_ace]] = 0.75
    ref = APOracle(None, wl.ace).evaluate(Systems.from_workload(wl), lam)
    many = dataclasses.replace(
        wl, pos=np.tile(wl.pos, (COPIES, 1)), box=np.tile(wl.box, (COPIES, 1, 1)),
        sys_offset=np.arange(COPIES + 1, dtype=np.int64) * n, masses=np.tile(wl.masses, COPIES),
        fixed=np.tile(wl.fixed, COPIES), vel=np.tile(wl.vel, (COPIES, 1)))
    assert many.n_atoms > 524288
    g = run_force(many, precision=precision, lam=np.tile(lam, COPIES), with_eam=False, with_rev=False,
                  capacity=96)
    for got, want in ((g["forces"].reshape(COPIES, n, 3), ref["forces"]),
                      (g["e_atom"].reshape(COPIES, n), ref["e_atom"]), (g["virial"], ref["virial"][0])):
        if precision == ap.AP_PREC_FP64:
            assert np.abs(got - want).max() <= 1e-10 * np.sqrt((want ** 2).mean())
        else:
            err = np.sqrt(((got - want) ** 2).reshape(COPIES, -1).sum(1).max())
            assert err <= 1e-5 * np.linalg.norm(want)
