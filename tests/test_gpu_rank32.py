"""Mixed rank kernels (tiles of 8 atoms, 16-row steps of 8-column chunks,
adjoint jobs) in both variants (AP_RANK_MODE 0: narrow where a rank has one, 1:
wide) at the edges of their tiling: odd and smallest n_max, every l_max, ranks
without channels, models on both sides of the narrow variant's limits, ragged
last tiles.

Tolerance 1e-5 (relative norm), the method's bar for the mixed path, as in the
other mixed tests."""
import numpy as np
import pytest

from gpu_helpers import run_force
from oracle.ap import APOracle
from oracle.geometry import Systems
from paper_2505_12958_amd import ap
from paper_2505_12958_amd import workloads as w

pytestmark = pytest.mark.gpu

TOL = 1e-5


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("shape,n_ace", [
    ((1, 0, 2), 1), ((1, 4, 4), 9), ((2, 3, 4), 8), ((3, 2, 4), 7), ((5, 3, 3), 17), ((6, 3, 4), 15),
    ((7, 1, 4), 9), ((7, 3, 3), 11), ((8, 4, 2), 5), ((8, 2, 4), 13), ((4, 4, 3), 128),
])
def test_mixed_ranks_match_the_oracle(shape, n_ace, mode, monkeypatch):
    monkeypatch.setenv("AP_RANK_MODE", str(mode))
    wl = w.make_bulk("edge", 4, w.A_W, 3, n_max=shape[0], l_max=shape[1], nu_max=shape[2], r_full=4.0)
    lam = np.zeros(wl.n_atoms)
    lam[np.random.default_rng(1).permutation(wl.n_atoms)[:n_ace]] = 0.75
    ref = APOracle(None, wl.ace).evaluate(Systems.from_workload(wl), lam)
    g = run_force(wl, precision=ap.AP_PREC_MIXED, lam=lam, with_eam=False)
    rel = lambda a, b: np.linalg.norm(a - b) / np.linalg.norm(b)
    assert rel(g["forces"], ref["forces"]) <= TOL
    assert rel(g["e_atom"], ref["e_atom"]) <= TOL
    assert rel(g["virial"], ref["virial"]) <= TOL
