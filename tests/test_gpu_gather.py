"""ACE force gather: the reverse slots found by searching the atom-major rows
(two-round search on rows of up to 64 entries when the capacity is a multiple
of 4, binary search otherwise) against the full reverse index, bit for bit,
and against the oracle.  Rows just below, at and above 64 entries.

Tolerance 1e-10 against the oracle, as in the other FP64 parity tests (the same
FP64 sums in another order)."""
import numpy as np
import pytest

from gpu_helpers import run_force
from oracle.ap import APOracle
from oracle.geometry import Systems
from paper_2505_12958_amd import ap
from paper_2505_12958_amd import workloads as w

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("a,capacity", [(3.165, 64), (3.165, 66), (2.74, 100), (2.72, 128), (2.53, 128),
                                        (2.5, 130)])
@pytest.mark.parametrize("precision", [ap.AP_PREC_FP64, ap.AP_PREC_MIXED])
def test_searched_slots_equal_the_reverse_index(a, capacity, precision):
    wl = w.make_bulk("rows", 5, a, 3, n_max=3, l_max=2, nu_max=3, jitter=0.03)
    lam = np.where(np.random.default_rng(2).random(wl.n_atoms) < 0.6, 0.5, 0.0)
    ref = run_force(wl, precision=precision, capacity=capacity, lam=lam, with_eam=False, with_rev=True)
    got = run_force(wl, precision=precision, capacity=capacity, lam=lam, with_eam=False, with_rev=False)
    assert ref["count"].max() > 50
    assert np.array_equal(got["forces"], ref["forces"])
    if precision == ap.AP_PREC_FP64:
        o = APOracle(None, wl.ace).evaluate(Systems.from_workload(wl), lam)["forces"]
        assert np.abs(got["forces"] - o).max() <= 1e-10 * np.sqrt((o ** 2).mean())
