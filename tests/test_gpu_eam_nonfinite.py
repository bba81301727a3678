"""Closed-form EAM where a listed neighbour's position is not finite (it left the
numbers after the list was built): a distance that is not a number, or infinite,
lies beyond every knot and adds neither density nor pair energy, as when the
knots are summed one by one, so energies stay those of the other bonds (to the
rounding of their sum, 1e-13 of a few eV); the force of every atom that lists it
is not finite, so the condition shows."""
import numpy as np
import pytest
import torch

from paper_2505_12958_amd import ap
from paper_2505_12958_amd import workloads as w

pytestmark = pytest.mark.gpu

PARAMS = dict(w.W_EAM, zbl=w.ZBL_C)


@pytest.mark.parametrize("ncell", [5, 17])  # 250 and 9,826 atoms: 16 and 4 threads per atom
@pytest.mark.parametrize("value", [np.nan, np.inf, -np.inf])
def test_energies_do_not_see_a_distance_that_is_no_number(ncell, value):
    wl = w.make_bulk("cell", ncell, 3.165, 4, n_max=2, l_max=1, nu_max=2, jitter=0.05)
    n, dev, bad = wl.n_atoms, "cuda", wl.n_atoms // 2
    S = ap.SystemsArg.from_workload(wl)
    pos = torch.tensor(np.ascontiguousarray(wl.pos.T), dtype=torch.float64, device=dev)
    ctx = ap.Context(None, None, ap.AP_PREC_FP64)
    ctx.set_eam_analytic(PARAMS)
    nl = ap.NeighbourList(n, 96, dev)
    ctx.build_neighbors(S, pos, nl)

    def energies(nl, p):
        e = torch.zeros(n, dtype=torch.float64, device=dev)
        F = torch.zeros((3, n), dtype=torch.float64, device=dev)
        ctx.eam_forces(S, p, nl, None, e, F)
        return e.cpu().numpy(), F.cpu().numpy().T

    rows = [np.asarray(r) for r in nl.rows()]
    listed = np.array([bad in r for r in rows])
    moved = pos.clone()
    moved[0, bad] = value
    e, F = energies(nl, moved)
    # the same bonds without that atom: each row that lists it loses the entry
    less = ap.NeighbourList(n, 96, dev)
    nbr, cnt = np.zeros((96, n), np.int32), np.zeros(n, np.int32)
    for i, r in enumerate(rows):
        r = r[r != bad]
        nbr[: len(r), i], cnt[i] = r, len(r)
    less.nbr.copy_(torch.tensor(nbr.reshape(less.nbr.shape), device=dev))
    less.count[:n].copy_(torch.tensor(cnt, device=dev))
    e0, _ = energies(less, pos)
    others = np.arange(n) != bad
    assert listed.sum() > 20 and np.isfinite(e[others]).all()
    assert np.abs(e - e0)[others].max() <= 1e-13 * np.abs(e0).max()
    assert not np.isfinite(F[listed]).all(axis=1).any()
    assert np.isfinite(F[others & ~listed]).all()
    ctx.close()
