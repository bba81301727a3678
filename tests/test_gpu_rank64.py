"""FP64 rank kernels (tiles of 4 atoms, 16 x 4 coefficient tiles, adjoint
jobs) at the edges of their tiling: odd and smallest n_max, every l_max, ranks
without channels, ragged last tiles, models outside the tiling (n_max > 8),
and more ACE atoms than one batch of the item buffers.

Tolerance 1e-10: the same FP64 sums in another order (a few thousand terms of
O(1), about 1e-13), as in the other FP64 parity tests."""
import numpy as np
import pytest
import torch

from gpu_helpers import run_force
from oracle.ap import APOracle
from oracle.geometry import Systems
from paper_2505_12958_amd import ap
from paper_2505_12958_amd import workloads as w

pytestmark = pytest.mark.gpu

TOL = 1e-10


def crystal(n_max, l_max, nu, seed=3, ncell=4):
    wl = w.make_bulk("edge", ncell, w.A_W, seed, n_max=n_max, l_max=l_max, nu_max=nu, r_full=4.0)
    return wl


@pytest.mark.parametrize("shape,n_ace", [
    ((1, 0, 2), 1), ((1, 4, 4), 5), ((2, 3, 4), 4), ((3, 2, 4), 7), ((5, 3, 3), 6), ((7, 1, 4), 9),
    ((8, 4, 2), 3), ((8, 2, 4), 13), ((9, 2, 3), 5), ((4, 4, 3), 128),
])
def test_fp64_ranks_match_the_oracle(shape, n_ace):
    wl = crystal(*shape)
    lam = np.zeros(wl.n_atoms)
    lam[np.random.default_rng(1).permutation(wl.n_atoms)[:n_ace]] = 0.75
    ref = APOracle(None, wl.ace).evaluate(Systems.from_workload(wl), lam)
    g = run_force(wl, lam=lam, with_eam=False)
    rms = np.sqrt((ref["forces"] ** 2).mean())
    assert np.abs(g["forces"] - ref["forces"]).max() <= TOL * rms
    assert np.abs(g["e_atom"] - ref["e_atom"]).max() <= TOL * np.abs(ref["e_atom"]).max()
    assert np.abs(g["virial"] - ref["virial"]).max() <= TOL * np.abs(ref["virial"]).max()


def test_more_ace_atoms_than_one_batch():
    """A periodic crystal of 13^3 copies of a 128-atom cell (281,216 ACE atoms,
    more than the 262,144 of one batch) has the cell's forces and energies."""
    base = crystal(2, 1, 2)
    c = 13
    L = base.box[0, 0, 0]
    sh = L * np.stack(np.meshgrid(*[np.arange(c)] * 3, indexing="ij"), -1).reshape(-1, 1, 3)
    big = crystal(2, 1, 2)
    big.pos = (base.pos[None] + sh).reshape(-1, 3)
    big.box = base.box * c
    big.sys_offset = np.array([0, len(big.pos)], np.int64)
    small = run_force(base, lam=np.ones(base.n_atoms), with_eam=False, with_rev=False)
    g = run_force(big, lam=np.ones(big.n_atoms), with_eam=False, with_rev=False)
    f = g["forces"].reshape(-1, base.n_atoms, 3)
    # positions of the copies round to about 2e-14 A, forces to the same relative size
    assert np.abs(f - small["forces"][None]).max() <= TOL * np.abs(small["forces"]).max()
    e = g["e_atom"].reshape(-1, base.n_atoms)
    assert np.abs(e - small["e_atom"][None]).max() <= TOL * np.abs(small["e_atom"]).max()
