"""Neighbour lists of the cell kernel, which decides most pairs in FP32 and the
close calls by the canonical rule: equal to the oracle's lists bit for bit with
pairs at the cutoff to within 1e-7, boxes of exactly two cutoffs (pairs at half
the box), one to four cells per axis, orthorhombic and sheared, atoms outside
the box and far outside along a free axis, rows of up to and beyond 64 entries
and several systems of different kinds in one call."""
import numpy as np
import pytest
import torch

from oracle.geometry import Systems
from paper_2505_12958_amd import ap

pytestmark = pytest.mark.gpu

RC = 5.5
SHEAR = np.eye(3) + np.array([[0.0, 0.11, -0.07], [0.05, 0.0, 0.13], [0.0, -0.09, 0.0]])


def at_cutoff(cells, seed):
    """Simple cubic at half the cutoff (pairs at exactly 5.5, half the box at
    four cells), each atom moved by up to 1e-7."""
    g = np.stack(np.meshgrid(*[np.arange(c) for c in cells], indexing="ij"), -1).reshape(-1, 3)
    rng = np.random.default_rng(seed)
    pos = g * (RC / 2) + rng.uniform(0.0, 1e-7, (len(g), 3))
    return pos[rng.permutation(len(pos))], np.diag([c * RC / 2 for c in cells])


def gas(edges, density, seed, out=0.0):
    rng = np.random.default_rng(seed)
    n = int(np.prod(edges) * density)
    return rng.uniform(-out, 1.0 + out, (n, 3)) * np.array(edges), np.diag(np.asarray(edges, float))


def sheared(case):
    return case[0] @ SHEAR, case[1] @ SHEAR


def free_axis():
    """Slab with a free z axis and atoms far above and below the box."""
    pos, box = gas((17.0, 23.0, 12.0), 0.06, 8)
    pos[::41, 2] += 1.0e3
    pos[7::53, 2] -= 300.0
    pos[11::97, 2] = 1.0e9
    return pos, box


PERIODIC = (True, True, True)
CASES = {
    "cutoff and half box": ([at_cutoff((4, 4, 4), 1)], PERIODIC),
    "cutoff, one to four cells": ([at_cutoff((4, 6, 9), 2)], PERIODIC),
    "cutoff, sheared": ([sheared(at_cutoff((7, 8, 9), 3))], PERIODIC),
    "three cells": ([gas((16.6, 17.5, 21.9), 0.06, 4)], PERIODIC),
    "two cells, sheared": ([sheared(gas((14.0, 13.0, 15.0), 0.06, 5, out=0.1))], PERIODIC),
    "cells, sheared, atoms outside": ([sheared(gas((18.0, 24.0, 29.0), 0.06, 6, out=0.2))], PERIODIC),
    "long rows": ([gas((22.0, 22.0, 22.0), 0.093, 7)], PERIODIC),
    "free axis": ([free_axis()], (True, True, False)),
    "all free": ([gas((3.0, 40.0, 9.0), 0.08, 9, out=0.3)], (False, False, False)),
    "mixed batch": ([gas((12.0, 17.0, 23.0), 0.06, 10), sheared(gas((13.0, 18.0, 23.0), 0.06, 11)),
                     at_cutoff((4, 4, 8), 12), sheared(at_cutoff((7, 7, 7), 13)),
                     gas((30.0, 12.0, 12.0), 0.002, 14)], PERIODIC),
}


@pytest.mark.parametrize("name", list(CASES))
def test_lists_equal_the_canonical_rule(name):
    systems, periodic = CASES[name]
    pos = np.concatenate([p for p, _ in systems])
    box = np.stack([b for _, b in systems])
    off = np.concatenate([[0], np.cumsum([len(p) for p, _ in systems])])
    ref = Systems(pos, box, off, periodic, RC).neighbour_lists()
    cap = 128
    assert max(len(j) for j, _ in ref) <= cap
    n = len(pos)
    ctx = ap.Context(None, None, ap.AP_PREC_FP64)
    S = ap.SystemsArg(box, off, periodic, RC)
    nl = ap.NeighbourList(n, cap, "cuda", False)
    ctx.build_neighbors(S, torch.tensor(np.ascontiguousarray(pos.T), dtype=torch.float64, device="cuda"), nl)
    torch.cuda.synchronize()
    rows, count = nl.rows(), nl.count.cpu().numpy()
    for i, (j, _) in enumerate(ref):
        assert count[i] == len(j) and np.array_equal(rows[i], j), f"{name}: atom {i}"
    ctx.close()
