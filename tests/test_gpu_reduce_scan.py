"""Per-system sums and list compaction where their launches change: systems of
one chunk each (summed by one kernel) and of none, one and many chunks (a
wavefront adds up to and more than 64 of them); lists of up to one scan tile
(one kernel) and beyond.  Sums to n eps sum |e| against exact summation, lists
equal."""
import math

import numpy as np
import pytest
import torch

from paper_2505_12958_amd import ap
from paper_2505_12958_amd import workloads as w

pytestmark = pytest.mark.gpu

CHUNK = 4096
RC = 5.5
GIVEN = 4  # rule kind: lambda is the caller's


def systems(sizes):
    off = np.concatenate([[0], np.cumsum(sizes)])
    return ap.SystemsArg(np.tile(np.eye(3) * 12.0, (len(sizes), 1, 1)), off, (True, True, True), RC), off


@pytest.mark.parametrize("sizes", [[1], [CHUNK], [7, CHUNK, 300], [CHUNK + 1], [0, 5, CHUNK + 1, 0],
                                   [64 * CHUNK, 3], [65 * CHUNK + 17, 2 * CHUNK, 1]])
def test_system_sums(sizes):
    S, off = systems(sizes)
    e = np.random.default_rng(1).normal(size=off[-1])
    ctx = ap.Context(None, None, ap.AP_PREC_FP64)
    out = torch.full((len(sizes),), 7.0, dtype=torch.float64, device="cuda")
    ctx.reduce_energy(S, torch.tensor(e, device="cuda"), out)
    torch.cuda.synchronize()
    for s, got in enumerate(out.cpu().numpy()):
        part = e[off[s]:off[s + 1]]
        assert abs(got - math.fsum(part)) <= max(1, len(part)) * 2.0 ** -52 * np.abs(part).sum()
    ctx.close()


@pytest.mark.parametrize("n", [1, 255, 4095, 4096, 4097, 9000])
@pytest.mark.parametrize("share", [0.0, 0.4, 1.0])
def test_compacted_list(n, share):
    S, _ = systems([n])
    rng = np.random.default_rng(n)
    lam = np.where(rng.random(n) < share, 0.5, 0.0)
    ctx = ap.Context(None, None, ap.AP_PREC_FP64)
    dev = dict(device="cuda")
    ace_list = torch.full((n,), -7, dtype=torch.int32, **dev)
    n_ace = torch.full((1,), -7, dtype=torch.int32, **dev)
    ctx.blend(S, torch.zeros((3, n), dtype=torch.float64, **dev), w.LambdaRule(GIVEN),
              torch.tensor(lam, **dev), ace_list, n_ace, None)
    torch.cuda.synchronize()
    want = np.nonzero(lam)[0]
    assert int(n_ace.item()) == len(want)
    assert np.array_equal(ace_list.cpu().numpy()[: len(want)], want)
    ctx.close()
