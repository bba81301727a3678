"""Selection in the centro-symmetry parameter (the nearest neighbours by an FP32
key, the smallest pair sums one after the other): bit for bit against the
oracle on crystals whose shells tie exactly or within FP32 rounding where the
choice is made, on random atoms, on rows of up to and beyond 64 entries, and for
the smallest and largest numbers of neighbours."""
import numpy as np
import pytest
import torch

from oracle.geometry import Systems
from oracle.switching import csp_all
from paper_2505_12958_amd import ap
from paper_2505_12958_amd import workloads as w

pytestmark = pytest.mark.gpu

RC = 5.5
RNG = np.random.default_rng(9)


def crystal(lattice, n, a, jitter):
    pos = w.lattice_points(lattice, (n,) * 3, a)
    return np.mod(pos + RNG.normal(0.0, 1.0, pos.shape) * jitter, n * a), np.eye(3) * n * a


CASES = {
    "bcc exact": crystal("bcc", 4, 3.0, 0.0),
    "bcc within fp32": crystal("bcc", 4, 3.165, 1e-9),
    "bcc thermal": crystal("bcc", 4, 3.165, 0.08),
    "fcc within fp32": crystal("fcc", 4, 3.615, 1e-9),
    "long rows": crystal("bcc", 6, 2.45, 0.05),
    "gas": (RNG.uniform(0.0, 14.0, (170, 3)), np.eye(3) * 14.0),
    "thin gas": (RNG.uniform(0.0, 20.0, (140, 3)), np.eye(3) * 20.0),
}


@pytest.mark.parametrize("name", list(CASES))
@pytest.mark.parametrize("n_csp", [2, 10, 12, 14, 16])
def test_csp_equals_the_oracle(name, n_csp):
    pos, box = CASES[name]
    n = len(pos)
    S = Systems(pos, box[None], [0, n], (True, True, True), RC)
    ref = csp_all(S, S.neighbour_lists(), n_csp)
    arg = ap.SystemsArg(box, [0, n], (True, True, True), RC)
    P = torch.tensor(np.ascontiguousarray(pos.T), dtype=torch.float64, device="cuda")
    ctx = ap.Context(None, None, ap.AP_PREC_FP64)
    nl = ap.NeighbourList(n, 160, "cuda", False)
    ctx.build_neighbors(arg, P, nl)
    sw = ap.DynamicSwitching(n, n_csp=n_csp, r_lo=2.0, r_hi=4.0)
    out = [torch.zeros(n, dtype=t, device="cuda") for t in (torch.float64, torch.int32)]
    ctx.switching_update(arg, P, nl, sw, out[0], out[1], torch.zeros(1, dtype=torch.int32, device="cuda"))
    torch.cuda.synchronize()
    assert np.array_equal(sw.csp_avg.cpu().numpy()[:n], ref)
    ctx.close()
