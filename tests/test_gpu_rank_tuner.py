"""The choice between the narrow and the wide variant of the mixed rank kernels:
what the cache file fixes, and when the library measures at all."""
import json

import numpy as np
import pytest
import torch

from paper_2505_12958_amd import ap
from paper_2505_12958_amd import workloads as w

pytestmark = pytest.mark.gpu


class Ace:
    """ACE forces of a crystal, every atom listed or none."""

    def __init__(self, ncell, n_max, l_max, nu):
        wl = self.wl = w.make_bulk("edge", ncell, w.A_W, 3, n_max=n_max, l_max=l_max, nu_max=nu, r_full=4.0)
        n, f64 = wl.n_atoms, dict(dtype=torch.float64, device="cuda")
        self.S = ap.SystemsArg.from_workload(wl)
        self.pos = torch.tensor(np.ascontiguousarray(wl.pos.T), **f64)
        self.nl = ap.NeighbourList(n, 64)
        self.lam, self.e, self.F = torch.ones(n, **f64), torch.zeros(n, **f64), torch.zeros((3, n), **f64)
        self.list = torch.arange(n, dtype=torch.int32, device="cuda")
        self.n_all = torch.tensor([n], dtype=torch.int32, device="cuda")
        self.n_none = torch.zeros(1, dtype=torch.int32, device="cuda")

    def neighbours(self, ctx):
        ctx.build_neighbors(self.S, self.pos, self.nl)

    def forces(self, ctx, n_ace=None):
        ctx.ace_forces(self.S, self.pos, self.nl, self.lam, self.list, self.n_all if n_ace is None else n_ace,
                       self.e, self.F)

    def run(self, n_ace=None):
        """One call on a new context: the variant it took."""
        ctx = ap.Context(None, self.wl.ace, ap.AP_PREC_MIXED)
        self.neighbours(ctx)
        self.forces(ctx, n_ace)
        torch.cuda.synchronize()
        mode = int(ctx.info("ace.rank_mode"))
        ctx.close()
        return mode


@pytest.fixture
def cache(tmp_path, monkeypatch):
    monkeypatch.delenv("AP_RANK_MODE", raising=False)
    monkeypatch.delenv("AP_AUTOTUNE", raising=False)
    monkeypatch.setenv("AP_AUTOTUNE_CACHE", str(tmp_path / "tune.json"))
    return tmp_path / "tune.json"


def test_a_cached_choice_is_taken_unless_it_is_of_the_earlier_kernels(cache):
    case = Ace(4, 3, 2, 3)
    mode = case.run()
    (key, val), = json.loads(cache.read_text()).items()
    assert val == mode and mode in (0, 1)
    for planted in (0, 1):
        cache.write_text(json.dumps({key: planted}))
        assert case.run() == planted
        assert json.loads(cache.read_text()) == {key: planted}
    # a key without the version is of kernels that are gone: ignored, and kept
    dev, version, rest = key.split("|", 2)
    assert rest.startswith("ace 3 2 3 3 ")
    cache.write_text(json.dumps({f"{dev}|{rest}": 1}))
    case.run()
    entries = json.loads(cache.read_text())
    assert set(entries) == {key, f"{dev}|{rest}"}


def test_a_model_with_one_variant_is_not_timed(cache):
    """(8, 4): too many components for a narrow variant.  The first call of a size
    bucket only enqueues: an event behind a long kernel is still pending after it."""
    big, small = Ace(6, 8, 4, 2), Ace(4, 8, 4, 2)
    ctx = ap.Context(None, big.wl.ace, ap.AP_PREC_MIXED)
    big.neighbours(ctx)
    big.forces(ctx)  # sizes the buffers
    small.neighbours(ctx)
    assert big.wl.n_atoms.bit_length() != small.wl.n_atoms.bit_length()
    torch.cuda.synchronize()
    t = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    t[0].record()
    torch.cuda._sleep(1_000_000)
    t[1].record()
    torch.cuda.synchronize()
    cycles = int(1_000_000 * 300.0 / t[0].elapsed_time(t[1]))  # 0.3 s
    behind = torch.cuda.Event()
    torch.cuda._sleep(cycles)
    behind.record()
    small.forces(ctx)
    pending = not behind.query()
    torch.cuda.synchronize()
    assert pending and int(ctx.info("ace.rank_mode")) == 0
    ctx.close()


def test_a_choice_on_an_empty_list_is_not_final(cache):
    case = Ace(4, 3, 2, 3)
    ctx = ap.Context(None, case.wl.ace, ap.AP_PREC_MIXED)
    case.neighbours(ctx)
    case.forces(ctx, case.n_none)
    assert not cache.exists()
    for _ in range(63):
        case.forces(ctx)
    assert not cache.exists()
    case.forces(ctx)  # call 64 measures again, now with every atom listed
    mode = int(ctx.info("ace.rank_mode"))
    (val,) = json.loads(cache.read_text()).values()
    assert val == mode and mode in (0, 1)
    ctx.close()
