"""Large 3D meshes, where the stage runs with a line of nodes per thread (N = 3 to 7): parity
with the oracle at the edges of its split (elements that do not fill a wave or a block, one or
two elements along a direction, both block sizes), on smooth states, on states whose pairs all
lie beyond the near-equal series of the logarithmic means, and on the time steps' own path
(wave speeds, update); ensembles that mix such runs with small ones.  Tolerances: the float64
parity bars of gpu_util.
"""
import math

import numpy as np
import pytest
import torch

import oracle
from paper_2108_06476_amd import dgx, inputs

from gpu_util import TOL_FP64, dev, err_v, host, state_err

pytestmark = pytest.mark.gpu

# the smallest meshes with a line per thread: N = 3 20 480 elements (40 960: blocks of four
# waves), N = 4 12 288, N = 5 5 120, N = 6 960, N = 7 8 192
CELLS = [(3, (32, 32, 20)), (3, (29, 27, 27)), (3, (1, 150, 140)), (3, (2, 129, 81)),
         (3, (37, 35, 33)), (4, (24, 23, 23)), (4, (1, 96, 128)), (5, (19, 17, 16)),
         (5, (64, 1, 81)), (6, (8, 11, 11)), (6, (31, 31, 1)), (7, (21, 20, 20))]


def _cfg(N, cells, surface):
    hi = tuple(2.0 * math.pi * c / max(cells) for c in cells)
    return dict(dim=3, polydeg=N, cells=cells, xmin=(0.0,) * 3, xmax=hi, gamma=1.4, volume="ec",
                surface=surface)


def _state(o, cfg, kind):
    if kind == "nodal":
        return inputs.random_nodal((o.E, o.NN), 3, 17)
    if kind == "jumps":   # ratios up to 1e4 between neighbours
        return inputs.random_nodal((o.E, o.NN), 3, 18, rho_range=(1e-2, 10.0), p_range=(1e-3, 10.0))
    return inputs.random_smooth(o.node_coords(), 19, periods=list(cfg["xmax"]))


@pytest.mark.parametrize("N,cells", CELLS)
@pytest.mark.parametrize("surface,kind", [("llf", "smooth"), ("hll", "smooth"), ("llf", "nodal"),
                                          ("hll", "jumps")])
def test_rhs_parity(N, cells, surface, kind):
    cfg = _cfg(N, cells, surface)
    o, s = oracle.Oracle(**cfg), dgx.Solver(**cfg)
    u = _state(o, cfg, kind)
    print("case", N, cells, surface, kind, flush=True)
    e = err_v(host(s.rhs(dev(u))), o.rhs(u), u, 3, 2.0 * math.pi / max(cells))
    assert s.check() == 0
    assert np.all(e <= TOL_FP64), e


@pytest.mark.parametrize("N,cells,kind", [
    (3, (29, 27, 27), "smooth"), (3, (37, 35, 33), "smooth"), (3, (29, 27, 27), "nodal"),
    (4, (24, 23, 23), "smooth"), (5, (19, 17, 16), "smooth"), (6, (8, 11, 11), "smooth"),
    (7, (21, 20, 20), "smooth"), (5, (19, 17, 16), "nodal")])
def test_steps_parity(N, cells, kind):
    """Two adaptive steps: the second's dt comes from the wave speeds of the first's last stage."""
    cfg = _cfg(N, cells, "llf")
    o, s = oracle.Oracle(**cfg), dgx.Solver(**cfg)
    u = _state(o, cfg, kind)
    print("case", N, cells, kind, flush=True)
    ref, tref = o.step(u, 2, cfl=0.5)
    ud, t = dev(u), dev(np.zeros(1))
    s.step(ud, 2, cfl=0.5, t=t)
    assert s.check() == 0
    assert np.all(state_err(host(ud), ref, 3) <= TOL_FP64)
    assert abs(float(t.item()) - tref) <= 1e-12 * tref


def test_non_physical_state_raises_the_flag():
    cfg = _cfg(3, (32, 32, 20), "llf")
    s = dgx.Solver(**cfg)
    u = inputs.constant_state((s.E, s.NN), 3)
    u[0, s.E - 1, 63] = -1.0
    s.rhs(dev(u))
    assert s.check() == 1


@pytest.mark.parametrize("runs", [[(5, (19, 17, 16)), (3, (5, 4, 3)), (4, (24, 23, 23)), (5, (4, 4, 3))],
                                  [(5, (18, 17, 17)), (3, (28, 28, 27))]])
def test_batch_equals_single_runs(runs):
    """Runs on both sides of the rule in one ensemble (and an ensemble of large runs alone):
    bitwise the results of each run alone, for even and odd step counts and for the
    right-hand side."""
    cfgs = [_cfg(N, cells, "llf") for N, cells in runs]
    singles = [dgx.Solver(**c) for c in cfgs]
    us = [inputs.tgv(s.node_coords(), perturb_seed=30 + i).contiguous() for i, s in enumerate(singles)]
    b = dgx.Batch(cfgs)
    print("case", runs, flush=True)
    dus = [torch.empty_like(u) for u in us]
    b.rhs(us, dus)
    for r, s in enumerate(singles):
        assert torch.equal(dus[r], s.rhs(us[r])), r
    for steps in (2, 3):
        ub = [u.clone() for u in us]
        tb = torch.zeros(len(us), dtype=torch.float64, device="cuda")
        b.step(ub, steps, cfl=0.5, t=tb)
        for r, s in enumerate(singles):
            u, t = us[r].clone(), torch.zeros(1, dtype=torch.float64, device="cuda")
            s.step(u, steps, cfl=0.5, t=t)
            assert torch.equal(ub[r], u) and float(tb[r]) == float(t[0]), (steps, r)
    assert b.check() == 0


def test_batch_branches_replayed():
    """The steps' graph, whose branches are the groups of runs, replayed with eager work and
    synchronisations between the replays."""
    runs = [(4, (24, 23, 23)), (5, (19, 17, 16)), (3, (29, 27, 27)), (3, (8, 7, 9)), (4, (3, 2, 2))]
    cfgs = [_cfg(N, cells, "llf") for N, cells in runs]
    singles = [dgx.Solver(**c) for c in cfgs]
    us = [inputs.tgv(s.node_coords(), perturb_seed=50 + i).contiguous() for i, s in enumerate(singles)]
    refs = [u.clone() for u in us]
    b = dgx.Batch(cfgs)
    for steps in (2, 4, 2, 6):
        b.step(us, steps, cfl=0.5)
        for r, s in enumerate(singles):
            s.step(refs[r], steps, cfl=0.5)
            assert torch.equal(us[r], refs[r]), (steps, r)
        us[0].mul_(1.0)
        torch.cuda.synchronize()
    assert b.check() == 0
