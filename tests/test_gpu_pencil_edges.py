"""The line-per-thread stages at the edges of their meshes, against the oracle: the smallest mesh of
each degree and the next odd ones, elements that leave waves of a block of four without work
(N = 3 from 40 960 elements), and time steps with the HLL flux.  States: smooth; nodes within 10 %
(every pair in the middle branch of the logarithmic means); and a mix of both with ratios up to 1e4
in some elements, so that a wave holds all three branches.  Bars: the float64 parity of gpu_util."""
import math

import numpy as np
import pytest
import torch

import oracle
from paper_2108_06476_amd import dgx, inputs

from gpu_util import TOL_FP64, dev, err_v, host, state_err

pytestmark = pytest.mark.gpu

CELLS = [(3, (41, 40, 25)), (4, (27, 25, 20)), (4, (1, 120, 113)), (5, (18, 20, 15)), (5, (72, 1, 76)), (6, (11, 11, 11)),
         (6, (37, 36, 1)), (7, (21, 21, 21)), (7, (98, 97, 1))]


def _cfg(N, cells, surface):
    hi = tuple(2.0 * math.pi * c / max(cells) for c in cells)
    return dict(dim=3, polydeg=N, cells=cells, xmin=(0.0,) * 3, xmax=hi, gamma=1.4, volume="ec",
                surface=surface)


def _state(o, cfg, kind):
    if kind == "middle":
        return inputs.random_nodal((o.E, o.NN), 3, 31, rho_range=(0.9, 1.1), p_range=(0.9, 1.1))
    u = inputs.random_smooth(o.node_coords(), 32, amp=0.01, periods=list(cfg["xmax"]))
    if kind == "mixed":
        u[:, 1::3] = inputs.random_nodal((o.E, o.NN), 3, 33, rho_range=(0.9, 1.1),
                                         p_range=(0.9, 1.1))[:, 1::3]
        u[:, 2::7] = inputs.random_nodal((o.E, o.NN), 3, 34, rho_range=(1e-2, 10.0),
                                         p_range=(1e-3, 10.0))[:, 2::7]
    return u


@pytest.mark.parametrize("N,cells", CELLS)
@pytest.mark.parametrize("surface,kind", [("llf", "smooth"), ("hll", "middle"), ("llf", "mixed")])
def test_rhs_parity(N, cells, surface, kind):
    print("case", N, cells, surface, kind, flush=True)
    cfg = _cfg(N, cells, surface)
    o, s = oracle.Oracle(**cfg), dgx.Solver(**cfg)
    u = _state(o, cfg, kind)
    e = err_v(host(s.rhs(dev(u))), o.rhs(u), u, 3, 2.0 * math.pi / max(cells))
    assert s.check() == 0
    assert np.all(e <= TOL_FP64), e


@pytest.mark.parametrize("N,cells,surface,kind", [
    (3, (41, 40, 25), "hll", "middle"), (3, (32, 32, 20), "hll", "smooth"),
    (4, (27, 25, 20), "hll", "middle"), (5, (18, 20, 15), "hll", "middle"), (6, (11, 11, 11), "hll", "middle"),
    (7, (21, 21, 21), "hll", "middle"), (7, (22, 21, 21), "llf", "smooth")])
def test_steps_parity(N, cells, surface, kind):
    """Two adaptive steps: the second's dt comes from the wave speeds of the first's last stage."""
    print("case", N, cells, surface, kind, flush=True)
    cfg = _cfg(N, cells, surface)
    o, s = oracle.Oracle(**cfg), dgx.Solver(**cfg)
    u = _state(o, cfg, kind)
    ref, tref = o.step(u, 2, cfl=0.2)
    ud, t = dev(u), torch.zeros(1, dtype=torch.float64, device="cuda")
    s.step(ud, 2, cfl=0.2, t=t)
    assert s.check() == 0
    d = state_err(host(ud), ref, 3)
    assert np.all(d <= TOL_FP64), d
    assert abs(float(t.item()) - tref) <= 1e-12 * tref
