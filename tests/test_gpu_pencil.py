"""Large 3D N = 3 meshes, where the stage runs with a line of nodes per thread: parity with the
oracle at the edges of its split (elements that do not fill a wave of four or a block of
sixteen, one or two elements along a direction, both block sizes), on smooth states, on states
whose pairs all lie beyond the near-equal series of the logarithmic means, and on the time
steps' own path (wave speeds, update).  Tolerances: the float64 parity bars of gpu_util.
"""
import math

import numpy as np
import pytest

import oracle
from paper_2108_06476_amd import dgx, inputs

from gpu_util import TOL_FP64, dev, err_v, host, state_err

pytestmark = pytest.mark.gpu

# 20 480 elements and more run with a line per thread, 40 960 and more in blocks of four waves
CELLS = [(32, 32, 20), (29, 27, 27), (1, 150, 140), (2, 129, 81), (37, 35, 33)]


def _cfg(cells, surface):
    hi = tuple(2.0 * math.pi * c / max(cells) for c in cells)
    return dict(dim=3, polydeg=3, cells=cells, xmin=(0.0,) * 3, xmax=hi, gamma=1.4, volume="ec",
                surface=surface)


def _state(o, cfg, kind):
    if kind == "nodal":
        return inputs.random_nodal((o.E, o.NN), 3, 17)
    if kind == "jumps":   # ratios up to 1e4 between neighbours
        return inputs.random_nodal((o.E, o.NN), 3, 18, rho_range=(1e-2, 10.0), p_range=(1e-3, 10.0))
    return inputs.random_smooth(o.node_coords(), 19, periods=list(cfg["xmax"]))


@pytest.mark.parametrize("cells", CELLS)
@pytest.mark.parametrize("surface,kind", [("llf", "smooth"), ("hll", "smooth"), ("llf", "nodal"),
                                          ("hll", "jumps")])
def test_rhs_parity(cells, surface, kind):
    cfg = _cfg(cells, surface)
    o, s = oracle.Oracle(**cfg), dgx.Solver(**cfg)
    u = _state(o, cfg, kind)
    print("case", cells, surface, kind, flush=True)
    e = err_v(host(s.rhs(dev(u))), o.rhs(u), u, 3, 2.0 * math.pi / max(cells))
    assert s.check() == 0
    assert np.all(e <= TOL_FP64), e


@pytest.mark.parametrize("cells,kind", [((29, 27, 27), "smooth"), ((37, 35, 33), "smooth"),
                                        ((29, 27, 27), "nodal")])
def test_steps_parity(cells, kind):
    """Two adaptive steps: the second's dt comes from the wave speeds of the first's last stage."""
    cfg = _cfg(cells, "llf")
    o, s = oracle.Oracle(**cfg), dgx.Solver(**cfg)
    u = _state(o, cfg, kind)
    print("case", cells, kind, flush=True)
    ref, tref = o.step(u, 2, cfl=0.5)
    ud, t = dev(u), dev(np.zeros(1))
    s.step(ud, 2, cfl=0.5, t=t)
    assert s.check() == 0
    assert np.all(state_err(host(ud), ref, 3) <= TOL_FP64)
    assert abs(float(t.item()) - tref) <= 1e-12 * tref


def test_non_physical_state_raises_the_flag():
    cfg = _cfg((32, 32, 20), "llf")
    s = dgx.Solver(**cfg)
    u = inputs.constant_state((s.E, s.NN), 3)
    u[0, s.E - 1, 63] = -1.0
    s.rhs(dev(u))
    assert s.check() == 1
