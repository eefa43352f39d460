"""The two elements of an interface evaluate one flux: what leaves the one enters the other.

The kernels with a line of nodes per thread form a face's flux once in each of its elements.  The
weighted sum of the right-hand side over the mesh then vanishes to the rounding of its terms.  Two
terms of that sum are systematic in every kernel, the rounding of the operator's table entries
(eps times the mean of the fluxes), and would hide a flux that differs between the two sides.  So
the state moves along y on average, in cells 1e6 times longer in y than in x and z: the fluxes of
mass, y momentum and energy through the x and z faces vanish in the mean, those through the y faces
by the cells' shape, and a side that sees another y momentum than its neighbour shows in full (the
dissipation lambda [[rho v_y]] has a part of one sign).

Bound: an entry of the right-hand side carries at most K = 32 roundings of the size
A = (2/h) max(|flux|, lambda |u|), independent from node to node; six standard deviations of the
mean over M nodes are 6 K 2^-53 A / sqrt(M).
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2108_06476_amd import dgx, inputs

from gpu_util import dev, host

pytestmark = pytest.mark.gpu

CELLS = {3: (32, 32, 20), 4: (28, 27, 27), 5: (19, 18, 18), 6: (12, 12, 11), 7: (22, 21, 21)}


def _state(xyz, cells, seed):
    periods = [2.0 * c for c in cells]
    rng = np.random.default_rng(seed)

    def field():   # a zero-mean random Fourier sum, |field| <= 1
        g, total = np.zeros_like(xyz[0]), 0.0
        for _ in range(4):
            k = rng.integers(1, 3, size=3) * rng.choice([-1, 1], size=3)
            arg = sum(2 * np.pi * k[d] * (xyz[d] / periods[d]) for d in range(3))
            a = rng.uniform(0.5, 1.0)
            g += a * np.sin(arg + rng.uniform(0, 2 * np.pi))
            total += a
        return g / total

    rho = 1.0 + 0.02 * field()
    vel = [0.05 * field(), 0.8 + 0.05 * field(), 0.05 * field()]
    return rho, vel, 1.0 + 0.02 * field()


@pytest.mark.parametrize("N,surface,volume", [(3, "llf", "ec"), (3, "hll", "ec"), (4, "llf", "ec"),
                                              (5, "hll", "ec"), (6, "llf", "ec"), (7, "llf", "ec"),
                                              (3, "llf", "shockcap_hg"), (3, "hll", "shockcap_hg")])
def test_interfaces_conserve(N, surface, volume):
    print("case", N, surface, volume, flush=True)
    cells = CELLS[N]
    stretch = (1.0, 1.0e6, 1.0)
    s = dgx.Solver(3, N, cells, (0.0,) * 3, tuple(2.0 * c * f for c, f in zip(cells, stretch)),
                   volume=volume, surface=surface)
    xyz = host(s.node_coords()) / np.array(stretch)[:, None, None]
    rho, vel, p = _state(xyz, cells, 41 + N)
    u = inputs.prim_to_cons(rho, vel, p)
    if volume == "shockcap_hg":
        alpha = np.random.default_rng(5).uniform(0.0, 1.0, s.E)
        du = host(s.rhs_alpha(dev(u), dev(alpha)))
    else:
        du = host(s.rhs(dev(u)))
    assert s.check() == 0
    w = oracle.lgl(N)[1]
    w3 = (w[:, None, None] * w[None, :, None] * w[None, None, :]).reshape(-1) / 8.0   # sum 1
    mean = (du.astype(np.longdouble) * w3).sum(axis=(1, 2)) / s.E
    lam = np.abs(vel[0]).max() + np.sqrt(1.4 * p / rho).max()
    A = lam * np.abs(u).reshape(5, -1).max(axis=1)      # 2/h = 1
    bound = 6 * 32 * 2.0 ** -53 * A / np.sqrt(float(s.num_nodes))
    print("mean / bound", (np.abs(mean) / bound).astype(float), flush=True)
    for v in (0, 2, 4):
        assert abs(float(mean[v])) <= bound[v], (v, float(mean[v]), bound[v])
