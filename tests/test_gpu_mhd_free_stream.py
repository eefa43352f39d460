"""Free stream of the entropy-conservative MHD volume on meshes with a line of nodes per thread: at
rest and without a field the pair flux reduces to the pressure {{rho}}/(2 {{beta}}), beta =
rho/(2 p), which has to cancel the interface flux's p.

What is left at an end node, in units of p times its lift factor (2/h)/w_0, is the rounding of the
operator's row, the same for every state, and the roundings of the state's own operations, which
spread around it.  Each product or sum contributes a standard deviation of about 5e-17, a reciprocal
of two Newton steps 7e-17: two products and a reciprocal in beta, a reciprocal and two products in
the mean pressure, four additions of partial sums of up to 1.35 lift factors, together 1.9e-16.
Bound: six of them, 1.14e-15, around the mean over 10 240 states.  (A reciprocal of one Newton step is
off by up to 2.3e-15, and by another amount for every state.)

The elements of a row along x share a state: the x momentum sees nothing of the other rows.
"""
import numpy as np
import pytest

import oracle
from paper_2108_06476_amd import dgx

from gpu_util import dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("surface", ["llf", "hll"])
def test_constant_pressure(surface):
    N, K, gamma = 3, 16, 5.0 / 3.0
    s = dgx.MhdSolver(N, K, surface=surface, volume="ec", gamma=gamma)
    lift = K / float(oracle.lgl(N)[1][0])
    rng = np.random.default_rng(11)
    got = []
    for _ in range(40):
        rho, p = rng.uniform(0.5, 2.0, (2, K * K, 1, 1))
        u = np.zeros((8, K * K, K, s.NN))
        u[0], u[4] = rho, p / (gamma - 1)
        du = host(s.rhs(dev(u.reshape(s.shape)))).reshape(8, K * K, K, s.NN)
        got.append(du[1, :, 5, [0, N]] / (p[:, 0, 0] * lift))   # both ends of a line
    assert s.check() == 0
    got = np.concatenate(got, axis=1)
    off = np.abs(got - got.mean(axis=1, keepdims=True)).max()
    print(f"{surface}: means {got.mean(axis=1)}, largest distance from them {off:.2e}", flush=True)
    assert off <= 1.14e-15
