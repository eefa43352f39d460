"""The weak MHD form on meshes with a line of nodes per thread takes the momentum as it is stored.

With a uniform density the mass equation with LLF interfaces is a sum of stored momenta alone: its
volume sum_m D_im (rho v)_m, its interface mean and a jump of the density that is zero.  So the
result is the same to the bit for every uniform density; momenta formed again as rho (m / rho) would
carry the roundings of that density's quotients.
"""
import numpy as np
import pytest
import torch

from paper_2108_06476_amd import dgx

from gpu_util import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,K", [(3, 16), (4, 14), (5, 12), (3, 8)])
def test_mass_equation_sees_the_stored_momentum(N, K):
    s = dgx.MhdSolver(N, K, surface="llf", volume="weak")
    rng = np.random.default_rng(60 + N)
    m = rng.uniform(-1.0, 1.0, (3, s.E, s.NN))
    got = []
    for rho in (1.0, 1.2345678901234567, 0.7071067811865476):
        u = np.zeros(s.shape)
        u[0], u[1:4], u[5:8] = rho, m, 0.1
        u[4] = 10.0 + 0.5 * (m ** 2).sum(axis=0) / rho
        got.append(s.rhs(dev(u))[0])
    assert s.check() == 0
    assert torch.equal(got[0], got[1]) and torch.equal(got[0], got[2])
