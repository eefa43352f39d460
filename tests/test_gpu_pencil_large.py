"""The line-per-thread stages (N = 3) near the largest mesh that they take: their 32-bit byte offsets
into a plane (2.1e9 of 2^32 here).

160^3 elements hold 262 M nodes, 10.5 GB per state (the line lies at 2^28 nodes).  The state is a 32^3
periodic state tiled five times per direction with cells of size exactly 1 on both meshes, and both
run in lines (in blocks of four waves and of one), so every element must have the bits of its copy
in the small mesh, whose parity with the oracle the tests of those kernels establish."""
import math

import pytest
import torch

from paper_2108_06476_amd import dgx, inputs

pytestmark = pytest.mark.gpu

KS, REP = 32, 5


def _tile(u, nv):
    return u.view(nv, KS, KS, KS, 64).repeat(1, REP, REP, REP, 1).view(nv, -1, 64)


def _equal_tiled(big, small, nv):
    b = big.view(nv, REP, KS, REP, KS, REP, KS, 64)
    return bool((b == small.view(nv, 1, KS, 1, KS, 1, KS, 64)).all().item())


@pytest.mark.parametrize("volume,surface", [("ec", "llf"), ("shockcap_hg", "hll")])
def test_rhs_and_step_near_the_limit(volume, surface):
    free, _ = torch.cuda.mem_get_info()
    if free < 80e9:
        pytest.skip(f"needs ~60 GB of free device memory, {free / 1e9:.0f} GB free")
    print("case", volume, surface, flush=True)
    small, big = (dgx.Solver(3, 3, (k,) * 3, (0.0,) * 3, (float(k),) * 3, volume=volume, surface=surface)
                  for k in (KS, KS * REP))
    xyz = small.node_coords()
    us = inputs.tgv((xyz * (2 * math.pi / KS) - math.pi).contiguous(), mach=0.8).contiguous()
    dus = small.rhs(us)
    ub = _tile(us, 5)
    dub = big.rhs(ub)
    assert _equal_tiled(dub, dus, 5), "right-hand side of the tiled state"
    del dub
    for _ in range(2):
        small.step(us, 1, cfl=0.5)
        big.step(ub, 1, cfl=0.5)
    assert small.check() == 0 and big.check() == 0
    assert _equal_tiled(ub, us, 5), "steps of the tiled state"
    big.close()
    small.close()


def test_mhd_rhs_and_step_near_the_limit():
    """Ideal MHD, weak form: 160^3 of the 161^3 elements that a handle takes at N = 3."""
    free, _ = torch.cuda.mem_get_info()
    if free < 110e9:
        pytest.skip(f"needs ~90 GB of free device memory, {free / 1e9:.0f} GB free")
    small, big = dgx.MhdSolver(3, KS), dgx.MhdSolver(3, KS * REP)
    us = inputs.alfven(small.node_coords()).contiguous()
    dus = small.rhs(us)
    ub = _tile(us, 8)
    dub = big.rhs(ub)
    # the cells are five times smaller: the operator's entries are five times as large, up to their
    # rounding (2^-53 of sums whose absolute row sum is 2 lift factors, of fluxes of order one)
    err = (dub.view(8, REP, KS, REP, KS, REP, KS, 64) / REP
           - dus.view(8, 1, KS, 1, KS, 1, KS, 64)).abs().max()
    assert float(err) <= 1e-12 * 6 * KS
    big.step(ub, 2, cfl=0.5)
    assert big.check() == 0 and bool(torch.isfinite(ub).all())
    big.close()
    small.close()
