"""Ensembles whose runs take several kernels (element tiles, a line of nodes per thread by degree):
the groups of runs overlap in every step, also the last of an odd count, which is not replayed from
the graph of a pair; and in a step that the caller's program records itself."""
import math
import time

import pytest
import torch

from paper_2108_06476_amd import dgx, inputs

pytestmark = pytest.mark.gpu


def _batch(runs):
    cfgs = [inputs.ensemble_config(dict(N=N, K=K)) for N, K in runs]
    us = [inputs.tgv(dgx.Solver(**c).node_coords(), perturb_seed=70 + i).contiguous()
          for i, c in enumerate(cfgs)]
    return cfgs, dgx.Batch(cfgs), us


def _time(f, n):
    best = math.inf
    for _ in range(9):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(n):
            f()
        torch.cuda.synchronize()
        best = min(best, (time.perf_counter() - t0) / n)
    return best


@pytest.mark.parametrize("runs", [[(3, 8), (4, 24), (5, 12), (5, 12), (5, 24)],
                                  [(4, 8), (4, 12), (4, 12), (4, 24), (5, 8), (5, 8), (5, 24)]])
def test_single_step_overlaps_its_groups(runs):
    """A call of one step against half a call of two.  Beyond the same stages it reads the state
    (wave speeds) and copies it, 120 bytes a node where a step moves 720 and computes: a tenth at
    the rates of both; bound 1.13 (a launch in turn for every group and stage: 1.18)."""
    _, b, us = _batch(runs)
    t = torch.zeros(len(runs), dtype=torch.float64, device="cuda")
    one = _time(lambda: b.step(us, 1, cfl=1e-9, t=t), 10)
    two = _time(lambda: b.step(us, 2, cfl=1e-9, t=t), 10)
    assert b.check() == 0
    print(f"{len(runs)} runs: one step {one * 1e6:.1f} us, two {two * 1e6:.1f} us", flush=True)
    assert one <= 1.13 * two / 2


def test_odd_steps_recorded_by_the_caller():
    """One step and a right-hand side captured in the caller's own graph, replayed with eager work
    and synchronisations between the replays: bitwise the steps of each run alone."""
    runs = [(4, 24), (3, 8), (5, 18), (3, 28)]
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        cfgs, b, us = _batch(runs)
        singles = [dgx.Solver(**c) for c in cfgs]
        refs = [u.clone() for u in us]
        dus = [torch.empty_like(u) for u in us]
        start = [u.clone() for u in us]
        b.rhs(us, dus)          # binds the arrays that the graph uses
        b.step(us, 1, cfl=0.3)
        for u, s in zip(us, start):
            u.copy_(s)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=side):
            b.step(us, 1, cfl=0.3)
        for rep in range(4):
            g.replay()
            for s, r in zip(singles, refs):
                s.step(r, 1, cfl=0.3)
            torch.cuda.synchronize()
            for i, (u, r) in enumerate(zip(us, refs)):
                assert torch.equal(u, r), (rep, i)
            us[0].mul_(1.0)
        assert b.check() == 0


def test_tuning_ranks_the_tiled_runs_only():
    """The tile shape is that of the runs in element tiles: with none of them tuning leaves it alone
    (timings of launches that do not depend on it would pick one by chance)."""
    _, b, us = _batch([(5, 24), (4, 24), (3, 28)])
    before = [u.clone() for u in us]
    shape = b.set_shape(256, 0)
    for _ in range(8):
        assert b.tune(us, budget_ms=200) == shape
    b.step(us, 2, cfl=0.3)
    singles = [dgx.Solver(**inputs.ensemble_config(dict(N=N, K=K))) for N, K in [(5, 24), (4, 24), (3, 28)]]
    for s, u0, u in zip(singles, before, us):
        s.step(u0, 2, cfl=0.3)
        assert torch.equal(u, u0)
