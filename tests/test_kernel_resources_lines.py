"""Register budgets of the stages with a line of nodes per thread and of the stages of meshes past
the cache, from the compiler's resource report of the last build.

A line per thread pays at two waves per SIMD with the line, its sums and its neighbours in registers:
a build that spills more than a few of them, or falls to one wave, loses what the split gains.  The
stages that store past the cache are kernels of their own, so that the plain ones carry no branch
for it, and keep the waves of those.
"""
import json
import os

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
RES = os.path.join(ROOT, "paper_2108_06476_amd", "_build", "resources.json")

# mangled-name prefix -> (kernels, minimum waves per SIMD, largest spill in bytes per lane)
BUDGETS = {
    "_ZN3dgx8k_pencilILi3E": (6, 2, 0),   # right-hand side and step: waves alone, in fours, blended
    "_ZN3dgx8k_pencilILi4E": (2, 2, 0),
    "_ZN3dgx8k_pencilILi5E": (2, 2, 32),
    "_ZN3dgx8k_pencilILi6E": (2, 2, 0),
    "_ZN3dgx8k_pencilILi7E": (2, 2, 32),
    "_ZN3dgx14k_batch_pencilILi": (6, 2, 32),
    "_ZN3dgx12k_pencil_mhdILi3E": (4, 2, 0),
    "_ZN3dgx12k_pencil_mhdILi4E": (1, 2, 0),
    "_ZN3dgx12k_pencil_mhdILi5E": (2, 2, 32),
    "_ZN3dgx10k_stage_ntILi3ELi3ELi0EfE": (1, 4, 0),   # mixed precision
    "_ZN3dgx10k_stage_ntILi3ELi3ELi1EdE": (1, 4, 0),   # central
    "_ZN3dgx10k_stage_ntILi3ELi3ELi2EdE": (1, 4, 0),   # shock capturing
    "_ZN3dgx10k_stage_ntILi3ELi3ELi3EdE": (1, 4, 0),   # weak form
    "_ZN3dgx15k_stage_curv_ntILi3ELi0EEE": (1, 3, 0),
}


@pytest.mark.parametrize("prefix", sorted(BUDGETS))
def test_occupancy_and_spills(prefix):
    if not os.path.exists(RES):
        pytest.skip("no resource report: build the library first")
    count, waves, spill = BUDGETS[prefix]
    hits = {k: v for k, v in json.load(open(RES)).items() if k.startswith(prefix)}
    assert len(hits) == count, sorted(hits)
    for name, r in hits.items():
        assert r["occupancy"] >= waves, (name, r)
        assert r["scratch"] <= spill, (name, r)
