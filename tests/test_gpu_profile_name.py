"""dgx_profile_read names the kernel family of the handle's RK stages, on both sides of the meshes
from which a line of nodes per thread is taken."""
import math

import pytest

from paper_2108_06476_amd import dgx

pytestmark = pytest.mark.gpu


def _solver(kind, polydeg, k, opt):
    if kind == "mhd":
        return dgx.MhdSolver(polydeg, k, **opt)
    if kind == "curv":
        return dgx.CurvSolver(polydeg, k, **opt)
    return dgx.Solver(kind, polydeg, (k,) * kind, (-math.pi,) * kind, (math.pi,) * kind, **opt)


@pytest.mark.parametrize("kind,polydeg,k,opt,name", [
    (2, 3, 8, {}, "k_stage"),
    (3, 3, 27, {}, "k_stage"), (3, 3, 28, {}, "k_pencil"),
    (3, 3, 28, {"precision": "mixed"}, "k_stage"), (3, 3, 28, {"surface": "none"}, "k_stage"),
    (3, 4, 23, {}, "k_stage"), (3, 4, 24, {}, "k_pencil"),
    (3, 5, 17, {}, "k_stage"), (3, 5, 18, {}, "k_pencil"),
    (3, 6, 10, {}, "k_stage"), (3, 6, 11, {}, "k_pencil"),
    (3, 7, 20, {}, "k_stage"), (3, 7, 21, {}, "k_pencil"),
    (3, 3, 25, {"volume": "shockcap_hg"}, "k_stage"), (3, 3, 26, {"volume": "shockcap_hg"}, "k_pencil"),
    ("curv", 3, 8, {}, "k_stage_curv_split"), ("curv", 3, 9, {}, "k_stage_curv"),
    ("mhd", 3, 4, {}, "k_stage_mhd_split"), ("mhd", 3, 17, {}, "k_stage_mhd"),
    ("mhd", 3, 18, {}, "k_pencil_mhd"), ("mhd", 4, 18, {}, "k_stage_mhd"),
    ("mhd", 3, 17, {"volume": "ec", "surface": "ec"}, "k_stage_mhd_ec"),
])
def test_profile_name(kind, polydeg, k, opt, name):
    assert _solver(kind, polydeg, k, opt).profile_read()[2] == name
