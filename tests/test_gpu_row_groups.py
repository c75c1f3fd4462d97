"""The products whose rows four waves share (rows * 4 <= 8192 waves, eight tiles a
row on average, no row of more than 64): the corner rows, the couplings and, in a
coarse block of more than 64 tile rows, the transposed coarse pass over its list of
nonzero tiles, beside the split forward pass.  Against the monolithic oracle, as
are the launch rules of test_gpu_small_shapes with a maximum that a NaN passes."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import test_gpu_small_shapes as shapes
from workloads.mesh import cube_mesh
from workloads.partition import box_partition

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def nan_is_the_largest(monkeypatch):
    monkeypatch.setattr(shapes, "max", lambda errors: np.max(np.fromiter(errors, float)), raising=False)


def _tiles(n, parts):
    """Tile rows per subdomain (interface, corner) and of the coarse block."""
    from paper_2204_13254_amd.solver import analyze
    c, t, _ = cube_mesh(n)
    a, per = analyze(c, t, box_partition(n, parts))
    up = lambda v: -(-np.asarray(v, dtype=np.int64) // 32)
    return up(per[:, 1]), up(per[:, 2]), int(up(a.n_corner))


@pytest.mark.parametrize("n,parts,nrhs", [(20, 4, 1), (20, 4, 2), (20, 4, 5), (24, 3, 1)])
@pytest.mark.parametrize("precision", ["fp64", "fp32_refine"])
def test_corner_rows(n, parts, nrhs, precision):
    kG, kC, _ = _tiles(n, (parts,) * 3)
    rows, tiles = int(kC.sum()), int((kC * kG).sum())
    assert 0 < 4 * rows <= 8192 and tiles >= 8 * rows and kG[kC > 0].max() <= 64
    assert shapes._steps(n, (parts,) * 3, nrhs, precision) <= shapes.BAR[precision]


@pytest.mark.parametrize("nrhs", [1, 2, 3, 17])
@pytest.mark.parametrize("precision", ["fp64", "fp32_refine"])
def test_coarse_block_of_more_than_64_tile_rows(nrhs, precision):
    # 108 tile rows; the inverse factor's last row holds all of them (split over
    # waves), its longest column 27 tiles (2231 in all)
    _, _, Kc = _tiles(18, (9, 9, 9))
    assert Kc > 64
    assert shapes._steps(18, (9, 9, 9), nrhs, precision) <= shapes.BAR[precision]


@pytest.mark.parametrize("n,parts,nrhs,precision,opt", [
    (5, (2, 2, 1), 1, "fp64", {}), (5, (2, 2, 1), 13, "fp32_refine", {}), (5, (1, 2, 2), 5, "fp64", dict(precond=0)),
    (5, (1, 2, 2), 5, "fp64", dict(method="dp2")), (16, (4, 4, 4), 2, "fp32_refine", {}),
    (12, (3, 3, 3), 31, "fp64", {}), (20, (4, 4, 4), 19, "fp32_refine", {}),
])
def test_launch_rules_over_four_steps(n, parts, nrhs, precision, opt):
    assert shapes._steps(n, parts, nrhs, precision, N=4, **opt) <= shapes.BAR[precision]
