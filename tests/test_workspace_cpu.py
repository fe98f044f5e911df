"""Workspaces hold what their kernels read and write: no tables for adjoints that run in
bundles."""
import pytest

from paper_1812_03358_amd import workloads as W


@pytest.fixture(scope="module")
def ltm():
    from paper_1812_03358_amd import ltm as m
    m.lib()
    return m


def test_no_tables_for_bundles(ltm):
    # a tile's slabs: the grid's diagonal in an eighth of the default depth (2 voxels)
    g = W.grid(256, 0.625)
    plan = ltm.Plan(g, [W.plenoptic_camera(2048, 128, (2, 1), 512, 30.0)], bind=False)
    assert plan.adjoint_kind() != ltm.ADJOINT_RAYS
    bundled = plan.workspace_bytes()
    t = plan.get_tiling(ltm.ADJOINT)
    plan.set_tiling(ltm.ADJOINT, 0, {"order": 26}, rebind=False)
    tiles = (128 // t.tile_u) * (128 // t.tile_v) * t.splits
    slabs = 256 * 0.625 * 3 ** 0.5 / t.chunk_mm
    assert plan.workspace_bytes() - bundled >= tiles * slabs * 28 > 10e6
    plan.set_tiling(ltm.ADJOINT, 0, t, rebind=False)
    assert plan.workspace_bytes() == bundled
