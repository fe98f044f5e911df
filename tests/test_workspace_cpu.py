"""Workspaces hold what their kernels read and write: no tables for adjoints that run in
bundles, and a transport's intermediate for the groups of angular rows that it filters."""
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


def test_transport_intermediate(ltm):
    # an 8 x 8 aperture has rows of 4, 6 and 8 cells inside its disc: three groups of
    # FP32 intermediates, and tables that take less than two
    import ctypes

    h, n = ctypes.c_void_p(), ctypes.c_uint64()
    g, c = ltm.make_grid(W.grid(100, 1.0)), ltm.make_cameras([W.single_lens_camera(800, (8, 8), 1)])
    assert ltm.lib().ltm_xport_create(ctypes.byref(g), c, ltm.BASIS_PILLBOX, ctypes.byref(h)) == 0
    assert ltm.lib().ltm_xport_workspace_bytes(h, ctypes.byref(n)) == 0
    ltm.lib().ltm_xport_destroy(h)
    one = 4 * 100 * 800 * 100
    assert 3 * one < n.value < 5 * one
