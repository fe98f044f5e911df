"""The transport's staged passes at the edges of their compiled band widths:
the smallest and the largest, the first and the last width of a kernel that
serves several, the first that leaves the staged path, detectors one pixel to
either side of the four-row limit, and rows that are no multiple of four.
Bars: relative L2 <= 1e-5 against the FP64 oracle (FP32 table entries and
stored intermediates, sums in FP64 or of at most a band's FP32 products)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import transport as OT
from paper_1812_03358_amd import workloads as W

pytestmark = pytest.mark.gpu
DIMS = (9, 7, 5)


def check(g, cam, width, project, backproject):
    from paper_1812_03358_amd import ltm
    op = ltm.Transport(g, cam, 1)
    assert op.bands()[2] == width
    x = W.uniform_random(int(np.prod(DIMS)), seed=11).reshape(DIMS[::-1])
    y = W.uniform_random(cam["det_nu"] * cam["det_nv"], seed=12)
    Ax = op.project(torch.from_numpy(x.reshape(-1)).cuda()).cpu().numpy().astype(np.float64)
    Aty = op.backproject(torch.from_numpy(y).cuda()).cpu().numpy().astype(np.float64)
    rx = np.asarray(project(g, cam, x, 1), np.float64).reshape(-1)
    ry = np.asarray(backproject(g, cam, y, 1), np.float64).reshape(-1)
    assert np.linalg.norm(Ax - rx) <= 1e-5 * np.linalg.norm(rx) > 0
    assert np.linalg.norm(Aty - ry) <= 1e-5 * np.linalg.norm(ry) > 0


@pytest.mark.parametrize("pitch,width,det,rows", [(0.06, 2, 130, 21), (0.14, 3, 130, 21), (0.68, 8, 130, 21),
                                                  (1.58, 16, 130, 21), (1.7, 17, 130, 21), (1.8, 18, 130, 21),
                                                  (2.38, 23, 130, 21), (2.46, 24, 130, 21), (2.58, 25, 130, 21),
                                                  (0.5, 6, 4096, 5), (0.5, 6, 4097, 5)])
def test_single_lens_band_widths(pitch, width, det, rows):
    check(W.grid(DIMS, pitch), W.single_lens_camera(det, (2, 2), 8, det_v=rows), width,
          OT.project, OT.backproject)


@pytest.mark.parametrize("pitch,width", [(0.42, 3), (1.18, 5), (2.24, 8), (2.66, 9), (2.98, 10), (3.74, 12),
                                         (4.18, 13), (5.2, 16), (5.7, 17), (6.68, 20), (7.18, 21), (8.16, 24),
                                         (8.64, 25)])
def test_plenoptic_band_widths(pitch, width):
    check(W.grid(DIMS, pitch), W.plenoptic_camera(72, 9, (2, 2), 8), width,
          OT.project_plenoptic, OT.backproject_plenoptic)
