"""How many products a weight gradient sums in one FP32 run.

All inputs and output gradients are 1 but for one gradient of 2^31 at the first voxel,
in one channel: what the run that holds it sums up later is below half a unit of its
last place (128) and lost, 32 products at a time, and no other run's sum is.  The
loss counts the run.  Bounds: the input layer's runs never held more than 16 rows of
a wave's 32 voxels (two million voxels in 1024 shares); rows that a slice-by-slice sum
served held at most one slice, H x W."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,H,W,cin,cout,bound", [(128, 128, 128, 1, 16, 16 * 32), (64, 64, 60, 128, 128, 64 * 60)])
def test_run_length(D, H, W, cin, cout, bound):
    from paper_1812_03358_amd import nn

    lib = nn._lib()
    x = torch.ones(D * H * W * cin, dtype=torch.bfloat16, device="cuda")
    dy = torch.ones(D * H * W * cout, dtype=torch.bfloat16, device="cuda")
    dy[3] = 2.0 ** 31
    dw = torch.zeros(cout, 27, cin, device="cuda")
    desc = nn.conv_desc(3, D, H, W, cin, 0, cout, 0, relu=0, out_f32=1)
    assert lib.ltm_nn_conv3d_wgrad(desc, nn._p(x.view(torch.int16)), None, nn._p(dy.view(torch.int16)), nn._p(dw), None) == 0
    centre = dw[:, 13].double()
    n = D * H * W
    assert (centre[:3] == n).all() and (centre[4:] == n).all()
    lost = (2.0 ** 31 + n - 1) - centre[3]
    print(f"lost {float(lost.min())} .. {float(lost.max())} of {n}, bound {bound}", flush=True)
    assert float(lost.abs().max()) <= bound
