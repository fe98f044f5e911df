"""The convolution kernels (forward, input and weight gradient) at the edges of their dispatch: each channel count and
channel-tile split of the whole-halo and of the plane-by-plane kernel, blocks
that end inside a tile in x, y and z, concatenated and upsampled inputs, channel
counts left to the general kernel, and outputs whose channels or alignment forbid
four-channel stores.  Against the FP64 oracle on BF16 operands, at the tolerances
of test_nn_gpu."""
import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import test_nn_gpu as T

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nn():
    from paper_1812_03358_amd import nn as N
    N._lib()
    return N


CASES = [
    # whole halo (at least 256 workgroups, or at most 16 channels)
    (9, 5, 17, 16, 0, 64, 3, 0), (9, 5, 17, 16, 0, 128, 3, 0), (17, 9, 33, 8, 8, 32, 3, 0),
    (57, 33, 17, 32, 0, 16, 3, 0), (57, 33, 17, 16, 16, 32, 3, 0), (57, 33, 17, 32, 0, 64, 3, 0),
    (57, 33, 17, 32, 0, 128, 3, 0), (58, 34, 18, 32, 0, 32, 3, 1),
    (29, 33, 17, 64, 0, 16, 3, 0), (29, 33, 17, 32, 32, 32, 3, 0), (29, 33, 17, 64, 0, 64, 3, 0),
    # plane by plane: one, two and four channel tiles per workgroup
    (30, 33, 17, 128, 0, 64, 3, 0), (15, 33, 17, 96, 0, 64, 3, 0), (7, 6, 17, 96, 0, 128, 3, 0),
    (3, 5, 19, 32, 64, 16, 3, 0), (10, 6, 18, 64, 0, 32, 3, 1), (1, 1, 1, 32, 0, 16, 3, 0),
    # weight gradient: rows of each chunk length, ended inside a chunk, one row of
    # one voxel past a chunk, one input channel, rows of 16 and of 8 voxels
    (2, 3, 65, 16, 0, 16, 3, 0), (2, 3, 127, 8, 8, 16, 3, 0), (3, 2, 129, 16, 0, 32, 3, 0), (4, 4, 62, 16, 16, 16, 3, 1),
    (2, 3, 33, 1, 0, 16, 3, 0), (3, 2, 100, 1, 0, 32, 3, 0), (2, 4, 16, 16, 0, 16, 3, 0), (2, 4, 8, 16, 0, 16, 3, 0),
    # the general kernels
    (7, 6, 5, 40, 0, 16, 3, 0), (5, 6, 7, 56, 0, 24, 3, 0), (4, 5, 6, 72, 0, 16, 3, 0),
]


@pytest.mark.parametrize("case", CASES)
def test_conv_dispatch(nn, case):
    T.test_conv_forward_dgrad_wgrad(nn, case)


@pytest.mark.parametrize("cin,cout,split,shift", [(16, 20, 20, 0), (32, 20, 12, 0), (32, 18, 7, 0), (16, 16, 16, 2),
                                                  (128, 16, 8, 2)])
def test_conv_store_forms(nn, cin, cout, split, shift):
    """Any split and any element alignment of the two outputs, BF16 and FP32."""
    lib = nn._lib()
    D, H, W = 3, 5, 18
    g = torch.Generator().manual_seed(cin + cout)
    x = torch.randn(D, H, W, cin, generator=g).bfloat16()
    w = (torch.randn(cout, 27, cin, generator=g) * (27 * cin) ** -0.5).bfloat16()
    b = torch.randn(cout, generator=g)
    ref = torch.nn.functional.conv3d(x.double().permute(3, 0, 1, 2)[None],
                                     w.double().reshape(cout, 3, 3, 3, cin).permute(0, 4, 1, 2, 3), b.double(), padding=1)
    ref = ref[0].permute(1, 2, 3, 0).reshape(-1, cout).clamp(min=0).numpy()
    wd = w.float().reshape(cout, -1).cuda()
    nf, nb = ctypes.c_uint64(), ctypes.c_uint64()
    assert lib.ltm_nn_packed_sizes(cout, cin, 3, ctypes.byref(nf), ctypes.byref(nb)) == 0
    wf = torch.empty(nf.value, dtype=torch.int16, device="cuda")
    assert lib.ltm_nn_pack_weights(nn._p(wd), cout, cin, 3, nn._p(wf), None, None) == 0
    xd, bd = x.view(torch.int16).cuda(), b.cuda()
    for f32 in (0, 1):
        dt = torch.float32 if f32 else torch.bfloat16
        o = [torch.full((D * H * W * c + 8,), 7.0, dtype=dt, device="cuda") for c in (split, max(cout - split, 1))]
        d = nn.ConvDesc(ksize=3, d=D, h=H, w=W, c0=cin, c1=0, cout=cout, upsample=0, relu=1, out_f32=f32, split=split)
        assert lib.ltm_nn_conv3d_forward(ctypes.byref(d), nn._p(xd), None, nn._p(wf), nn._p(bd), nn._p(o[0][shift:]),
                                         nn._p(o[1][shift:]) if cout > split else None, None) == 0
        for c, out, part in ((split, o[0], ref[:, :split]), (cout - split, o[1], ref[:, split:])):
            if not c:
                continue
            got = out.double().cpu().numpy()
            n = D * H * W * c
            assert (got[:shift] == 7).all() and (got[shift + n:] == 7).all()
            err = np.abs(got[shift:shift + n].reshape(-1, c) - part)
            # one BF16 rounding (2^-9 of the value) and FP32 sums of values of order 1
            assert (err <= (0 if f32 else 2.0 ** -8) * np.abs(part) + 2e-5).all()


@pytest.mark.parametrize("W,cin", [(33, 16), (16, 32), (33, 1)])
def test_wgrad_of_element_aligned_buffers(nn, W, cin):
    """Buffers aligned to an element only take the gathering kernels."""
    lib = nn._lib()
    D, H, cout = 2, 3, 16
    g = torch.Generator().manual_seed(W + cin)
    x = torch.randn(D * H * W * cin + 3, generator=g).bfloat16().view(torch.int16).cuda()
    dy = torch.randn(D * H * W * cout + 3, generator=g).bfloat16().view(torch.int16).cuda()
    desc = nn.conv_desc(3, D, H, W, cin, 0, cout, 0, relu=0, out_f32=1)
    got = []
    for a, b in ((x[3:], dy[3:]), (x[3:].clone(), dy[3:].clone())):
        dw = torch.zeros(cout, 27 * cin, device="cuda")
        assert lib.ltm_nn_conv3d_wgrad(ctypes.byref(desc), nn._p(a), None, nn._p(b), nn._p(dw), None) == 0
        got.append(dw.cpu().numpy())
    assert T.rel(got[0], got[1]) < 1e-5
