"""The bundled adjoint with a wave to a unit and with a workgroup to one, each known to
be what runs: against the oracle and the ray-by-ray adjoint, with values out of range,
in view subsets, in batches of one kind and of several, and with one FP64 accumulator for
cameras that are faster into one each.  Tolerances of test_bundles_gpu."""
import numpy as np
import pytest

import test_bundles_gpu as T
from paper_1812_03358_amd import workloads as W

pytestmark = pytest.mark.gpu

RAYS, WAVES, GROUPS = 0, 1, 2
PHI = (45.0, 30.0, 120.0, 0.0)   # windows of 3 to 5 voxels, both accumulators
CASES = {
    "waves": (WAVES, W.grid((40, 36, 38), 3.0), [W.plenoptic_camera(192, 16, (8, 1), 80, p) for p in PHI]),
    "groups": (GROUPS, W.grid((40, 36, 38), 3.0), [W.plenoptic_camera(160, 10, (2, 2), 80, p) for p in PHI]),
    # units larger than what a wave (128) and a workgroup (576) hold at once
    "waves_large_units": (WAVES, W.grid((20, 24, 18), 6.0), [W.plenoptic_camera(480, 16, (4, 1), 37, 20.0)]),
    "groups_large_units": (GROUPS, W.grid((20, 24, 18), 6.0), [W.plenoptic_camera(360, 12, (2, 2), 37, 20.0)]),
    # cell counts around the passes of 16
    "waves_17": (WAVES, W.grid((20, 18, 16), 8.0), [W.plenoptic_camera(272, 17, (2, 2), 37)]),
    "waves_33": (WAVES, W.grid((24, 20, 32), 5.0), [W.plenoptic_camera(272, 17, (2, 2), 64)]),
    # hexagonal lenslets of many and of few pixels, pixel blocks of a single lens
    "groups_hex": (GROUPS, W.grid((30, 26, 28), 2.0), [W.hex_plenoptic_camera(560, None, (2, 2), 60, 25.0)]),
    "groups_single": (GROUPS, W.grid((24, 20, 22), 4.0), [W.single_lens_camera(53, (8, 8), 50, 30.0, det_v=41)]),
    "waves_single": (WAVES, W.grid((24, 20, 22), 4.0), [W.single_lens_camera(403, (1, 1), 50, 20.0, det_v=341)]),
    "rays_hex": (RAYS, W.grid((30, 26, 28), 2.0), [W.hex_plenoptic_camera(200, None, (2, 2), 60, 25.0)]),
}


@pytest.fixture(scope="module")
def ltm():
    from paper_1812_03358_amd import ltm as m
    return m


def _plans(ltm, name):
    kind, g, cams = CASES[name]
    a, b = T._plans(ltm, g, cams)
    assert all(a.adjoint_kind(k) == kind and b.adjoint_kind(k) == RAYS for k in range(len(cams)))
    return a, b


@pytest.mark.parametrize("name", sorted(CASES))
def test_kind_against_oracle_and_rays(ltm, name, monkeypatch):
    _plans(ltm, name)
    monkeypatch.setitem(T.CASES, name, CASES[name][1:])
    T.test_bundled_adjoint(ltm, name)


@pytest.mark.parametrize("value", [float("inf"), float("nan"), 3e38])
@pytest.mark.parametrize("name", ["waves", "groups"])
def test_values_out_of_range(ltm, name, value):
    # a few such pixels: the voxels their rays do not touch are as without them
    import torch

    a, b = _plans(ltm, name)
    _, g, cams = CASES[name]
    _, y = T._inputs(g, cams, 73)
    side = cams[0]["det_nu"]
    k = [(side // 2 + 8) * side + side // 2 + 8, (side // 2 - 7) * side + side // 2 + 4]
    yd = torch.from_numpy(y).cuda()
    yd[k] = 0.0
    clean = a.backproject(yd).cpu().numpy()
    one = torch.zeros_like(yd)
    one[k] = 1.0
    touched = b.backproject(one).cpu().numpy() != 0.0
    assert 0 < touched.sum() < touched.size
    yd[k] = value
    x = a.backproject(yd).cpu().numpy()
    assert np.allclose(x[~touched], clean[~touched], rtol=1e-5, atol=1e-6 * np.abs(clean).max())
    if value == 3e38:
        assert np.abs(x[touched]).max() > 1e30
    else:
        assert not np.isfinite(x[touched]).all()


@pytest.mark.parametrize("name", ["waves", "groups"])
def test_subsets(ltm, name):
    import torch

    a, _ = _plans(ltm, name)
    _, g, cams = CASES[name]
    yd = torch.from_numpy(T._inputs(g, cams, 75)[1]).cuda()
    full = a.backproject(yd).double()
    parts = torch.zeros_like(full)
    for i in range(4):
        a.set_ray_subset(4, i)
        parts += a.backproject(yd).double() / 4
    assert float((parts - full).norm() / full.norm()) < 1e-6


@pytest.mark.parametrize("names", [("waves",), ("groups",), ("waves", "groups"), ("waves", "rays"),
                                   ("groups", "rays"), ("waves", "rays", "groups")])
def test_batch_of_kinds(ltm, names):
    import torch

    plans = []
    for n in names:
        a, b = _plans(ltm, "waves" if n == "rays" else n)
        plans.append(b if n == "rays" else a)
    gen = torch.Generator(device="cuda").manual_seed(5)
    xs = [torch.rand(p.n_voxels, device="cuda", generator=gen) for p in plans]
    ys = [torch.empty(p.n_meas, device="cuda") for p in plans]
    outs = [torch.empty_like(x) for x in xs]
    ltm.Batch(plans, xs, ys, outs).sweep()
    for p, x, o in zip(plans, xs, outs):
        want = p.backproject(p.project(x)).double()
        assert float((o.double() - want).norm() / want.norm()) < 1e-6


def test_batch_of_more_units_than_items(ltm):
    # 1.6 million units: a batch camera's work items number less than 2^20, so an item
    # covers two of them
    import torch

    plan = ltm.Plan(W.grid(64, 4.0), [W.single_lens_camera(4096, (8, 8), 3, det_v=3072)])
    assert plan.adjoint_kind() == GROUPS
    x, y = torch.rand(plan.n_voxels, device="cuda"), torch.empty(plan.n_meas, device="cuda")
    out = torch.empty_like(x)
    ltm.Batch([plan], [x], [y], [out]).sweep()
    want = plan.backproject(plan.project(x)).double()
    assert float((out.double() - want).norm() / want.norm()) < 1e-6
    plan.set_tiling(ltm.ADJOINT, 0, {"order": 26})
    rays = plan.backproject(y).double()
    assert float((out.double() - rays).norm() / rays.norm()) < 1e-6


def test_time_of_rows_of_a_power_of_two_blocks(ltm):
    # rows of 128 blocks keep no XCD to the same columns: 1024^2 pixels take no longer
    # than 1016^2 do, but for their number (twice as long before)
    import torch

    def ms(det):
        plan = ltm.Plan(W.grid(100, 1.0), [W.single_lens_camera(det, (4, 4), 200)])
        assert plan.adjoint_kind() != RAYS
        y, x = torch.rand(plan.n_meas, device="cuda"), torch.empty(plan.n_voxels, device="cuda")
        t = []
        for _ in range(5):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            plan.backproject(y, x)
            b.record()
            b.synchronize()
            t.append(a.elapsed_time(b))
        return min(t)

    a, b = ms(1016), ms(1024)
    print(f"1016: {a:.2f} ms, 1024: {b:.2f} ms", flush=True)
    assert b < 1.5 * a


def test_one_accumulator_for_both_orientations(ltm):
    # between 2^22 and 2^23 voxels the fixed accumulator of the allocation-free entry
    # point holds one of the two that these cameras call for
    import torch

    g = W.grid((164, 162, 160), 1.0)
    cams = [W.plenoptic_camera(192, 12, (2, 2), 100, p) for p in (0.0, 90.0)]
    assert 1 << 22 < 164 * 162 * 160 <= 1 << 23
    plan = ltm.Plan(g, cams)
    assert all(plan.adjoint_kind(k) != RAYS for k in range(2))
    y = torch.from_numpy(W.uniform_random(plan.n_meas, 81)).cuda()
    want = plan.backproject(y)
    got = torch.full_like(want, float("nan"))
    plan.backproject_noalloc(y, got)
    assert float((got.double() - want.double()).norm() / want.double().norm()) < 1e-6
    other = plan.backproject(torch.cat([torch.zeros(192 * 192, device="cuda"), y[192 * 192:]]))
    assert float((other.double() - want.double()).norm() / want.double().norm()) > 0.1   # both cameras count
