"""Autotuning an adjoint that runs in bundles: a saved tiling of the same bundles is taken
over as it was saved."""
import numpy as np
import pytest
import torch

from paper_1812_03358_amd import autotune, workloads as W

pytestmark = pytest.mark.gpu


def test_saved_bundled_tiling(tmp_path):
    from paper_1812_03358_amd import ltm
    g = W.grid((20, 24, 18), 6.0)
    cams = [W.plenoptic_camera(192, 16, (2, 2), 37, 20.0)]
    rng = np.random.default_rng(3)
    x = torch.from_numpy(rng.random(20 * 24 * 18).astype(np.float32)).cuda()
    y = torch.from_numpy(rng.random(192 * 192).astype(np.float32)).cuda()
    cache = str(tmp_path / "tilings.tsv")
    plan = ltm.Plan(g, cams)
    assert plan.adjoint_kind() != ltm.ADJOINT_RAYS
    current = plan.get_tiling(ltm.ADJOINT)
    autotune.autotune_plan(plan, x, y, reps=1, cache=cache)
    # the adjoint's line with another slab depth: the same bundles, another tiling
    lines = open(cache).read().splitlines()
    k = next(i for i, line in enumerate(lines) if "|AT|" in line)
    key, _, ms = lines[k].split("\t")
    saved = [current.tile_u, current.tile_v, current.block_u, current.block_v, current.order, current.splits,
             current.brick_floats, 0, 17.0]
    lines[k] = "\t".join([key, " ".join(str(v) for v in saved), ms])
    open(cache, "w").write("\n".join(lines) + "\n")
    plan = ltm.Plan(g, cams)
    want = plan.backproject(y)
    autotune.autotune_plan(plan, x, y, reps=1, cache=cache)
    assert plan.get_tiling(ltm.ADJOINT).chunk_mm == 17.0
    got = plan.backproject(y)
    assert float((got - want).norm() / want.norm()) < 1e-6
