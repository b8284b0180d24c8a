"""The gather's depth term, whose division by the depth range is a product with
its reciprocal and two fused steps, or a division where the reciprocal could
leave the normal numbers: ranges either side of both limits and ordinary ones,
over views with sky (infinite depths and differences that are no number).
Held to the oracle within the stage's 1e-5."""

import dataclasses

import numpy as np
import pytest

from paper_2210_06158_amd import synth
from test_gpu_parity import STAGE_TOL, run_pair

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env(orc):
    import torch
    from paper_2210_06158_amd import dof
    scene, cam, lens, params = synth.scene_small()
    osc = orc.OracleScene(scene)
    osc.build_bvh()
    gs = dof.Scene(scene)
    gs.build_bvh()
    return dict(torch=torch, dof=dof, osc=osc, gs=gs), cam, lens, params


@pytest.mark.parametrize("depth_range", [1e-38, 9e-31, 1.1e-30, 1e-3, 0.1, 7.0, 9e29, 1.1e30, 3e38])
@pytest.mark.parametrize("window", [0, 40])
@pytest.mark.parametrize("w,h", [(66, 50), (256, 256)])
def test_depth_ranges(env, orc, depth_range, window, w, h):
    e, cam, lens, params = env
    cam = dataclasses.replace(cam, width=w, height=h)
    p = dataclasses.replace(params, depth_range=depth_range)
    gb = orc.gbuffer(e["osc"], cam, lens)
    o, d = run_pair(e, orc, cam, lens, p, gb, knobs={"gather_window": window} if window else None)
    np.testing.assert_allclose(d["gather"], o["gather"], rtol=STAGE_TOL, atol=STAGE_TOL)
