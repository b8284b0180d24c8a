"""The prefilter at the edges of its tiles and of the texels that it stages:
taps up to 5 texels away are staged (a radius of 40), farther ones are read in
global memory; with the timing of stages on, the dilation is a launch of its
own.  The same operations in the same order either way: equal to the oracle
within 1e-6 of the value (nine divisions and sums of binary32: 2^-21)."""

import dataclasses

import numpy as np
import pytest

from paper_2210_06158_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("w,h", [(2, 2), (30, 34), (64, 32), (130, 66)])
@pytest.mark.parametrize("r_max", [8.0, 39.0, 48.0, 200.0])
@pytest.mark.parametrize("timing", [False, True])
def test_prefilter(orc, w, h, r_max, timing):
    import torch
    from paper_2210_06158_amd import dof
    scene, cam, lens, params = synth.scene_small()
    cam = dataclasses.replace(cam, width=w, height=h)
    lens = dataclasses.replace(lens, fnum=2e-4)    # radii that reach r_max
    p = dataclasses.replace(params, r_max=r_max)
    osc = orc.OracleScene(scene)
    osc.build_bvh()
    gs = dof.Scene(scene)
    gs.build_bvh()
    gb = orc.gbuffer(osc, cam, lens)
    want = orc.render_frame(osc, cam, lens, p, gb)
    fr = dof.Frame(w, h, p, ray_records=True, timing=timing)
    g = tuple(torch.from_numpy(x).cuda() for x in (gb.colour, gb.depth, gb.normal))
    fr.render(gs, cam, lens, g, None, dof.history_alloc(w, h))
    torch.cuda.synchronize()
    d = fr.debug()
    assert np.array_equal(d["tile_dil"], want["tile_dil"])
    np.testing.assert_allclose(d["pre"], want["pre"], rtol=1e-6, atol=1e-6)
