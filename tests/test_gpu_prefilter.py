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


def nine_taps(colr, sp):
    """The prefilter of a plane (h, w, 4) with one tap distance, in binary64."""
    h, w = colr.shape[:2]
    c = colr.astype(np.float64)

    def axis(n, k):
        s = np.arange(n, dtype=np.float32) + np.float32(k) * np.float32(sp)
        lo = np.floor(s)
        a = np.clip(lo, 0, n - 1).astype(int)
        return a, np.clip(lo + 1, 0, n - 1).astype(int), (s - lo).astype(np.float64)

    num, den = np.zeros((h, w, 3)), np.zeros((h, w))
    for dy in (-1, 0, 1):
        ya, yb, fy = axis(h, dy)
        for dx in (-1, 0, 1):
            xa, xb, fx = axis(w, dx)
            row = [c[y][:, xa] + (c[y][:, xb] - c[y][:, xa]) * fx[None, :, None] for y in (ya, yb)]
            v = row[0] + (row[1] - row[0]) * fy[:, None, None]
            wt = 1 / (1 + np.abs(v[..., 3] - c[..., 3]))
            num += wt[..., None] * v[..., :3]
            den += wt
    return num / den[..., None]


@pytest.mark.parametrize("r_max,timing", [(3e10, False), (1e30, False), (float("inf"), False), (float("inf"), True)])
@pytest.mark.parametrize("w,h", [(30, 34), (130, 66)])
def test_radius_without_a_limit(w, h, r_max, timing):
    """Radii past the integers, of a frame whose nearest texel's CoC reaches
    them: up to 16 * 2^31 the neighbourhood is the whole frame, beyond, and for
    no limit at all, it is empty, with the dilation in a launch of its own or not."""
    import torch
    from paper_2210_06158_amd import dof
    scene, cam, lens, params = synth.scene_small()
    cam = dataclasses.replace(cam, width=w, height=h)
    p = dataclasses.replace(params, r_max=r_max)
    gs = dof.Scene(scene)
    gs.build_bvh()
    g = gs.render_gbuffer(cam, lens, fmt=dof.RGBA32F)
    g[1].view(-1)[0] = 1e-20
    print(f"{w}x{h} r_max {r_max} timing {timing}", flush=True)
    fr = dof.Frame(w, h, p, timing=timing)
    fr.render(gs, cam, lens, g, None, dof.history_alloc(w, h))
    torch.cuda.synchronize()
    d = fr.debug()
    most = d["tile_max"].max()
    assert most > 1e9
    assert np.all(d["tile_dil"] == (most if r_max < 16 * 2.0 ** 31 else 0))
    sp = np.float32(max(d["tile_dil"][0, 0] * np.float32(0.25), np.float32(1.41421356237)) * np.float32(0.5))
    assert (sp >= 2.0 ** 31) == (r_max < 1e20)
    at = np.abs(d["colr"][..., 3]) < 1e3   # the near texel's own radius leaves the others no weight that counts
    np.testing.assert_allclose(d["pre"][at][:, :3], nine_taps(d["colr"], sp)[at], rtol=1e-6, atol=1e-6)
