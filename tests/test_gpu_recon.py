"""The reconstruction where its work changes: a pixel whose blend weight is 0
is the median and reads no taps, the others are packed into as few waves as
hold them, and a frame whose colours are so large that sums over taps may
overflow reads every tap.  Sizes: one tile of 16 x 16 half-res pixels, its
edges and remainders.

Every value is held to the oracle's within 1e-5 of the largest colour (the
81 weights of a pixel's taps are rounded once each: 81 * 2^-24 = 5e-6), and a
pixel of weight 0 to the median, bit for bit."""

import dataclasses

import numpy as np
import pytest

from paper_2210_06158_amd import synth
from test_gpu_parity import run_pair

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def envs(orc):
    import torch
    from paper_2210_06158_amd import dof
    out = {}
    for scale in (1.0, 4e18):    # 4e18: beyond the bound of a tame frame; its square is finite
        scene, cam, lens, params = synth.scene_small()
        scene = dataclasses.replace(scene, albedo=(scene.albedo * scale).astype(np.float32))
        osc = orc.OracleScene(scene)
        osc.build_bvh()
        gs = dof.Scene(scene)
        gs.build_bvh()
        out[scale] = (dict(torch=torch, dof=dof, osc=osc, gs=gs), cam, lens, params)
    return out


@pytest.mark.parametrize("w,h", [(2, 2), (30, 34), (32, 32), (66, 62), (130, 40)])
@pytest.mark.parametrize("scale", [1.0, 4e18])
@pytest.mark.parametrize("var_w", [0.0, 2.0, 2000.0])
def test_weights_of_zero_and_not(envs, orc, scale, var_w, w, h):
    env, cam, lens, params = envs[scale]
    cam = dataclasses.replace(cam, width=w, height=h)
    p = dataclasses.replace(params, mask_mode=synth.MASK_ALL, var_recon_w=var_w / scale ** 2)
    gb = orc.gbuffer(env["osc"], cam, lens)
    hist, prev = None, None
    for frame in range(3):
        o, d = run_pair(env, orc, cam, lens, p, gb, hist_in=hist, prev_cam=prev, prev_lens=lens if prev else None)
        assert np.array_equal(d["mask"], o["mask"])
        tol = 1e-5 * scale
        np.testing.assert_allclose(d["rtmed"], o["rtmed"], rtol=1e-5, atol=tol)
        np.testing.assert_allclose(d["recon"], o["recon"], rtol=1e-5, atol=tol)
        still = np.clip(d["var_blur"] * np.float32(p.var_recon_w), 0, p.b_max) == 0
        med = d["rtmed"].reshape(d["recon"].shape)
        at = still.reshape(d["recon"].shape[:2]) & (med[..., 3] > 0)
        assert np.array_equal(d["recon"][at][:, :3], med[at][:, :3])
        hist, prev = o["hist_out"], cam


# 756 and 784 tiles of 16 x 16: the last frame whose pixels' taps four waves
# share, and one with a lane per pixel (a batch's items always have that, and
# are held to the frame's bits elsewhere)
@pytest.mark.parametrize("w,h", [(896, 864), (896, 896)])
def test_either_tile(envs, orc, w, h):
    env, cam, lens, params = envs[1.0]
    cam = dataclasses.replace(cam, width=w, height=h)
    gb = orc.gbuffer(env["osc"], cam, lens)
    o, d = run_pair(env, orc, cam, lens, params, gb)
    np.testing.assert_allclose(d["rtmed"], o["rtmed"], rtol=1e-5, atol=1e-5)
    np.testing.assert_allclose(d["recon"], o["recon"], rtol=1e-5, atol=1e-5)


# one tile of either kind, and ragged ones
@pytest.mark.parametrize("w,h", [(32, 32), (38, 34), (896, 896)])
def test_circle_of_confusion_that_is_no_number(envs, w, h):
    """A history whose CoC is infinite gives pixels whose CoC is NaN, here all
    of a tile: no tap counts there, so the pixel is the median with its own
    hit ratio, bit for bit (exact)."""
    import torch
    from paper_2210_06158_amd import dof
    env, cam, lens, params = envs[1.0]
    cam = dataclasses.replace(cam, width=w, height=h)
    p = dataclasses.replace(params, mask_mode=synth.MASK_ALL, var_recon_w=2.0)
    gs = env["gs"]
    print(f"{w}x{h}", flush=True)
    g = gs.render_gbuffer(cam, lens)
    fr = dof.Frame(w, h, p, ray_records=True)
    hist = [dof.history_alloc(w, h), dof.history_alloc(w, h)]
    fr.render(gs, cam, lens, g, None, hist[0])
    n = (w // 2) * (h // 2)
    hist[0][8 * n:12 * n].view(n, 4).copy_(torch.tensor([np.inf, np.inf, 0.0, 1.0]))   # near and far CoC, luma mean and moment
    cam1 = dataclasses.replace(cam, frame=1)
    fr.render(gs, cam1, lens, g, hist[0], hist[1], prev_cam=cam, prev_lens=lens)
    torch.cuda.synchronize()
    d = fr.debug()
    t1, med, rec = d["temporal"][1], d["rtmed"].reshape(d["recon"].shape), d["recon"]
    nan = np.isnan(t1[..., 0])
    assert nan[:16, :16].all() and (d["var_blur"].reshape(nan.shape)[:16, :16] > 0).all()
    assert np.array_equal(rec[nan][:, :3], med[nan][:, :3]) and np.array_equal(rec[nan][:, 3], t1[nan][:, 1])


def _wild(fr):
    """The mark of a frame whose colours may sum to no number (third counter)."""
    import ctypes as C
    import torch
    from paper_2210_06158_amd import dof
    v = dof.DofDebugView()
    dof.check(dof.lib().dof_debug_view_get(C.c_void_p(fr.scratch.data_ptr()), fr.W, fr.H, C.byref(fr.ps), C.byref(v)))
    return int(fr._view(v.counters - fr.scratch.data_ptr(), 12, torch.int32).cpu()[2])


@pytest.mark.parametrize("w,h", [(32, 32), (130, 40), (896, 896)])
@pytest.mark.parametrize("batch", [False, True])
def test_sums_that_overflow(envs, orc, batch, w, h):
    """Colours of 1e37: the median is finite, but the sum over a pixel's taps
    often is not, and 0 times it is no 0, so pixels of weight 0 read their taps
    here too.  Where a sum overflows is the oracle's, but for pixels that a
    colour 2e-5 larger or smaller (twice the taps' rounding) decides otherwise.
    The next frame in the same buffers is an ordinary one."""
    import torch
    from paper_2210_06158_amd import dof
    env, cam, lens, params = envs[1.0]
    base = synth.scene_small()[0]
    cam = dataclasses.replace(cam, width=w, height=h)
    p = dataclasses.replace(params, mask_mode=synth.MASK_ALL, var_recon_w=2.0)
    want = []
    for scale in (1e37, 1e37 * (1 - 2e-5), 1e37 * (1 + 2e-5)):
        sc = dataclasses.replace(base, albedo=(base.albedo * scale).astype(np.float32))
        osc = orc.OracleScene(sc)
        osc.build_bvh()
        gb = orc.gbuffer(osc, cam, lens)
        want.append((sc, gb, orc.render_frame(osc, cam, lens, p, gb)))
    print(f"{w}x{h} batch {batch}", flush=True)
    sc, gb, o = want[0]
    wild = dof.Scene(sc)
    wild.build_bvh()
    fr = dof.Frame(w, h, p, ray_records=True)
    hist = dof.history_alloc(w, h)

    def frame(gs, gb):
        g = tuple(torch.from_numpy(x).cuda() for x in (gb.colour, gb.depth, gb.normal))
        if batch:
            b = dof.Batch(1, p, ray_records=True)
            b.set([fr.item(gs, cam, lens, g, None, hist)])
            b.run()
        else:
            fr.render(gs, cam, lens, g, None, hist)
        torch.cuda.synchronize()
        return fr.debug()

    d = frame(wild, gb)
    assert _wild(fr) != 0
    got, exp = d["recon"], o["recon"].reshape(d["recon"].shape)
    fin = [np.isfinite(x[2]["recon"].reshape(got.shape)) for x in want]
    sure = (fin[1] == fin[2]) & (fin[0] == fin[1])
    assert (sure & ~fin[0])[..., :3].any() and (sure & fin[0])[..., :3].any() and sure.mean() > 0.999
    assert np.array_equal(np.isnan(got)[sure], np.isnan(exp)[sure]) and np.array_equal(np.isfinite(got)[sure], fin[0][sure])
    at = (sure & fin[0])[..., :3]
    med = d["rtmed"].reshape(got.shape)[..., :3]
    assert np.array_equal(got[..., :3][at], med[at])     # weight 0: luma variances of infinity minus infinity count as 0
    np.testing.assert_allclose(got[..., :3][at], exp[..., :3][at], rtol=1e-5, atol=0)
    np.testing.assert_allclose(got[..., 3], exp[..., 3], rtol=1e-5, atol=1e-5)

    gb = orc.gbuffer(env["osc"], cam, lens)
    o = orc.render_frame(env["osc"], cam, lens, p, gb)
    d = frame(env["gs"], gb)
    assert _wild(fr) == 0
    np.testing.assert_allclose(d["recon"], o["recon"], rtol=1e-5, atol=1e-5)
