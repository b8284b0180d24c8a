"""The ray mask's edge filter where its sums leave the binary32 numbers: depths
so small that twice or four times the disparity overflows, beside ordinary
ones, zeros and the sky, and normals of any length.  Ray counts equal the
oracle's (exact)."""

import dataclasses

import numpy as np
import pytest

from paper_2210_06158_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("w,h", [(2, 2), (32, 32), (130, 66)])
@pytest.mark.parametrize("kind", ["disparity", "normal", "columns"])
def test_counts_where_sums_overflow(orc, kind, w, h):
    import torch
    from paper_2210_06158_amd import dof
    scene, cam, lens, params = synth.scene_small()
    cam = dataclasses.replace(cam, width=w, height=h)
    osc = orc.OracleScene(scene)
    osc.build_bvh()
    gs = dof.Scene(scene)
    gs.build_bvh()
    gb = orc.gbuffer(osc, cam, lens)
    rng = synth.SplitMix64(w * 3 + h)
    colour, depth, normal = gb.colour.copy(), gb.depth.copy(), gb.normal.copy()
    big = np.asarray([1.0, 1e30, 3e37, 9e37, 1.6e38, 2.5e38, 3.3e38])
    # 12 x 12 blocks of one value each, so that whole footprints share it, on the left half
    pick = (rng.uniform(((h + 11) // 12) * ((w + 11) // 12)) * big.size).astype(int).reshape((h + 11) // 12, -1)
    blk = np.kron(pick, np.ones((12, 12), int))[:h, :w]
    left = (np.arange(w) < (w + 1) // 2)[None, :] & np.ones((h, 1), bool)
    if kind == "normal":
        normal[left] = (normal * np.where(rng.uniform(h * w).reshape(h, w) < 0.5, -1, 1)[..., None] * big[blk][..., None])[left]
    else:
        depth[left] = (lens.focus / big[blk])[left]
        if kind == "columns":     # both signs of difference within a footprint, and disparities of infinity
            depth[:, ::5] = lens.focus / 2.9e38
            depth[:, 3::11] = 0.0
    gb = orc.GBuffer(colour, depth.astype(np.float32), normal.astype(np.float32))
    want = orc.render_frame(osc, cam, lens, params, gb)
    print(f"{kind} {w}x{h}", flush=True)
    fr = dof.Frame(w, h, params)
    g = tuple(torch.from_numpy(x).cuda() for x in (gb.colour, gb.depth, gb.normal))
    fr.render(gs, cam, lens, g, None, dof.history_alloc(w, h))
    torch.cuda.synchronize()
    assert np.array_equal(fr.mask.cpu().numpy(), want["mask"])
