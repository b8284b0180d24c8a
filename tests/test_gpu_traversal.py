"""The traversal at the sizes where its hand-out of rays changes: a launch
with no more rays than lanes deals them over its waves and shares them between
lanes, a larger one takes runs from the work counters.  Every hit and distance
equals the oracle's, bit for bit (exact: no tolerance)."""

import numpy as np
import pytest

from paper_2210_06158_amd import synth
from test_gpu_parity import ladder_scene

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def scenes(orc):
    """A soup, a single triangle and the 62-level ladder (whose stacks overflow)."""
    from paper_2210_06158_amd import dof
    out = {}
    for name, sc in (("soup", synth.Scene(*synth.random_triangles(400, seed=11), leaf_split=2)),
                     ("one", synth.Scene(*synth.random_triangles(1, seed=12))), ("ladder", ladder_scene())):
        osc = orc.OracleScene(sc)
        osc.build_bvh()
        gs = dof.Scene(sc)
        gs.build_bvh()
        out[name] = (osc, gs)
    return out


# 1 ray; one wave's lanes and its neighbours; a few rays per wave; the default
# grid's lanes at six waves per SIMD (393216) and one more
@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 1000, 4097, 393215, 393216, 393217])
@pytest.mark.parametrize("name", ["soup", "one", "ladder"])
def test_rays_at_the_edges_of_the_hand_out(scenes, orc, name, n):
    import torch
    osc, gs = scenes[name]
    rng = synth.SplitMix64(17 * n)
    if name == "ladder":
        o = np.stack([rng.uniform(n, -2e6, 2e6), rng.uniform(n, -2e6, 2e6), np.full(n, -3e7)], 1)
        d = np.stack([rng.uniform(n, -0.1, 0.1), rng.uniform(n, -0.1, 0.05), np.ones(n)], 1)
    else:
        o = rng.uniform(3 * n, -6, 6).reshape(n, 3)
        d = rng.uniform(3 * n, -3, 3).reshape(n, 3) - o
    o, d = o.astype(np.float32), d.astype(np.float32)
    print(f"{name}: {n} rays", flush=True)
    hit, t = gs.trace_rays(torch.from_numpy(o).cuda(), torch.from_numpy(d).cuda())
    want, tw = orc.closest_hit(osc, o, d, use_bvh=False)
    assert np.array_equal(hit.cpu().numpy(), want)
    assert np.array_equal(t.cpu().numpy().view(np.uint32), tw.view(np.uint32))


# one block, fewer blocks than work counters, as many, and more that they do
# not divide; grab 100 leaves a remainder in every run's start
@pytest.mark.parametrize("blocks", [1, 2, 7, 8, 9, 17])
@pytest.mark.parametrize("grab", [0, 16, 100])
def test_every_run_is_handed_out(orc, blocks, grab):
    """131072 rays on a few blocks: every ray's hit and distance (exact)."""
    import dataclasses
    import torch
    from paper_2210_06158_amd import dof
    scene, cam, lens, params = synth.scene_small()
    params = dataclasses.replace(params, mask_mode=synth.MASK_ALL, m=8)
    osc = orc.OracleScene(scene)
    osc.build_bvh()
    gs = dof.Scene(scene)
    gs.build_bvh()
    gb = orc.gbuffer(osc, cam, lens)
    want = orc.render_frame(osc, cam, lens, params, gb)
    print(f"{blocks} blocks, runs of {grab}", flush=True)
    fr = dof.Frame(cam.width, cam.height, params, ray_records=True, trace_blocks=blocks,
                   knobs={"trace_grab": grab} if grab else None)
    g = tuple(torch.from_numpy(x).cuda() for x in (gb.colour, gb.depth, gb.normal))
    fr.render(gs, cam, lens, g, None, dof.history_alloc(cam.width, cam.height))
    torch.cuda.synchronize()
    d = fr.debug()
    assert d["n_rays"] == want["n_rays"] > 128 * blocks
    assert np.array_equal(d["ray_hit"], want["ray_hit"])
    assert np.array_equal(d["ray_t"].view(np.uint32), want["ray_t"].view(np.uint32))


@pytest.mark.parametrize("batch", [False, True])
@pytest.mark.parametrize("leaf_batch", [0, 1])
def test_counters_of_a_scene_of_one_leaf(batch, leaf_batch):
    """No node to visit and one triangle test a ray (exact)."""
    import dataclasses
    import torch
    from paper_2210_06158_amd import dof
    scene, cam, lens, params = synth.scene_small()
    scene = dataclasses.replace(scene, verts=scene.verts[:1], albedo=scene.albedo[:1], leaf_split=0)
    cam = dataclasses.replace(cam, width=66, height=50)
    params = dataclasses.replace(params, mask_mode=synth.MASK_ALL, m=5)
    gs = dof.Scene(scene)
    gs.build_bvh()
    g = gs.render_gbuffer(cam, lens)
    fr = dof.Frame(66, 50, params, knobs={"trace_leaf_batch": leaf_batch} if leaf_batch else None)
    hist = dof.history_alloc(66, 50)
    print(f"batch {batch} leaf batch {leaf_batch}", flush=True)
    if batch:
        b = dof.Batch(1, params, knobs={"trace_leaf_batch": leaf_batch} if leaf_batch else None)
        b.set([fr.item(gs, cam, lens, g, None, hist)])
        b.run()
        _, rays, visits, tests = b.totals()
    else:
        fr.render(gs, cam, lens, g, None, hist)
        torch.cuda.synchronize()
        w = fr.stats.cpu().numpy().view(np.uint32)
        rays, (visits, tests) = int(w[1]), (int(x) for x in w[2:6].view(np.uint64))
    assert (rays, visits, tests) == (33 * 25 * 5, 0, 33 * 25 * 5)


@pytest.mark.parametrize("w,h", [(34, 18), (512, 512)])
@pytest.mark.parametrize("formats", [("f32", "f16"), ("f16", "f32"), ("f32", "f32")])
def test_depth_beside_images_in_one_memory(w, h, formats):
    """A program that wants the depths alone may pass one buffer for both
    images; the depths are those of separate buffers (exact)."""
    import dataclasses
    import torch
    from paper_2210_06158_amd import dof
    scene, cam, lens, _ = synth.scene_small()
    cam = dataclasses.replace(cam, width=w, height=h)
    gs = dof.Scene(scene)
    gs.build_bvh()
    want = gs.render_gbuffer(cam, lens)[1]
    whole = torch.zeros(w * h * 4, dtype=torch.float32, device="cuda")
    img = {"f32": whole.view(h, w, 4), "f16": whole.view(torch.float16)[:w * h * 4].view(h, w, 4)}
    depth = torch.zeros((h, w), device="cuda")
    print(f"{w}x{h} {formats}", flush=True)
    for _ in range(2):
        gs.render_gbuffer_into(cam, lens, img[formats[0]], depth, img[formats[1]])
    torch.cuda.synchronize()
    assert torch.isfinite(want).any()
    assert torch.equal(depth.view(torch.int32), want.view(torch.int32))
