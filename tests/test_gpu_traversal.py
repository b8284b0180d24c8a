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
# grid's lanes at six blocks of 128 per SIMD (393216) and one more
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
