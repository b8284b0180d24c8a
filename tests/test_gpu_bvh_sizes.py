"""The tree at the leaf counts where its build changes: one block of leaves
and the next, the one-workgroup sort's last, the block count up to which one
workgroup merges all exits, the counts at which the sort's tiles grow; and
scenes whose keys are all equal (ties in reference order).  Keys, references, children, parents
and child boxes equal the oracle's bit for bit (exact: no tolerance)."""

import numpy as np
import pytest

from paper_2210_06158_amd import synth

pytestmark = pytest.mark.gpu
LEAF = 0x80000000


def soup(n, kind):
    if kind == "equal":      # one centre: one key
        v, a = synth.random_triangles(1, seed=5)
        return synth.Scene(np.repeat(v, n, 0), np.repeat(a, n, 0), leaf_split=0)
    v, a = synth.random_triangles(n, seed=n, spread=40.0, size=0.5)
    if kind == "pairs":      # every key at least twice
        v[1::2] = v[0:-1:2][:v[1::2].shape[0]]
    return synth.Scene(v, a, leaf_split=0)


@pytest.mark.parametrize("n,kind", [(2, "soup"), (63, "soup"), (1023, "soup"), (1024, "soup"), (1025, "soup"),
                                    (2048, "pairs"), (4096, "soup"), (4097, "soup"), (4097, "equal"), (3000, "equal"),
                                    (65536, "soup"), (65537, "soup"), (66000, "pairs"), (524288, "soup"),
                                    (524289, "soup"), (600000, "equal")])
def test_tree_at_the_edges_of_the_build(orc, n, kind):
    import torch
    from paper_2210_06158_amd import dof
    sc = soup(n, kind)
    osc = orc.OracleScene(sc)
    ob = osc.build_bvh()
    gs = dof.Scene(sc)
    print(f"{kind}: {n} leaves", flush=True)
    for _ in range(2):       # again over its own state
        gs.build_bvh()
    torch.cuda.synchronize()
    view = {k: (v if k == "nleaf" else v.cpu().numpy()) for k, v in gs.bvh_view().items()}
    assert view["nleaf"] == n
    assert np.array_equal(view["keys"].view(np.uint64), ob["keys"])
    assert np.array_equal(view["ids"].view(np.uint32), ob["refs"])
    nodes = view["nodes"].reshape(n - 1, 16)
    nu = nodes.view(np.uint32)
    left, right = ob["left"][:n - 1], ob["right"][:n - 1]
    assert np.array_equal(nu[:, 12], left) and np.array_equal(nu[:, 13], right)
    parent = np.full(2 * n - 1, 0xFFFFFFFF, np.uint32)
    for ch in (left, right):
        c = ch.astype(np.int64)
        parent[np.where(c & LEAF, (n - 1) + (c & 0x7FFFFFFF), c)] = np.arange(n - 1)
    assert np.array_equal(view["parent"].view(np.uint32), parent)
    for ch, cols in ((left, (0, 2, 8, 1, 3, 9)), (right, (4, 6, 10, 5, 7, 11))):
        c = ch.astype(np.int64)
        leaf = (c & LEAF) != 0
        want = np.where(leaf[:, None], ob["leaf_bounds"][np.where(leaf, c & 0x7FFFFFFF, 0)], ob["bounds"][np.where(leaf, 0, c)])
        assert np.array_equal(nodes[:, cols].view(np.uint32), want.astype(np.float32).view(np.uint32))
    words = view["nodes16"].view(np.uint32).reshape(n - 1, 8)
    assert np.array_equal(words[:, 6], left) and np.array_equal(words[:, 7], right)
    tris = view["tris"].reshape(n, 12)
    assert np.array_equal(tris[:, 3].view(np.uint32), ob["ids"])
    assert np.array_equal(tris[:, [0, 1, 2, 4, 5, 6, 8, 9, 10]], sc.verts[ob["ids"]])


# the sort's tiles are of 2048 keys up to 131072, of 4096 up to 1048576, of 8192
# beyond: full tiles, and a last one of a single key
@pytest.mark.parametrize("n,kind", [(131072, "soup"), (131073, "soup"), (1048576, "soup"), (1048577, "soup"),
                                    (1048577, "equal")])
def test_tree_where_the_sorts_tiles_grow(orc, n, kind):
    test_tree_at_the_edges_of_the_build(orc, n, kind)
