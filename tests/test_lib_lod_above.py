"""Leaf flags name the finest level-of-detail node above the leaf (1: none): compared with a walk over
all nodes of the packed tree.  It decides where a level-of-detail march may go on by ropes."""
import numpy as np
import pytest

import paper_1212_3333_amd as amr
import workloads

HIERARCHIES = {
    "single": lambda: workloads.single_level((13, 6, 9)),
    "blocks": lambda: workloads.lod_blocks(2),
    "random": lambda: workloads.random_tiny(6, refine=2),
    "several roots, r = 4": lambda: workloads.random_tiny(4, refine=4, multi_root=True),
    "cosmology-like": lambda: workloads.cosmology_like(1, root=32, nlevels=4, target_patches=40),
}


@pytest.mark.parametrize("name", sorted(HIERARCHIES))
def test_finest_lod_node_above_each_leaf(name):
    h = HIERARCHIES[name]()
    scene = amr.pack(amr.build_tree(h), h, host=True)
    nodes, nleaves = scene.node_records(), scene.scene.nleaves
    # the level-of-detail records follow the leaves'
    leaves = scene._records(scene.scene.leaves, scene.leaf_records().dtype, nleaves + scene.scene.nlod)
    step = [float(np.min(h.h0)) / h.refine ** p.level for p in h.patches]
    todo, seen = [(0, [])], 0
    while todo:
        ni, above = todo.pop()
        n = nodes[ni]
        if n["meta"] & 3 == 3:
            up = int(leaves[n["child"]]["level_flags"]) >> 14
            assert up >= 1
            if not above:
                assert up == 1
            else:
                assert up - 2 in above
                own = lambda r: step[leaves[nleaves + r]["patch"]]
                assert own(up - 2) == min(own(r) for r in above)
            seen += 1
            continue
        rec = int(n["meta"]) >> 8
        above = above + [rec - 1] if rec else above
        todo += [(int(n["child"]), above), (int(n["child"]) + 1, above)]
    assert seen == nleaves
