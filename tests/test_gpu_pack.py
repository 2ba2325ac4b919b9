"""Packing on the GPU against the host packer: pool, nodes, leaf records (value ranges among them),
patch headers, face records and ropes agree byte for byte in every brick layout, for nested, non-nested
and several-root hierarchies, r = 2 and 4, patches of one cell, odd sizes, and cells that are NaN
or infinite.  Both form the ghost layers in FP64 by the same operations, so no tolerance applies."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


def _odd():
    h = workloads.random_tiny(4, refine=4)
    h.patches[-1].cells[...] = -0.0
    h.patches[0].cells.reshape(-1)[::17] = np.nan
    h.patches[0].cells.reshape(-1)[5] = np.inf
    h.patches[1].cells.reshape(-1)[-1] = -np.inf
    return h


def _one_cell():
    h = workloads.single_level((1, 1, 1))
    return h


HIERARCHIES = {
    "single": lambda: workloads.single_level((13, 6, 9)),
    "one cell": _one_cell,
    "tiny": lambda: workloads.tiny_samr(2),
    "blocks": lambda: workloads.lod_blocks(2),
    "random": lambda: workloads.random_tiny(6, refine=2),
    "random, r = 4, NaN and infinities": _odd,
    "several roots": lambda: workloads.random_tiny(11, multi_root=True, max_patches=9),
    "deep": lambda: workloads.deep_range(0, root=16, nlevels=9, block=8, radius_cells=12.0),
    "cosmology-like": lambda: workloads.cosmology_like(1, root=32, nlevels=4, target_patches=40),
}


@pytest.mark.parametrize("layout", [0, 1, 2])
@pytest.mark.parametrize("name", sorted(HIERARCHIES))
def test_device_pack_matches_host_pack(gpu, name, layout):
    h = HIERARCHIES[name]()
    tree = gpu.build_tree(h)
    host = gpu.pack(tree, h, host=True, brick_layout=layout)
    dev = gpu.pack(tree, h, brick_layout=layout)
    n = host.pool.nbytes - 256           # the pad after the last brick is not part of the data
    got = dev.pool.cpu().numpy()
    assert np.array_equal(got[:n], host.pool[:n])
    assert np.array_equal(dev.meta.cpu().numpy(), host.meta)
    a, b = dev.scene, host.scene
    assert (a.v_min, a.v_max) == (b.v_min, b.v_max)
    assert (a.nnodes, a.nleaves, a.npatches, a.nlod, a.depth) == (b.nnodes, b.nleaves, b.npatches, b.nlod, b.depth)
