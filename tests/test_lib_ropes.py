"""Ropes against restarts, on the host: the walk the kernels take from one leaf to the next (from the
rope of the exit face, or the root where two faces share the exit) meets the leaves and exits of a
kD-restart from the root, bit for bit, for rays in general position, along the axes, through
edges and corners of the cell lattice, and from inside the box."""
import numpy as np
import pytest

import paper_1212_3333_amd as amr
import workloads


def _ropes(sc):
    base = sc.meta.ctypes.data
    n = sc.scene.nleaves + sc.scene.nlod
    off = (sc.scene.face_taps - base + n * 6 * 64 + 255) // 256 * 256
    assert off + 24 * sc.scene.nleaves <= sc.scene.meta_bytes
    return sc.meta[off:off + 24 * sc.scene.nleaves].view(np.int32).reshape(-1, 6)


def _restart(nodes, o, d, inv, tmin, tmax):
    ni = 0
    while True:
        s, child, axis = nodes["split"][ni], int(nodes["child"][ni]), int(nodes["meta"][ni]) & 3
        if axis == 3:
            return child, tmax
        if d[axis] == 0.0:
            ni = child if o[axis] < s else child + 1
            continue
        near = child if (o[axis] < s or (o[axis] == s and d[axis] < 0.0)) else child + 1
        ts = (s - o[axis]) * inv[axis]
        if ts <= 0.0 or ts >= tmax:
            ni = near
        elif ts <= tmin:
            ni = 2 * child + 1 - near
        else:
            ni, tmax = near, ts


def _rope_step(nodes, leaves, ropes, o, d, inv, tmin, tmax, start):
    ni, visits = start, 0
    while True:
        visits += 1
        s, child, axis = nodes["split"][ni], int(nodes["child"][ni]), int(nodes["meta"][ni]) & 3
        if axis == 3:
            break
        low = o[axis] < s or (o[axis] == s and d[axis] < 0.0)
        ts = (s - o[axis]) * inv[axis]
        far = d[axis] != 0.0 and ts > 0.0 and ts <= tmin
        ni = child if low != far else child + 1
    face, tie = -1, False
    for a in range(3):
        up = d[a] > 0.0
        ts = ((leaves["hi"] if up else leaves["lo"])[child][a] - o[a]) * inv[a]
        ahead = d[a] != 0.0 and ts > tmin
        if ahead and ts == tmax:
            tie = True
        if ahead and ts < tmax:
            tmax, face, tie = ts, 2 * a + int(up), False
    return child, tmax, int(ropes[child, face]) if face >= 0 and not tie else 0, visits


def _clip(lo, hi, o, d, inv):
    t0, t1 = 0.0, np.inf
    for a in range(3):
        if d[a] == 0.0:
            if not lo[a] <= o[a] < hi[a]:
                return None
            continue
        ta, tb = (lo[a] - o[a]) * inv[a], (hi[a] - o[a]) * inv[a]
        t0, t1 = max(t0, min(ta, tb)), min(t1, max(ta, tb))
    return (t0, t1) if t1 > t0 else None


def _rays(rng, lo, hi, lattice, n):
    """Origins and directions: general, axis-parallel, through lattice points, diagonal, inside."""
    ext = hi - lo
    for i in range(n):
        kind = i % 5
        target = lo + rng.random(3) * ext
        o = lo + 0.5 * ext + rng.normal(size=3) * 2 * ext
        if kind == 1:
            d = np.zeros(3)
            d[rng.integers(3)] = rng.choice([-1.0, 1.0])
            o = target - 2.0 * np.max(ext) * d
            if i % 2:
                o = np.round((o - lo) / lattice) * lattice + lo
            yield o, d
            continue
        if kind == 2:
            target = lo + np.round((target - lo) / lattice) * lattice
        if kind == 3:
            d = rng.choice([-1.0, 0.0, 1.0], 3)
            if not np.any(d):
                d[0] = 1.0
            o = lo + np.round((target - lo) / lattice) * lattice - d * np.max(ext)
            yield o, d / np.sqrt(np.sum(d * d))
            continue
        if kind == 4:
            o = lo + rng.random(3) * ext
        d = target - o
        yield o, d / np.sqrt(np.sum(d * d))


HIERARCHIES = {
    "single": lambda: workloads.single_level(),
    "tiny": lambda: workloads.tiny_samr(3),
    "blocks": lambda: workloads.lod_blocks(1),
    "random": lambda: workloads.random_tiny(5, refine=2),
    "random, r = 4": lambda: workloads.random_tiny(8, refine=4),
    "several roots": lambda: workloads.random_tiny(11, multi_root=True, max_patches=9),
    "deep": lambda: workloads.deep_range(0, root=16, nlevels=12, block=8, radius_cells=12.0),
}


@pytest.mark.parametrize("name", sorted(HIERARCHIES))
def test_rope_walk_matches_restart(name):
    h = HIERARCHIES[name]()
    tree = amr.build_tree(h)
    sc = amr.pack(tree, h, host=True)
    nodes, leaves, ropes = sc.node_records(), sc.leaf_records(), _ropes(sc)
    assert ropes.min() >= 0 and ropes.max() < sc.scene.nnodes
    lo, hi = np.array(sc.scene.box_lo[:]), np.array(sc.scene.box_hi[:])
    rng = np.random.default_rng(17)
    total = visits = ties = rays = 0
    for o, d in _rays(rng, lo, hi, np.array(sc.scene.hfine[:]) * 4, 250):
        with np.errstate(divide="ignore"):
            inv = np.where(d != 0.0, 1.0 / d, 0.0)
        c = _clip(lo, hi, o, d, inv)
        if c is None:
            continue
        rays += 1
        t, t1 = c
        start = 0
        while t < t1:
            want, tb = _restart(nodes, o, d, inv, t, t1)
            got, tg, start, v = _rope_step(nodes, leaves, ropes, o, d, inv, t, t1, start)
            assert (got, tg) == (want, tb), (name, o, d, t)
            assert tb > t
            total, visits, ties = total + 1, visits + v, ties + int(start == 0 and tb < t1)
            t = tb
    assert rays > 100 and total >= rays
    print(name, rays, total, visits / total, ties)
