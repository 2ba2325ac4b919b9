"""Scenes whose pool is below 4 GB take kernels with 32-bit brick offsets, larger ones 64-bit offsets:
the same cells by the same operations, so images, segment traces and the adjoint's inputs agree bit
for bit.  A small scene stands for a large one by its pool_bytes, which chooses the kernels only.
Checkpointed and nearest-cell forwards resolve the queued taps one per lane, plain ones one sample per
lane, in the same order per sample: checkpointed images equal plain ones bit for bit."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

MODES = {
    "unlit": dict(),
    "lit": dict(lighting=1),
    "nearest": dict(interp=1),
    "nearest lit": dict(interp=1, lighting=1),
    "point light": dict(lighting=2, light=(0.5, 0.6, 0.4)),
    "batch": dict(persistent=1, tile_w=8, tile_h=8, blocks_per_cu=2, waves_per_simd=2),
    "batch lit": dict(persistent=1, tile_w=8, tile_h=8, blocks_per_cu=2, waves_per_simd=3, lighting=1),
    "learned": dict(tau_e=5e-4, tau_s=0.0),
}


def _scene(amr, name):
    import torch
    if name == "small":
        h, lut, _, prm = workloads.small_nested(0)
    else:                                    # patches of a few cells: most samples have taps outside
        h = workloads.random_tiny(4, refine=4)
        lut = workloads.lut_bumps(np.random.default_rng(4), sigma_scale=6.0)
        prm = workloads.default_params(v_hi=float(max(p.cells.max() for p in h.patches)))
    tree = amr.build_tree(h)
    return amr.pack(tree, h), torch.from_numpy(np.asarray(lut, np.float32)).cuda(), dict(prm, k_a=0.3, k_d=0.7)


CAMS = [(1, 1), (33, 17), (67, 41)]


@pytest.mark.parametrize("data", ["small", "tiny patches"])
@pytest.mark.parametrize("mode", sorted(MODES))
def test_large_pool_kernels_agree(gpu, mode, data):
    import torch
    from paper_1212_3333_amd import learned
    amr = gpu
    scene, lut, prm = _scene(amr, data)
    prm.update(MODES[mode])
    cams = [workloads.perspective_orbit(w, h, 0.4 + w, 0.3, radius=1.7) for w, h in CAMS]
    kw = {}
    if mode.startswith("batch"):
        kw = dict(d_cams=amr.camera_table(cams), d_queue=amr.queue_buffer(len(cams)))
    elif mode == "learned":
        kw = dict(d_mlp=amr.mlp_pack(learned.init_weights(1, "cuda")))
    views = [cams] if kw.get("d_cams") is not None else cams
    small = [amr.render(scene, c, lut, prm, **kw)["rgba"].clone() for c in views]
    assert 0 < scene.scene.pool_bytes < 1 << 32
    scene.scene.pool_bytes = 1 << 32
    large = [amr.render(scene, c, lut, prm, **kw)["rgba"].clone() for c in views]
    torch.cuda.synchronize()
    for a, b in zip(small, large):
        assert float(a.abs().max()) > 0 or a.numel() <= 4
        assert torch.equal(a, b)


@pytest.mark.parametrize("large", [False, True])
@pytest.mark.parametrize("data", ["small", "tiny patches"])
@pytest.mark.parametrize("tape_cap", [0, 7, 256])
def test_checkpointed_image_equals_plain(gpu, tape_cap, data, large):
    import torch
    amr = gpu
    scene, lut, prm = _scene(amr, data)
    prm.update(lighting=1)
    if large:
        scene.scene.pool_bytes = 1 << 32
    for w, h in CAMS:
        cam = workloads.perspective_orbit(w, h, 0.7 + w, -0.2, radius=1.7)
        plain = amr.render(scene, cam, lut, prm)["rgba"].clone()
        ck, _ = amr.render_checkpointed(scene, cam, lut, prm, tape_cap=tape_cap)
        torch.cuda.synchronize()
        assert torch.equal(ck["rgba"], plain)
