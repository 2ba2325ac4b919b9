"""Unlit images of many pixels are marched with one lane per ray, smaller ones and every render that records
more than checkpoints with four: the images agree bit for bit, in every layout, for both samplings, with a level of detail, with a tile
schedule, in groups and in persistent batches, at sizes on either side of the rule."""
import pytest

import workloads

pytestmark = pytest.mark.gpu

W, H = 1573, 1000          # 1573000 pixels: one lane from 1572864 on


@pytest.fixture(scope="module")
def scene_of(gpu):
    h = workloads.cosmology_like(3, root=32, nlevels=4, target_patches=40)
    tree = gpu.build_tree(h)
    scenes = {}

    def make(layout):
        if layout not in scenes:
            scenes[layout] = gpu.pack(tree, h, brick_layout=layout)
        return scenes[layout]
    return make


def _setup():
    import torch
    lut = torch.from_numpy(workloads.lut_cosmology(0)).cuda()
    return lut, dict(workloads.default_params(), v_lo=0.0, v_hi=3.0, lighting=0, t_min=1e-2)


def _cam(w, h, az=0.7):
    return workloads.perspective_orbit(w, h, az, 0.4, radius=1.5)


@pytest.mark.parametrize("layout", [0, 1, 2])
@pytest.mark.parametrize("kw", [{}, dict(interp=1), dict(lod=2.0), dict(t_min=0.0)], ids=str)
@pytest.mark.parametrize("w,h", [(W, H), (1572, 1000), (1, 1600000 // 50), (3001, 999)])
def test_frame(gpu, scene_of, layout, kw, w, h):
    import torch
    lut, prm = _setup()
    scene, cam, p = scene_of(layout), _cam(w, h), dict(prm, **kw)
    ref = gpu.render(scene, cam, lut, p, stats=True)
    got = gpu.render(scene, cam, lut, p)["rgba"]
    assert torch.equal(got, ref["rgba"]) and float(ref["rgba"].max()) > 0.0
    sched = gpu.Schedule(cam, "cuda")
    for _ in range(3):
        assert torch.equal(gpu.render(scene, cam, lut, p, **sched.params())["rgba"], ref["rgba"])


def test_group(gpu, scene_of):
    import torch
    lut, prm = _setup()
    scene = scene_of(2)
    cams = [_cam(W, H, 0.3 * i) for i in range(3)] + [_cam(2000, 1400)]
    ref = torch.cat([gpu.render(scene, c, lut, prm, stats=True)["rgba"].view(-1, 4) for c in cams])
    assert torch.equal(gpu.render(scene, cams, lut, prm)["rgba"], ref)


@pytest.mark.parametrize("kw", [{}, dict(xcd_tiles=1), dict(tile_w=16, tile_h=4, queue_order=1), dict(tile_w=64, tile_h=1, xcd_tiles=1)],
                         ids=str)
@pytest.mark.parametrize("sizes", [[(W, H), (1600, 1001)], [(640, 480), (33, 500), (128, 128)], [(3000, 1200), (64, 64)]], ids=str)
def test_persistent(gpu, scene_of, sizes, kw):
    import torch
    lut, prm = _setup()
    scene = scene_of(2)
    cams = [_cam(w, h, 0.2 * i) for i, (w, h) in enumerate(sizes)]
    ref = torch.cat([gpu.render(scene, c, lut, prm, stats=True)["rgba"].view(-1, 4) for c in cams])
    q, dc = gpu.queue_buffer(len(cams)), gpu.camera_table(cams)
    for lit in (0, 1):
        p = dict(prm, persistent=1, lighting=lit, **kw)
        if lit:
            ref = torch.cat([gpu.render(scene, c, lut, dict(prm, lighting=1))["rgba"].view(-1, 4) for c in cams])
        for stamped in (False, True):
            stamps = torch.zeros(len(cams) + 1, dtype=torch.int64, device="cuda")
            got = gpu.render(scene, cams, lut, p, d_queue=q, d_cams=dc, **(dict(d_stamps=stamps) if stamped else {}))["rgba"]
            assert torch.equal(got, ref)
            if stamped:
                s = stamps.cpu()
                assert int(s[-1]) > 0 and bool((s[:-1] >= s[-1]).all())


@pytest.mark.parametrize("cap", [2, 4])
@pytest.mark.parametrize("sizes", [[(2048, 2048)], [(2047, 2049)], [(2050, 2047), (2051, 2061)]], ids=str)
def test_checkpoints(gpu, scene_of, sizes, cap):
    """The images, checkpoints and headers of a checkpointed forward (one lane from 2^22 pixels on) are
    those of the recording render, whose quads write them."""
    import torch
    lut, prm = _setup()
    scene, cams = scene_of(2), [_cam(w, h, 0.3 * i) for i, (w, h) in enumerate(sizes)]
    n = sum(w * h for w, h in sizes)
    got = []
    for kw in ({}, dict(stats=True)):
        ck = gpu.Checkpoints(n, "cuda", 2, cap)
        ck.buf.zero_()
        got.append((gpu.render(scene, cams, lut, prm, **ck.params(), **kw)["rgba"].flatten(), ck.buf))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
    assert int(got[0][1].view(n, -1)[:, 20:24].view(torch.int32).max()) == cap      # rays ran out of records
