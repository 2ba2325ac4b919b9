"""Packing beside other work on the GPU: a call on one stream does not wait for work on another, and what
it allocates on the GPU is given back."""
import time

import pytest

import workloads

pytestmark = pytest.mark.gpu


def _busy(torch, stream):
    """An event behind some 0.4 s of work on the stream."""
    with torch.cuda.stream(stream):
        torch.cuda._sleep(int(1e9))
        e = torch.cuda.Event()
        e.record()
    return e


@pytest.mark.parametrize("other", ["null", "side"])
def test_pack_waits_for_its_own_stream_only(gpu, other):
    import torch
    amr = gpu
    h = workloads.cosmology_like(1, root=32, nlevels=4, target_patches=40)
    tree = amr.build_tree(h)
    keep = [amr.pack(tree, h)]
    src = torch.ones(1 << 24, dtype=torch.uint8)
    dst = torch.empty_like(src, device="cuda")
    busy = torch.cuda.default_stream() if other == "null" else torch.cuda.Stream()
    # two streams can share a hardware queue, where a copy on one waits for the other's work: take one on
    # which a plain copy does not
    for _ in range(16):
        s = torch.cuda.Stream()
        torch.cuda.synchronize()
        e = _busy(torch, busy)
        with torch.cuda.stream(s):
            dst.copy_(src)
            s.synchronize()
        free = not e.query()
        torch.cuda.synchronize()
        if free:
            break
    assert free, "every stream shares the busy one's queue"
    with torch.cuda.stream(s):
        keep.append(amr.pack(tree, h))          # torch's blocks for this stream
        torch.cuda.synchronize()
        e = _busy(torch, busy)
        t = time.perf_counter()
        keep.append(amr.pack(tree, h))
        t = time.perf_counter() - t
        assert not e.query(), "packing took %.3f s and ended after the other stream's work" % t
    torch.cuda.synchronize()
    assert torch.equal(keep[0].pool[:-256], keep[2].pool[:-256]) and torch.equal(keep[0].meta, keep[2].meta)


def test_pack_gives_its_memory_back(gpu):
    import torch
    amr = gpu
    h = workloads.single_level((256, 256, 192))          # 50 MB of cells
    tree = amr.build_tree(h)
    scene = amr.pack(tree, h)
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    for _ in range(3):
        del scene
        scene = amr.pack(tree, h)
    for _ in range(100):            # the runtime frees a little after the stream has been waited for
        torch.cuda.synchronize()
        held = before - torch.cuda.mem_get_info()[0]
        if held < 16 << 20:
            break
        time.sleep(0.02)
    assert held < 16 << 20


def test_packs_from_several_threads(gpu):
    """Four threads pack their hierarchies at once, each on its own stream, again and again."""
    import threading
    import torch
    amr = gpu
    hs = [workloads.cosmology_like(i, root=32, nlevels=4, target_patches=20 + 10 * i) for i in range(4)]
    trees = [amr.build_tree(h) for h in hs]
    refs = [amr.pack(t, h) for t, h in zip(trees, hs)]
    torch.cuda.synchronize()
    bad = []

    def work(i):
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            for _ in range(6):
                got = amr.pack(trees[i], hs[i])
                s.synchronize()
                if not (torch.equal(got.pool[:-256], refs[i].pool[:-256]) and torch.equal(got.meta, refs[i].meta)):
                    bad.append(i)
    th = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for x in th:
        x.start()
    for x in th:
        x.join()
    assert not bad
