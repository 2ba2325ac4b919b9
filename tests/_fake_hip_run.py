"""Packs a small hierarchy for a chosen GPU against the stand-in runtime of fake_hip.cpp and prints
what was called: python _fake_hip_run.py FAKE_LIB POOL_DEVICE META_DEVICE STREAM_DEVICE CURRENT FAIL_MALLOC [LIMIT [CAPTURING [FAIL_LAUNCH]]]
(STREAM_DEVICE -1: the null stream; LIMIT memory: again and again, with one more allocation left to
the worker threads each time, until it succeeds; LIMIT threads: with 0 .. 6 threads to be had; the line
"rcs" then holds every return code).  A process of its own, since the stand-in has to be loaded before
anything that brings the real runtime along."""
import ctypes
import importlib.util
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def main():
    fake = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
    pool_dev, meta_dev, stream_dev, current, fail = (int(v) for v in sys.argv[2:7])
    spec = importlib.util.spec_from_file_location("_lib", os.path.join(ROOT, "paper_1212_3333_amd", "_lib.py"))
    L = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(L)
    lib = ctypes.CDLL(L.LIB_PATH)
    vp, i64 = ctypes.c_void_p, ctypes.c_int64
    lib.amr_build_kdtree.argtypes = [vp, vp, ctypes.c_int32, vp]
    lib.amr_pack_pool.argtypes = [vp, vp, ctypes.c_int32, vp, vp, vp, vp, vp, vp, vp]
    lib.amr_last_error.restype = ctypes.c_char_p
    fake.fake_alloc.argtypes, fake.fake_alloc.restype = [ctypes.c_size_t, ctypes.c_int], vp
    fake.fake_stream.argtypes = [vp, ctypes.c_int]
    fake.fake_log.restype = ctypes.c_char_p
    fake.fake_held.restype = ctypes.c_long

    limit = sys.argv[7] if len(sys.argv) > 7 else ""
    boxes = [(0, (0, 0, 0), (8, 8, 8)), (1, (4, 4, 4), (6, 8, 6))]
    if limit:      # more leaf records than one thread takes at a time
        boxes = [(0, (2 * i, 2 * j, 2 * k), (2, 2, 2)) for k in range(5) for j in range(5) for i in range(5)]
        boxes += [(1, (6, 6, 6), (4, 4, 4))]
    patches = (L.amr_patch * len(boxes))()
    keep = []
    for i, (level, lo, dims) in enumerate(boxes):
        cells = (ctypes.c_float * (dims[0] * dims[1] * dims[2]))(*range(dims[0] * dims[1] * dims[2]))
        keep.append(cells)
        patches[i].level = level
        patches[i].lo[:] = lo
        patches[i].dims[:] = dims
        patches[i].cells = ctypes.addressof(cells)
    dom = L.amr_domain()
    dom.origin[:] = (0.0, 0.0, 0.0)
    dom.h0[:] = (0.125,) * 3
    dom.refine, dom.nlevels = 2, 2
    tree = vp()
    assert lib.amr_build_kdtree(ctypes.byref(dom), patches, len(boxes), ctypes.byref(tree)) == 0, lib.amr_last_error()
    opts = L.amr_pack_opts()
    opts.brick_layout, opts.nthreads = 2, 4
    pb, mb = i64(0), i64(0)
    assert lib.amr_pack_pool(tree, patches, len(boxes), ctypes.byref(opts), None, ctypes.byref(pb), None, ctypes.byref(mb),
                             None, None) == 0
    pool, meta = fake.fake_alloc(pb.value, pool_dev), fake.fake_alloc(mb.value, meta_dev)
    stream = vp(None)
    if stream_dev >= 0:
        stream = vp(0x1000)
        fake.fake_stream(stream, stream_dev)
    fake.fake_call_stream(stream)
    fake.fake_capturing(int(sys.argv[8]) if len(sys.argv) > 8 else 0)
    fake.fake_fail_launch(int(sys.argv[9]) if len(sys.argv) > 9 else 0)
    fake.fake_fail_malloc(fail)
    fake.hipSetDevice(current)
    fake.fake_clear()
    held = fake.fake_held()
    scene = L.amr_scene()

    def pack():
        return lib.amr_pack_pool(tree, patches, len(boxes), ctypes.byref(opts), pool, ctypes.byref(pb), meta,
                                 ctypes.byref(mb), ctypes.byref(scene), stream)

    rcs = []
    for k in range(5000) if limit == "memory" else range(7) if limit == "threads" else ():
        fake.fake_limits(ctypes.c_long(k if limit == "memory" else -1), k if limit == "threads" else -1)
        rcs.append(pack())
        if limit == "memory" and rcs[-1] == 0:
            break
    fake.fake_limits(ctypes.c_long(-1), -1)
    fake.fake_clear()
    rc = pack()
    dev = ctypes.c_int(-1)
    fake.hipGetDevice(ctypes.byref(dev))
    if rcs:
        print("rcs", *rcs)
    sys.stdout.write(fake.fake_log().decode())
    print("end rc=%d current=%d leaked=%d" % (rc, dev.value, fake.fake_held() - held))


main()
