"""Renders cameras of given sizes against the stand-in runtime of fake_hip.cpp, which takes no launch that HIP
would not: python _fake_hip_render.py FAKE_LIB FORM WxH[,WxH...] -> "rc N most-blocks M" and the calls made.
FORM: unlit, lit, nearest, light (point light), sched, sched-lit, ckpt."""
import ctypes
import importlib.util
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def main():
    fake = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
    form, sizes = sys.argv[2], [tuple(int(v) for v in s.split("x")) for s in sys.argv[3].split(",")]
    spec = importlib.util.spec_from_file_location("_lib", os.path.join(ROOT, "paper_1212_3333_amd", "_lib.py"))
    L = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(L)
    lib = ctypes.CDLL(L.LIB_PATH)
    vp = ctypes.c_void_p
    lib.amr_last_error.restype = ctypes.c_char_p
    lib.amr_sched_bytes.restype = lib.amr_render_work_bytes.restype = ctypes.c_int64
    fake.fake_log.restype = ctypes.c_char_p
    fake.fake_most_blocks.restype = ctypes.c_uint64
    at = 0x10000                                   # never read: no kernel runs
    s = L.amr_scene()
    s.pool = s.nodes = s.leaves = s.patches = s.leaf_faces = s.face_taps = at
    s.pool_bytes = s.meta_bytes = 1 << 20
    s.nnodes = s.nleaves = s.npatches = s.nlevels = 1
    s.brick_layout = 2
    cams = (L.amr_camera * len(sizes))()
    for c, (w, h) in zip(cams, sizes):
        c.width, c.height, c.tan_half_fov = w, h, 0.4
    q = L.amr_render_params()
    q.d_lut, q.v_hi, q.step_frac = at, 1.0, 0.5
    q.lighting = {"lit": 1, "sched-lit": 1, "light": 2, "ckpt": 1}.get(form, 0)
    q.interp = int(form == "nearest")
    npix = sum(w * h for w, h in sizes)
    if form.startswith("sched"):
        q.d_sched, q.sched_bytes = at, lib.amr_sched_bytes(cams, len(sizes))
    if form == "light":
        q.d_work, q.work_bytes, q.light_jobs = at, lib.amr_render_work_bytes(cams, len(sizes), ctypes.byref(q)), 0
    if form == "ckpt":
        q.d_ckpt, q.ckpt_every, q.ckpt_max, q.ckpt_bytes = at, 4, 2, npix * 96 + 4096
    fake.fake_clear()
    rc = lib.amr_render(ctypes.byref(s), cams, len(sizes), ctypes.byref(q), vp(at), None, None)
    print("rc", rc, "most-blocks", fake.fake_most_blocks(), lib.amr_last_error().decode() if rc else "")
    sys.stdout.write(fake.fake_log().decode())


main()
