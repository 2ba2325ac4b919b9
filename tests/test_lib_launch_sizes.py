"""Image sizes that the raycaster's launches take, on the host: the runtime's stand-in (fake_hip.cpp) refuses a
launch of 2^32 threads or more along an axis, as HIP does.  Images of up to 32768 pixels on a side are
rendered, whatever their shape, and with a tile schedule fewer than 2^26 tiles; beyond, nothing is
enqueued.  At most three blocks in four of a launch lie outside the image."""
import os
import shutil
import subprocess
import sys

import pytest

from test_lib_pack_device import fake  # noqa: F401  (the built stand-in)

HERE = os.path.dirname(os.path.abspath(__file__))
FORMS = ["unlit", "lit", "nearest", "light", "ckpt"]


def render(lib, form, sizes):
    r = subprocess.run([sys.executable, os.path.join(HERE, "_fake_hip_render.py"), lib, form, sizes], capture_output=True,
                       text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    head, *calls = r.stdout.strip().splitlines()
    return int(head.split()[1]), int(head.split()[3]), [c.split()[0] for c in calls], head


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("size", ["1x1", "16384x64", "16385x64", "64x16392", "20000x100", "32768x32768", "32768x1"])
def test_sizes_that_are_rendered(fake, form, size):  # noqa: F811
    rc, _, calls, text = render(fake, form, size)
    assert rc == 0 and calls and set(calls) == {"launch"}, text


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("size", ["32769x8", "8x32769"])
def test_sizes_that_are_refused(fake, form, size):  # noqa: F811
    rc, _, calls, text = render(fake, form, size)
    assert rc != 0 and not calls, text


# super-tiles: 16x16 pixels lit, 32x32 unlit
@pytest.mark.parametrize("form,sizes,ok", [
    ("sched", "20000x100", True), ("sched", "100000x64", True), ("sched", "32768x32768", True),
    ("sched", "65504x65536", True), ("sched", "65536x65536", False),
    ("sched-lit", "32768x32768", True), ("sched-lit", "65504x65536", True), ("sched-lit", "65536x65536", False),
    ("sched", ",".join(["32768x8192"] * 8), True), ("sched-lit", ",".join(["32768x16384"] * 8), False)])
def test_scheduled_sizes(fake, form, sizes, ok):  # noqa: F811
    rc, _, calls, text = render(fake, form, sizes)
    assert (rc == 0) == ok and ("launch-refused" not in calls) and bool(calls) == ok, text


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("w,h", [(517, 389), (1024, 64), (64, 1024), (16384, 16), (1025, 1025), (901, 677), (8, 20000)])
def test_blocks_of_a_launch(fake, form, w, h):  # noqa: F811
    """At most four times as many super-tiles (of 64 one-wave blocks) as the frame has, to a multiple of eight."""
    _, blocks, _, text = render(fake, form, "%dx%d" % (w, h))
    st = -(-w // 32) * -(-h // 32)
    assert blocks <= 64 * (4 * st + 7), text


def test_tile_numbering(tmp_path):
    gxx = shutil.which("g++")
    if not gxx:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "tiles_model")
    r = subprocess.run([gxx, "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined", "-I",
                        os.path.join(os.path.dirname(HERE), "paper_1212_3333_amd", "csrc"),
                        os.path.join(HERE, "tiles_model.cpp"), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stderr
