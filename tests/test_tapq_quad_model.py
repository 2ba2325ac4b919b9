"""The deferred-tap queue as the lit kernels use it with four lanes per ray, played on the host
(tests/tapq_quad_model.cpp, built with AddressSanitizer and UndefinedBehaviorSanitizer): the stepped loop with
and without checkpoints and the persistent kernel's per-segment loop, each with the queue that is resolved
one sample per lane and with the one that is resolved one tap per lane.  Driven by seeded streams, from
no queued sample to every sample queued with all six taps, with early ends and empty rays, and by the
streams of a real view (the oracle's segment lists, see test_tapq_model)."""
import os
import shutil
import subprocess

import numpy as np
import pytest

import workloads
from test_tapq_model import _view_waves

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
KTAPQ = 64
MODES = [(loop, lst, ckpt) for loop in (0, 1) for lst in (0, 1) for ckpt in ((0, 1) if loop == 0 else (0,))]


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    gxx = shutil.which("g++")
    if not gxx:
        pytest.skip("g++ not available")
    exe = str(tmp_path_factory.mktemp("tapq") / "tapq_quad_model")
    r = subprocess.run([gxx, "-std=c++17", "-O1", "-g", "-fno-omit-frame-pointer", "-fsanitize=address,undefined",
                        "-fno-sanitize-recover=undefined", "-I", os.path.join(ROOT, "paper_1212_3333_amd", "csrc"),
                        os.path.join(ROOT, "tests", "tapq_quad_model.cpp"), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return exe


def _run(exe, mode, waves):
    """waves: lists of 16 rays, each a list of segments, each a list of flags."""
    out = ["%d %d %d %d" % (*mode, len(waves))]
    for rays in waves:
        assert len(rays) == 16
        for segs in rays:
            out.append(" ".join([str(len(segs))] + ["%d %s" % (len(s), " ".join(map(str, s))) for s in segs]))
    r = subprocess.run([exe], input="\n".join(out) + "\n", capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, (r.returncode, r.stdout, r.stderr[-3000:])
    s = {k: int(v) for k, v in (kv.split("=") for kv in r.stdout.split()[1:])}
    assert s["max_count"] <= KTAPQ and s["max_taps"] <= (6 * KTAPQ if mode[1] else 0)
    return s


def _synthetic(seed, p_queue, taps, nwaves=24, p_end=0.002):
    rng = np.random.default_rng(seed)
    waves = []
    for _ in range(nwaves):
        rays = []
        for _ in range(16):
            segs = []
            for _ in range(0 if rng.random() < 0.05 else int(rng.integers(1, 40))):
                n = int(rng.geometric(0.08)) - 1 if rng.random() < 0.9 else 0
                m = np.where(rng.random(n) < p_queue, rng.integers(1, 64, n) if taps == "any" else taps, 0)
                segs.append([int(v) for v in m + 64 * (rng.random(n) < p_end)])
            rays.append(segs)
        waves.append(rays)
    return waves


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("p_queue,taps", [(0.0, 1), (0.19, 1), (0.19, "any"), (0.6, "any"), (1.0, 1), (1.0, 63), (1.0, "any")])
def test_synthetic_streams(model, mode, p_queue, taps):
    s = _run(model, mode, _synthetic(7 + int(100 * p_queue), p_queue, taps))
    assert s["samples"] > 1000 and (s["queued"] > 0) == (p_queue > 0)


@pytest.mark.parametrize("mode", MODES)
def test_one_ray_and_full_pressure(model, mode):
    one = [[] for _ in range(16)]
    one[9] = [[63] * 299 + [127]]
    full = [[[63] * 200] for _ in range(16)]                       # every step fills the empty queue
    ends = [[[1, 64 + 1, 1, 1, 1]] for _ in range(16)]             # a quad mate ends the ray
    s = _run(model, mode, [one, full, ends])
    assert s["queued"] == 300 + 16 * 200 + 16 * 2
    assert s["max_count"] == 64 and (mode[1] == 0 or s["max_taps"] == 384)


def _quads(waves, seed):
    """Waves of 64 lanes of segments (n, leaf, patch, off, flags) as waves of 16 rays with random pending taps."""
    rng = np.random.default_rng(seed)
    out = []
    for lanes in waves:
        for q in range(4):
            rays = []
            for segs in lanes[16 * q:16 * q + 16]:
                rays.append([[int((rng.integers(1, 64) if f in (1, 2) else 0) + (64 if f >= 2 else 0)) for f in s[4]] for s in segs])
            out.append(rays)
    return out


def test_view_streams(model):
    h, lut, cams, prm = workloads.small_nested(0)
    waves, _, _ = _view_waves(h, cams[1], lut, dict(prm, lighting=True), [(tx, ty) for ty in range(0, 32, 5) for tx in range(0, 32, 5)])
    for mode in MODES:
        s = _run(model, mode, _quads(waves, 1))
        assert s["queued"] > 0 and s["flushes"] > 0
