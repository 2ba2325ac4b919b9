"""Which GPU amr_pack_pool allocates, copies and launches on, with two GPUs played on the host
(fake_hip.cpp): kernels run only where the pool, the metadata and the stream belong to one GPU, and on
that GPU; the caller's current device is what it was afterwards, and nothing stays allocated.  Any other
combination is packed on the host and copied.  Host memory that runs out in a worker thread is an error
returned, and threads that cannot be started are done without."""
import os
import shutil
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    gxx = shutil.which("g++")
    if not gxx:
        pytest.skip("g++ not available")
    lib = str(tmp_path_factory.mktemp("fake_hip") / "libfake_hip.so")
    r = subprocess.run([gxx, "-std=c++17", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include",
                        os.path.join(HERE, "fake_hip.cpp"), "-o", lib, "-ldl"], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return lib


def run(fake, pool, meta, stream, current, fail_malloc=0, limit="", capturing=0, fail_launch=0):
    r = subprocess.run([sys.executable, os.path.join(HERE, "_fake_hip_run.py"), fake] +
                       [str(v) for v in (pool, meta, stream, current, fail_malloc, limit, capturing, fail_launch)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    lines = r.stdout.strip().splitlines()
    assert lines[-1] == "end rc=%d current=%d leaked=0" % (5 if fail_launch else 0, current), r.stdout
    if limit:
        return [int(v) for v in lines[0].split()[1:]]
    return [(w, int(d)) for w, d in (ln.split() for ln in lines[:-1])]


@pytest.mark.parametrize("current", [0, 1])
@pytest.mark.parametrize("stream", [-1, 1])
def test_packs_on_the_gpu_of_the_pool(fake, stream, current):
    calls = run(fake, 1, 1, stream, current)
    assert sum(w == "launch" for w, _ in calls) >= 3 and any(w == "copy" for w, _ in calls)
    assert {d for _, d in calls} == {1}


@pytest.mark.parametrize("pool,meta,stream", [(1, 1, 0), (0, 0, 1), (0, 1, 0), (1, 0, -1), (1, -1, -1)])
def test_packs_on_the_host_across_gpus(fake, pool, meta, stream):
    calls = run(fake, pool, meta, stream, 0)
    assert {w for w, _ in calls} == {"copy"}


@pytest.mark.parametrize("allocation", [1, 2])
def test_packs_on_the_host_without_room(fake, allocation):
    calls = run(fake, 1, 1, -1, 0, fail_malloc=allocation)
    assert not any(w == "launch" for w, _ in calls)
    assert [d for w, d in calls if w == "copy"][-2:] == [0, 0]          # as the caller's device has it


@pytest.mark.parametrize("stream", [-1, 1])
def test_waits_for_no_other_stream(fake, stream):
    """No call that waits for the whole GPU, no stream of its own (the runtime puts those on hardware
    queues that others use), every copy on the caller's."""
    calls = run(fake, 1, 1, stream, 1)
    assert {w for w, _ in calls} == {"malloc", "copy", "launch", "free"}


def test_a_stream_being_captured_sees_copies_only(fake):
    assert {w for w, _ in run(fake, 1, 1, 1, 1, capturing=1)} == {"copy"}


def test_an_error_leaves_no_copy_behind(fake):
    """A launch that fails (AMR_EHIP): the copies enqueued before it read host memory that is freed."""
    calls = run(fake, 1, 1, 1, 1, fail_launch=1)
    assert not any(w == "source-changed" for w, _ in calls) and any(w == "free" for w, _ in calls)


@pytest.mark.parametrize("pool", [1, -1])
def test_host_memory_runs_out_in_a_worker(fake, pool):
    rcs = run(fake, pool, pool, -1, 0, limit="memory")
    assert rcs[-1] == 0 and len(rcs) > 100 and set(rcs[:-1]) == {4}      # AMR_ENOMEM


@pytest.mark.parametrize("pool", [1, -1])
def test_threads_that_cannot_be_started(fake, pool):
    assert run(fake, pool, pool, -1, 0, limit="threads") == [0] * 7
