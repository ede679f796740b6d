"""The autotuner leaves out candidates whose step fails (CPU: its host code with the entry points
it calls and the HIP runtime replaced, tests/native/tune_mock.cpp)."""
import os
import shutil
import subprocess

import pytest

from paper_2609_29977_amd import bmpc
from paper_2609_29977_amd.build import CSRC, FLAGS, HIPCC

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CANDIDATES = 4  # sweep mappings per window depth; the replaced plan allows depths 1..4


@pytest.fixture(scope="module")
def tuner(tmp_path_factory):
    if shutil.which(HIPCC) is None:
        pytest.skip("hipcc not available")
    d = tmp_path_factory.mktemp("tune")
    objs = []
    for src in (os.path.join(CSRC, "tune.hip"), os.path.join(ROOT, "tests", "native",
                                                             "tune_mock.cpp")):
        objs.append(str(d / (os.path.basename(src) + ".o")))
        cmd = [HIPCC, "--cuda-host-only", *FLAGS, "-O1", "-x", "hip", "-c", src, "-o", objs[-1]]
        r = subprocess.run(cmd, capture_output=True, text=True)
        assert r.returncode == 0, r.stderr
    exe = str(d / "tuner")
    # the device code's image is not there, and is not loaded by the replaced runtime
    r = subprocess.run(["g++", "-no-pie", *objs, "-o", exe, "-Wl,--unresolved-symbols=ignore-all"],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return exe


@pytest.mark.parametrize("fp32", [0, 1])
@pytest.mark.parametrize("failing", [(), (1,), (2, 4), (1, 2, 3), (1, 2, 3, 4)])
def test_failing_candidates_are_left_out(tuner, failing, fp32):
    run = subprocess.run([tuner, str(sum(1 << d for d in failing)), str(fp32)],
                         capture_output=True, text=True, timeout=60)
    assert run.returncode == 0, run.stderr
    status, count, depth, ms = run.stdout.split()
    left = [d for d in (1, 2, 3, 4) if d not in failing]
    assert int(count) == CANDIDATES * len(left)
    if left:
        assert (int(status), int(depth), float(ms)) == (bmpc.OK, left[0], float(left[0]))
    else:
        assert int(status) == bmpc.ERR_DEVICE
