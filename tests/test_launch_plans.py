"""The launch plans of random networks, on the host (tests/launch_plans.cpp,
compiled here with the dispatcher; nothing runs on a GPU)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
# units of unequal size in the ERASE schedules: a chain's first unit holds the
# block on x, and block counts that are no multiple of a third of the network
UNEVEN = ["bf16 4096 512 x:1:c0:512,512 p:5:c0:512,512", "bf16 1651 512 x:1:c0:508,512 p:8:c0:508,512",
          "bf16 4096 1677 x:10:c0:512,256,128", "bf16 4096 1677 x:7:c0:512,256,128",
          "bf16 4096 1677 x:7:c2:1024,1024,512", "bf16 4096 512 x:7:c0:512,512"]
# first layers of chained blocks with a long contraction into few input columns
# (the undetached schedule's input gradient)
LONG = ["bf16 4096 512 x:1:c0:512 p:3:c0:1024,512", "bf16 3343 953 x:4:c0:563,21,608 p:2:c0:1326,596,608",
        "bf16 1810 1114 x:2:c0:26,1114 p:1:c0:1616,1114"]


@pytest.fixture(scope="module")
def checker(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None or not os.path.isdir("/opt/rocm/include"):
        pytest.skip("no host compiler or HIP headers")
    exe = str(tmp_path_factory.mktemp("plans") / "launch_plans")
    r = subprocess.run([cxx, "-std=c++17", "-O1", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                        "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2608_18469_amd", "csrc"),
                        os.path.join(ROOT, "tests", "launch_plans.cpp"), "-o", exe, "-L/opt/rocm/lib", "-lamdhip64",
                        "-lpthread", "-Wl,-rpath,/opt/rocm/lib"], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    return exe


def test_launch_plans(checker):
    r = subprocess.run([checker, "7", "5000", *UNEVEN, *LONG], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stdout[-4000:]
