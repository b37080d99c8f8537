"""Host-side parts of the library compiled for the CPU alone, with the device calls stubbed."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1710_03431_amd", "csrc")
NATIVE = os.path.join(ROOT, "tests", "native")
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


def run_native(tmp_path, check, *sources):
    """Compile the check and the library's sources without device code, link them without the
    HIP runtime (the check supplies the calls they make) and run."""
    objs = []
    for src in [os.path.join(NATIVE, check)] + [os.path.join(CSRC, s) for s in sources]:
        obj = str(tmp_path / (os.path.basename(src) + ".o"))
        subprocess.run([HIPCC, "--offload-host-only", "-x", "hip", "--offload-arch=gfx950", "-O1", "-fPIC", "-std=c++17",
                        "-I" + os.path.join(ROOT, "include"), "-I" + CSRC, "-c", src, "-o", obj], check=True)
        objs.append(obj)
    exe = str(tmp_path / "check")
    subprocess.run(["g++", *objs, "-o", exe, "-lpthread"], check=True)
    return subprocess.run([exe], capture_output=True, text=True)


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
def test_workspace_cache_never_hands_out_a_smaller_block(tmp_path):
    """Mixed sizes and both parities of the block solver's buffer exchange."""
    res = run_native(tmp_path, "scratch_check.cpp", "scratch.hip")
    assert res.returncode == 0, res.stdout + res.stderr
