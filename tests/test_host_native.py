"""The library's host code compiled for the CPU alone and linked against a HIP runtime without a
device (tests/native/hip_stub.cpp), which records launches and waits and can run out of memory."""
import os
import re
import shutil
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1710_03431_amd", "csrc")
NATIVE = os.path.join(ROOT, "tests", "native")
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"

pytestmark = pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")


def compile_host(src, out):
    obj = os.path.join(out, os.path.basename(src) + ".o")
    subprocess.run([HIPCC, "--offload-host-only", "-x", "hip", "--offload-arch=gfx950", "-O1", "-fPIC", "-std=c++17",
                    "-I" + os.path.join(ROOT, "include"), "-I" + CSRC, "-I" + NATIVE, "-c", src, "-o", obj],
                   check=True)
    return obj


@pytest.fixture(scope="module")
def library(tmp_path_factory):
    """Host objects of every source and of the stub."""
    out = str(tmp_path_factory.mktemp("host"))
    srcs = [os.path.join(CSRC, f) for f in sorted(os.listdir(CSRC)) if f.endswith(".hip")]
    with ThreadPoolExecutor(max_workers=4) as ex:
        objs = list(ex.map(lambda s: compile_host(s, out), srcs + [os.path.join(NATIVE, "hip_stub.cpp")]))
    nm = subprocess.run(["nm", "-u", *objs], capture_output=True, text=True, check=True).stdout
    fat = sorted(set(re.findall(r"__hip_fatbin_\w+", nm)))   # device code left out
    return out, objs, ["-Wl,--defsym=%s=0" % f for f in fat]


def run_check(library, name):
    out, objs, syms = library
    exe = os.path.join(out, name + ".exe")
    obj = compile_host(os.path.join(NATIVE, name + ".cpp"), out)
    subprocess.run(["g++", "-no-pie", obj, *objs, *syms, "-o", exe, "-lpthread"], check=True)
    res = subprocess.run([exe], capture_output=True, text=True)
    assert res.returncode == 0, res.stdout + res.stderr


def test_workspace_cache_never_hands_out_a_smaller_block(library):
    """Mixed sizes and both parities of the block solver's buffer exchange; the bound, an allocation
    that needs the idle blocks, the release call, the last context, several threads."""
    run_check(library, "scratch_check")


def test_create_without_host_memory(library):
    """Each host allocation of aqt_create failing in turn."""
    run_check(library, "nomem_check")


def test_packed_operands(library):
    """Every allocation of a change of precision failing in turn; a change of precision while a
    batch on another stream reads the operands."""
    run_check(library, "pack_check")


def test_per_tile_sums_of_large_runs(library):
    """Memory limits at and below what the wider tiles need; the bound beyond which they are taken."""
    run_check(library, "plan_check")


def test_batch_widths_up_to_32_levels(library):
    """At the two limits of the rule, with and without autotuning; explicit widths, among them the
    4 that small batches report; the batch's per-tile sums."""
    run_check(library, "batch_check")


def test_chains_of_the_iterative_eigensolver(library):
    """Heads that fail together, in the first chunk and in a later one, whose first chain starts
    from the chunk before; fewer chains in less memory; the workspace of a short grid."""
    run_check(library, "chains_check")
