"""Kernels that one call needs are compiled in one run of the compiler: each has its own figures, and is the kernel that it is alone."""
import os
import re
import struct
import subprocess
import sys

import pytest

from paper_2009_10924_amd import binding as B

pytestmark = pytest.mark.skipif(not B.codegen_available(), reason="the HIP run-time compiler is not installed here")
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = """
from paper_2009_10924_amd import binding as B
from workloads import layernorm_backward_graph, rmsnorm_backward_graph, transformer_block_backward_graph
small = rmsnorm_backward_graph(512, 760, "bf16")
plan = B.Plan(B.Graph.from_spec(small), "auto")
print("chosen", plan.info["candidate"], "vgprs", plan.info["vgprs"])
print(plan.describe())
print(B.Program(B.Graph.from_spec(transformer_block_backward_graph(2, 16, 4, 32, 128, "bf16"))).describe())
"""
ALONE = """
from paper_2009_10924_amd import binding as B
from workloads import rmsnorm_backward_graph
plan = B.Plan(B.Graph.from_spec(rmsnorm_backward_graph(512, 760, "bf16")), "auto", candidate=%s)
print("vgprs", plan.info["vgprs"])
"""


def _run(text, cache):
    os.makedirs(cache, exist_ok=True)
    env = dict(os.environ, FS_CODEGEN_CACHE_DIR=str(cache))
    r = subprocess.run([sys.executable, "-c", text], env=env, cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    return r.stdout


def _kernels(cache):
    """The kernels that the kept code objects were made for, by entry: (their own code's registers and LDS, kernels in it)."""
    found = {}
    for name in sorted(os.listdir(cache)):
        data = open(os.path.join(cache, name), "rb").read()
        n_source, n_code = struct.unpack("QQ", data[:16])
        entry = re.search(rb'extern "C" __global__ void [^{]*?(fs_gen_\w+)\(', data[16:16 + n_source])[1].decode()
        code = os.path.join(cache, name + ".elf")
        with open(code, "wb") as f:
            f.write(data[16 + n_source:])
        notes = subprocess.run(["/opt/rocm/llvm/bin/llvm-readelf", "--notes", code], capture_output=True, text=True).stdout
        os.remove(code)
        each = {re.search(r"\.name: +(fs_gen_\w+)", k)[1]: k for k in notes.split(".agpr_count:")[1:]}
        figure = lambda key: int(re.search(key + r": +(\d+)", each[entry])[1])  # noqa: E731
        found[entry] = (figure(r"\.vgpr_count"), figure(r"\.group_segment_fixed_size"), len(each))
    return found


@pytest.mark.skipif(not os.path.exists("/opt/rocm/llvm/bin/llvm-readelf"), reason="no tool to read code objects")
def test_each_kernel_of_one_run_has_its_own_figures(tmp_path):
    text = _run(PROGRAM, tmp_path / "a")
    kernels = _kernels(tmp_path / "a")
    listed = re.findall(r"entry=(fs_gen_(?:sums|merged)_\w+) .*?vgprs=(\d+) lds=(\d+)", text)
    assert len(listed) == 4   # the small plan's, and the block's three
    for entry, vgprs, lds in listed:
        assert kernels[entry][:2] == (int(vgprs), int(lds)), entry
    together = {e: k[2] for e, k in kernels.items()}
    assert together[listed[0][0]] == 2 and all(together[e] == 3 for e, _, _ in listed[1:]), together
    # read back from the directory, and compiled alone
    assert _run(PROGRAM, tmp_path / "a") == text
    m = re.search(r"chosen (\d+) vgprs (\d+)", text)
    assert _run(ALONE % m[1], tmp_path / "b").strip() == f"vgprs {m[2]}"
