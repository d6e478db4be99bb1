"""The one-launch form of small patterns with column sums, and merged launches of explored programs, as the host sees them: what the
listings say of them and where they are not taken."""
import re

import pytest

from paper_2009_10924_amd import binding as B
from workloads import (bias_gelu_dbias_graph, layernorm_backward_graph, rmsnorm_backward_graph, rmsnorm_graph, transformer_block_backward_graph)

pytestmark = pytest.mark.skipif(not B.codegen_available(), reason="the HIP run-time compiler is not installed here")


def _plan(spec, scheme="auto", **opts):
    return B.Plan(B.Graph.from_spec(spec), scheme, **opts)


# the chosen kernel compiled in (two families) and generated
@pytest.mark.parametrize("make", [layernorm_backward_graph, bias_gelu_dbias_graph, rmsnorm_backward_graph])
def test_source_and_listing_name_the_kernel_that_runs(make):
    plan = _plan(make(64, 768, "bf16"))
    line = [l for l in plan.describe().splitlines() if l.startswith("at_once ")]
    assert len(line) == 1
    m = re.search(r"entry=(fs_gen_sums_[0-9a-f]{8}) block=256 vgprs=(\d+) lds=(\d+)$", line[0])
    assert m and 16 <= int(m[2]) <= 256 and int(m[3]) > 0, line
    source = plan.source()
    assert source.count(f" {m[1]}(") == 1 and "@ENTRY@" not in source
    assert ("fs_gen_row_" in source) == plan.info["kernel"].startswith("row_generated")
    assert _plan(rmsnorm_graph(64, 768)).source().count("fs_gen_sums_") == 0


def test_merged_launches_name_their_kernels():
    prog = B.Program(B.Graph.from_spec(transformer_block_backward_graph(2, 16, 4, 32, 128, "bf16")))
    lines = [l for l in prog.describe().splitlines() if l.startswith("merged ")]
    assert lines and all(re.search(r" entry=fs_gen_merged_[0-9a-f]{8} workgroups=[1-9]\d* vgprs=\d+ lds=\d+$", l) for l in lines), lines
