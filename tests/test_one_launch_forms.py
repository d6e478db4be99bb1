"""The one-launch form of small patterns with column sums, and merged launches of explored programs, as the host sees them: what the
listings say of them and where they are not taken."""
import re

import pytest

from paper_2009_10924_amd import binding as B
from workloads import (bias_gelu_dbias_graph, gelu_backward_graph, layernorm_backward_bias_graph, layernorm_backward_graph, log_softmax_graph,
                       rmsnorm_backward_graph, rmsnorm_graph, silu_gate_graph, transformer_block_backward_graph,
                       transpose_graph)

from .gpu_util import side_by_side

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
    source = plan.source()   # of the listed launches, of the one launch where those are compiled in
    runs = "fs_gen_row_" if plan.info["kernel"].startswith("row_generated") else m[1]
    assert source.count("__global__") == 1 and f" {runs}" in source and "@ENTRY@" not in source
    assert _plan(rmsnorm_graph(64, 768)).source().count("fs_gen_sums_") == 0


def test_merged_launches_name_their_kernels():
    prog = B.Program(B.Graph.from_spec(transformer_block_backward_graph(2, 16, 4, 32, 128, "bf16")))
    lines = [l for l in prog.describe().splitlines() if l.startswith("merged ")]
    assert lines and all(re.search(r" entry=fs_gen_merged_[0-9a-f]{8} workgroups=[1-9]\d* vgprs=\d+ lds=\d+$", l) for l in lines), lines


def _steps_of_launches(members):
    """(launches of the program's stages, the steps of each merged launch)"""
    prog = B.Program(B.Graph.from_spec(side_by_side(members)))
    merged = [re.search(r" steps=([\d,]*) ", l)[1] for l in prog.describe().splitlines() if l.startswith("merged ")]
    return prog.info["n_kernels"], merged


def test_steps_that_would_cost_a_launch_more_than_it_saves_stay_out_of_it():
    """A step that streams 32 bytes a lane goes to a launch without looping workgroups unless they are at work as long; on 64 bytes it
    stays.  Where the longest workgroups are not all resident they come first; where those with row reductions need a second
    round, nothing is merged."""
    norms = [layernorm_backward_bias_graph(512, 768, "bf16"), rmsnorm_backward_graph(512, 1536, "bf16")]
    assert _steps_of_launches(norms + [silu_gate_graph(16384, 2048, "bf16")]) == (3, ["0,1", "2"])
    assert _steps_of_launches(norms + [silu_gate_graph(1024, 2048, "bf16")]) == (3, ["0,1,2", ""])
    wide = [layernorm_backward_bias_graph(2048, 1024, "bf16")] * 2
    assert _steps_of_launches(wide + [silu_gate_graph(2048, 4096, "bf16")]) == (3, ["0,1,2", ""])
    assert _steps_of_launches([gelu_backward_graph(1024, 3072), layernorm_backward_bias_graph(8192, 768, "bf16")]) == (3, ["1,0", ""])
    assert _steps_of_launches([gelu_backward_graph(8192, 3072), layernorm_backward_bias_graph(8192, 768, "bf16")]) == (3, ["0,1", ""])
    assert _steps_of_launches([layernorm_backward_bias_graph(32768, 768, "bf16"), rmsnorm_backward_graph(32768, 1536, "bf16"),
                               silu_gate_graph(4096, 2048, "bf16")]) == (3, [])


def _merged(spec_or_graph):
    graph = spec_or_graph if isinstance(spec_or_graph, B.Graph) else B.Graph.from_spec(spec_or_graph)
    prog = B.Program(graph)
    return prog, [l for l in prog.describe().splitlines() if l.startswith("merged ")]


def _moves(n):
    """Transposes, each a step of its own and of another size."""
    return [transpose_graph((64 + 8 * i, 128, 12, 64), (0, 2, 1, 3), "bf16") for i in range(n)]


def test_programs_that_are_not_merged():
    """More than twelve steps, a row on 512 lanes, a row in chunks."""
    assert len(_merged(side_by_side(_moves(12)))[1]) == 1 and not _merged(side_by_side(_moves(13)))[1]
    for cols, merged in ((4096, 1), (12000, 0), (70000, 0)):
        prog, lines = _merged(side_by_side(_moves(2) + [log_softmax_graph(700, cols, "f32")]))
        assert len(lines) == merged, (cols, prog.describe())


def test_a_sum_that_a_later_step_reads_keeps_the_steps_apart():
    def program(reads):
        g = B.Graph()
        for k in range(2):
            g.output(g.op("transpose", [g.input("bf16", (64 + 8 * k, 128, 768))], perm=(1, 0, 2)), "bf16")
        x, w = g.input("f32", (4096, 768)), g.input("f32", (4096, 768))
        s = g.op("reduce_sum", [g.op("mul", [x, w])], axis=0)
        g.output(s, "f32")
        other = s if reads else g.input("f32", (768,))
        y = g.op("mul", [w, g.op("broadcast", [other], dims=(4096, 768), map=(1,))])
        g.output(g.op("div", [y, g.op("broadcast", [g.op("reduce_max", [y], axis=1)], dims=(4096, 768), map=(0,))]), "f32")
        g.finalize()
        return g
    assert _merged(program(False))[1]
    prog, lines = _merged(program(True))
    assert not lines and prog.info["n_steps"] >= 3, prog.describe()


def test_workspace_that_serves_two_tensors_in_turn_keeps_the_steps_apart():
    def program(links):   # normalised rows, transposed in between: each link lies in the workspace
        g = B.Graph()
        for k in range(2):
            g.output(g.op("transpose", [g.input("bf16", (64 + 8 * k, 128, 768))], perm=(1, 0, 2)), "bf16")
        dims = (64, 128, 64)
        x = g.input("f32", dims)
        for link in range(links + 1):
            y = g.op("mul", [g.op("exp", [x]), g.op("broadcast", [g.op("reduce_max", [x], axis=2)], dims=dims, map=(0, 1))])
            if link < links:
                x, dims = g.op("transpose", [y], perm=(1, 0, 2)), (dims[1], dims[0], dims[2])
        g.output(y, "f32")
        g.finalize()
        return _merged(g)

    def places(prog):
        return re.findall(r"output 0 (ws\+\d+)", prog.describe())
    prog, lines = program(2)
    assert lines and len(set(places(prog))) == len(places(prog)) == 2
    prog, lines = program(3)
    assert not lines and len(set(places(prog))) < len(places(prog)) == 3
