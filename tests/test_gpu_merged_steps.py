"""A program run as a whole takes its independent steps, and the folds of column sums, in few launches; stage by stage every step
has its own.  Both store the same bits, run after run on one workspace, also where an output shares memory with an input (which
sends the whole run step by step)."""
import numpy as np
import pytest

from paper_2009_10924_amd import binding as B
from workloads import (gelu_backward_graph, layernorm_backward_bias_graph, make_inputs, rmsnorm_backward_graph, silu_gate_graph,
                       transformer_block_backward_graph)

from .gpu_util import side_by_side

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not B.codegen_available(), reason="needs the run-time compiler")]


def _runner(spec, graph):
    import torch
    inp = make_inputs(spec, seed=6)
    stream = torch.cuda.current_stream().cuda_stream

    def run(prog, staged, times=1, shared=()):
        ins = [B.to_device(inp[t.name], t.dtype) for t in spec.inputs]
        outs = B.alloc_outputs(spec)
        for t in outs:
            t.fill_(float("nan"))
        for o, i in shared:
            outs[o] = ins[i] if i >= 0 else outs[~i]
        ws = prog.make_workspace()
        ws.fill_(255)
        a, b = [t.data_ptr() for t in ins], [t.data_ptr() for t in outs]
        for _ in range(times):
            if staged:
                for k in range(prog.info["n_stages"]):
                    prog.bind_stage(k, a, b, ws.data_ptr(), ws.numel(), stream)()
            else:
                prog.bind(a, b, ws.data_ptr(), ws.numel(), stream)()
        torch.cuda.synchronize()
        return [B.to_host(t, dt).view(np.uint8).copy() for (_, dt), t in zip(spec.outputs, outs)]
    return run


def _merged(prog):
    return [l for l in prog.describe().splitlines() if l.startswith("merged ")]


# one row per lane group and many, rows on workgroups, packed transposes, a batch of few rows, the benchmark's block
@pytest.mark.parametrize("dims,dtype", [((2, 16, 4, 32, 128), "bf16"), ((6, 16, 4, 32, 512), "f16"), ((3, 34, 12, 64, 3072), "f16"), ((5, 67, 8, 64, 2048), "bf16"),
                                        ((29, 88, 12, 32, 1536), "f16"), ((32, 128, 12, 64, 3072), "bf16")])
def test_whole_run_equals_stage_by_stage(dims, dtype):
    spec = transformer_block_backward_graph(*dims, dtype)
    graph = B.Graph.from_spec(spec)
    prog = B.Program(graph)
    apart = B.Program(graph, no_joint_folds=True)
    lines = _merged(prog)
    assert len(lines) == 3 < prog.info["n_kernels"] and not _merged(apart), prog.describe()
    run = _runner(spec, graph)
    want = run(prog, True)
    for got in (run(prog, False), run(prog, False, times=3), run(apart, False)):
        for (name, _), a, b in zip(spec.outputs, got, want):
            assert np.array_equal(a, b), name


def test_an_output_that_shares_memory_with_an_input():
    """The gradient of the scores over the gradient of the probabilities: every step still finds its inputs."""
    spec = transformer_block_backward_graph(3, 24, 4, 32, 128, "bf16")
    graph = B.Graph.from_spec(spec)
    prog = B.Program(graph)
    assert _merged(prog)
    names = [t.name for t in spec.inputs]
    shared = [(k, names.index("up_probs")) for k, (n, _) in enumerate(spec.outputs)
              if any(o.out == n and o.opcode != "transpose" for o in spec.ops) and dict((t.name, tuple(t.dims)) for t in spec.inputs)["up_probs"]
              == tuple(B.output_shapes(spec)[n])]
    assert len(shared) == 1
    run = _runner(spec, graph)
    for (name, _), a, b in zip(spec.outputs, run(prog, False, shared=shared), run(prog, True, shared=shared)):
        assert np.array_equal(a, b), name


def test_outputs_that_share_memory():
    """The results of two steps in one buffer: the later step's stays, and what reads the earlier one has read it by then."""
    spec = transformer_block_backward_graph(3, 24, 4, 32, 128, "bf16")
    graph = B.Graph.from_spec(spec)
    prog = B.Program(graph)
    assert _merged(prog)
    same = [k for k, (n, _) in enumerate(spec.outputs) if n.endswith("_dxc")]   # of one type and shape, each by a step of its own
    assert len(same) == 3
    run = _runner(spec, graph)
    for a, b in ((1, 0), (2, 0), (2, 1)):
        shared = [(same[a], ~same[b])]
        for (name, _), x, y in zip(spec.outputs, run(prog, False, shared=shared), run(prog, True, shared=shared)):
            assert np.array_equal(x, y), (name, shared)


# a gate beside the sums, one moved behind them, the longer workgroups first, and three programs of one launch for all sums
@pytest.mark.parametrize("members", [lambda: [layernorm_backward_bias_graph(33, 768, "bf16"), rmsnorm_backward_graph(70, 1536, "bf16"), silu_gate_graph(100, 2048, "bf16")],
                                     lambda: [layernorm_backward_bias_graph(64, 768, "f16"), rmsnorm_backward_graph(64, 1536, "f16"), silu_gate_graph(16384, 2048, "bf16")],
                                     lambda: [gelu_backward_graph(1024, 3072), layernorm_backward_bias_graph(8192, 768, "bf16")],
                                     lambda: [layernorm_backward_bias_graph(129, 768, "f32"), layernorm_backward_bias_graph(65, 512, "f32")]])
def test_independent_patterns_equal_launches_of_their_own(members):
    spec = side_by_side(members())
    graph = B.Graph.from_spec(spec)
    prog = B.Program(graph)
    assert len(_merged(prog)) == 2
    run = _runner(spec, graph)
    want = run(B.Program(graph, no_joint_folds=True), False)
    for got in (run(prog, False), run(prog, False, times=3)):
        for (name, _), a, b in zip(spec.outputs, got, want):
            assert np.array_equal(a, b), name
