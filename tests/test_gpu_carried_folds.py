"""The joint folds of a program that ride in its last step's launch: the sums are those of folds in launches of their own, bit
for bit, stage by stage and several times over on one workspace; run as a whole, such a program takes merged launches, which store
the same bits too."""
import numpy as np
import pytest

from paper_2009_10924_amd import binding as B
from workloads import make_inputs, transformer_block_backward_graph

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,dtype", [((2, 16, 4, 32, 128), "bf16"), ((3, 24, 12, 32, 1536), "f16"), ((5, 67, 8, 64, 2048), "bf16")])
def test_joint_folds_in_the_last_steps_launch(dims, dtype):
    import torch
    if not B.codegen_available():
        pytest.skip("column sums inside patterns need the run-time compiler")
    spec = transformer_block_backward_graph(*dims, dtype)
    inp = make_inputs(spec, seed=4)
    dev_in = [B.to_device(inp[t.name], t.dtype) for t in spec.inputs]
    stream = torch.cuda.current_stream().cuda_stream

    def run(prog, stages, times):
        outs = B.alloc_outputs(spec)
        ws = prog.make_workspace()
        ins, ptrs = [t.data_ptr() for t in dev_in], [t.data_ptr() for t in outs]
        for _ in range(times):
            for t in outs:
                t.fill_(float("nan"))
            if stages:
                for k in range(prog.info["n_stages"]):
                    prog.bind_stage(k, ins, ptrs, ws.data_ptr(), ws.numel(), stream)()
            else:
                prog.bind(ins, ptrs, ws.data_ptr(), ws.numel(), stream)()
        torch.cuda.synchronize()
        return [B.to_host(t, dt).view(np.uint8).copy() for (_, dt), t in zip(spec.outputs, outs)]

    graph = B.Graph.from_spec(spec)
    carried, apart = B.Program(graph), B.Program(graph, no_joint_folds=True)
    assert " with_step=" in carried.describe() and carried.info["n_kernels"] == carried.info["n_steps"]
    want = run(apart, False, 1)
    for stages, times in ((False, 1), (False, 3), (True, 2)):
        for (name, _), a, b in zip(spec.outputs, run(carried, stages, times), want):
            assert np.array_equal(a, b), (name, stages, times)
