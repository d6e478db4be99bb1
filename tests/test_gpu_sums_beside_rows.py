"""Small patterns with column sums in one launch: some workgroups form the sums over all rows, the others run the rows.  Edges of the
rule and of the tiles, results against the oracle, and calls whose outputs share memory (which take the fold's own launch)."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2009_10924_amd import binding as B
from workloads import bias_gelu_dbias_graph, layernorm_backward_graph, make_inputs, rmsnorm_backward_graph, softmax_graph

from .gpu_util import check, floors_for, note, run_spec

pytestmark = pytest.mark.skipif(not B.codegen_available(), reason="needs the run-time compiler")
GRAPHS = {"gelu": bias_gelu_dbias_graph, "layernorm": layernorm_backward_graph, "rmsnorm": rmsnorm_backward_graph}


def _at_once(spec, **opts):
    return [l for l in B.Plan(B.Graph.from_spec(spec), "auto", **opts).describe().splitlines() if l.startswith("at_once")]


# two rows of one or two steps, rows below and beyond a batch, one lane more than a tile of columns, a last tile of one element, the last row
# count of the rule for each number of columns per workgroup, rows on workgroups
SHAPES = [(2, 8, "f32"), (3, 16, "bf16"), (127, 17, "f16"), (129, 64, "f32"), (1024, 64, "bf16"), (1024, 33, "f32"), (512, 768, "bf16"), (513, 760, "f16"),
          (65, 1001, "f16"), (390, 1001, "f32"), (512, 768, "f32"), (31, 385, "f32"), (256, 3072, "bf16"), (255, 3073, "f16"), (192, 8192, "bf16"),
          (95, 8191, "f32"), (33, 12288, "f16")]


@pytest.mark.gpu
@pytest.mark.parametrize("kind", sorted(GRAPHS))
@pytest.mark.parametrize("rows,cols,dtype", SHAPES)
def test_against_the_oracle(kind, rows, cols, dtype):
    spec = GRAPHS[kind](rows, cols, dtype)
    assert _at_once(spec) or (rows, cols) == (513, 760)
    inp = make_inputs(spec, seed=rows + cols)
    ref = O.evaluate(spec, inp)
    floors = floors_for(spec, inp, ref)
    got, _, _, _ = run_spec(spec, inp, repeat=3)
    for name, dt in spec.outputs:
        e = check(got[name], ref[name].reshape(got[name].shape), dt, floors.get(name, 0.0), f"{spec.name}/{name}")
        note(f"{spec.name}/{name}: {e}")


@pytest.mark.gpu
@pytest.mark.parametrize("kind", sorted(GRAPHS))
def test_an_output_over_an_input(kind):
    """The gradient of the input over the gradient of the output: the sums still see every row as it was."""
    import torch
    spec = GRAPHS[kind](200, 768, "bf16")
    assert _at_once(spec)
    inp = make_inputs(spec, seed=2)
    ref = O.evaluate(spec, inp)
    floors = floors_for(spec, inp, ref)
    plan = B.Plan(B.Graph.from_spec(spec), "auto")
    names = [t.name for t in spec.inputs]
    shapes = B.output_shapes(spec)
    for i, t in enumerate(spec.inputs):
        if tuple(t.dims) != (200, 768):
            continue
        dev_in = [B.to_device(inp[n.name], n.dtype) for n in spec.inputs]
        dev_out = B.alloc_outputs(spec)
        k = [j for j, (n, _) in enumerate(spec.outputs) if tuple(shapes[n]) == (200, 768)][0]
        dev_out[k] = dev_in[i]
        plan.execute(dev_in, dev_out, plan.make_workspace())
        torch.cuda.synchronize()
        for (name, dt), o in zip(spec.outputs, dev_out):
            got = O.to_f64(B.to_host(o, dt), dt)
            check(got, ref[name].reshape(got.shape), dt, floors.get(name, 0.0), f"{spec.name}/{name} over {names[i]}")


def test_where_it_is_not_offered():
    """A caller's own choice of a shape, sizes beyond the rule, no column sums, and sums of what a row reduction went into."""
    small = layernorm_backward_graph(64, 768, "bf16")
    assert _at_once(small) and not _at_once(small, candidate=0)
    assert not _at_once(layernorm_backward_graph(1025, 64, "bf16")) and not _at_once(rmsnorm_backward_graph(513, 768, "bf16"))
    assert not _at_once(softmax_graph(64, 128, "f32"))
    g = B.Graph()
    x = g.input("f32", (64, 128))
    m = g.op("reduce_max", [x], axis=1)
    y = g.op("sub", [x, m])
    g.output(y, "f32")
    g.output(g.op("reduce_sum", [y], axis=0), "f32")
    g.finalize()
    assert "at_once" not in B.Plan(g, "auto").describe()


@pytest.mark.gpu
def test_under_capture_on_another_stream_and_without_a_workspace():
    """Replayed from a captured graph, on a stream of its own beside the default one's work, and through fs_execute_static: the same bits."""
    import torch
    from .test_gpu_graph_capture import _capture_and_replay
    for kind in sorted(GRAPHS):
        spec = GRAPHS[kind](200, 768, "bf16")
        assert _at_once(spec)
        plan = B.Plan(B.Graph.from_spec(spec), "auto")
        inp = make_inputs(spec, seed=3)
        ins = [B.to_device(inp[t.name], t.dtype) for t in spec.inputs]
        outs, again = B.alloc_outputs(spec), B.alloc_outputs(spec)
        ws = plan.make_workspace()
        i, o, a = ([t.data_ptr() for t in ts] for ts in (ins, outs, again))

        def call(stream):
            plan.execute_ptrs(i, o, ws.data_ptr(), ws.numel(), stream)
        _capture_and_replay(call, outs, lambda k: ins[0].mul_(1.0))
        call(torch.cuda.current_stream().cuda_stream)
        side = torch.cuda.Stream()
        for run in (lambda: plan.execute_ptrs(i, a, ws.data_ptr(), ws.numel(), side.cuda_stream), lambda: plan.execute_static_ptrs(i, a, side.cuda_stream)):
            for t in again:
                t.fill_(float("nan"))
            torch.cuda.synchronize()
            run()
            ins[0].mul_(1.0)   # (the default stream's own)
            side.synchronize()
            torch.cuda.synchronize()
            for x, y in zip(again, outs):
                assert torch.equal(x.view(torch.uint8), y.view(torch.uint8)), kind
