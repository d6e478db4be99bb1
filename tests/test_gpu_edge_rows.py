"""Rows of an odd number of 16-bit elements, whose steps lie on the tensor's grid of whole vectors: the first and the last step of
every row slide inwards, by every amount, in every shape the generator offers.  Against the float64 oracle; in place, bit for bit,
the same as into another buffer (a step that slid stores elements of its neighbour a second time)."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2009_10924_amd import binding as B
from tests.gpu_util import all_candidates, floors_for, note, run_spec
from workloads import attention_scores_graph, log_softmax_graph, softmax_graph
from workloads.inputs import make_inputs

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not B.codegen_available(), reason="needs the run-time compiler")]


def _on_grid(spec, **opts):
    return "EDGE_" in B.Plan(B.Graph.from_spec(spec), "auto", **opts).source().rsplit('extern "C"', 1)[-1]


# every phase of a row against the grid (17 rows), one row, a last step of one element and of seven, rows that need the lane's last step
SHAPES = [("scores", 17, 9), ("scores", 3, 15), ("scores", 17, 57), ("scores", 5, 119), ("scores", 17, 121), ("scores", 9, 249), ("scores", 1, 505),
          ("softmax", 17, 1025), ("softmax", 2, 2041), ("log_softmax", 17, 2049), ("log_softmax", 9, 8191), ("log_softmax", 1, 16385),
          ("log_softmax", 9, 50257), ("log_softmax", 3, 65529), ("log_softmax", 3, 114681), ("log_softmax", 2, 131065)]


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("kind,rows,cols", SHAPES)
def test_rows_of_odd_length_in_every_shape(kind, rows, cols, dtype):
    if kind == "scores":
        spec = attention_scores_graph(3, 2, rows, cols, dtype=dtype)
    else:
        spec = (softmax_graph if kind == "softmax" else log_softmax_graph)(rows, cols, dtype)
    inp = make_inputs(spec, seed=cols)
    ref = O.evaluate(spec, inp)
    n = B.Plan(B.Graph.from_spec(spec), "auto").info["n_candidates"]
    some = 0
    for i in range(n):
        try:
            some += _on_grid(spec, candidate=i)
        except B.FsError as e:
            assert "scratch memory" in e.text
    assert some > 0 or cols < 17 or cols == 8191, "no shape of this pattern has its steps on the grid"   # (8191: every shape is full)
    worst = all_candidates(spec, inp, ref, floors_for(spec, inp, ref), unfused=False)
    note(f"{spec.name}: {some} of {n} candidates on the grid, worst {worst}")


@pytest.mark.parametrize("rows,cols,dtype", [(17, 2049, "bf16"), (9, 50257, "f16")])
def test_in_place(rows, cols, dtype):
    import torch
    spec = log_softmax_graph(rows, cols, dtype)
    assert _on_grid(spec)
    inp = make_inputs(spec, seed=3)
    _, raw, _, plan = run_spec(spec, inp)
    x = B.to_device(inp[spec.inputs[0].name], dtype)
    plan.execute_ptrs([x.data_ptr()], [x.data_ptr()], 0, 0, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert np.array_equal(B.to_host(x, dtype).view(np.uint8), raw[spec.outputs[0][0]].view(np.uint8))


@pytest.mark.parametrize("kind,cols,dtype", [("softmax", 74000, "f32"), ("log_softmax", 106496, "f32"), ("log_softmax", 131072, "f32"), ("log_softmax", 90113, "f32"),
                                             ("softmax", 114688 + 8, "bf16"), ("log_softmax", 128256, "f16")])
def test_chunks_in_lds(kind, cols, dtype):
    """Rows beyond a workgroup's registers whose next chunks wait in LDS, with chunks left for memory and without, and a row that ends
    just behind one; three passes over a row and two."""
    spec = (softmax_graph if kind == "softmax" else log_softmax_graph)(3, cols, dtype)
    inp = make_inputs(spec, seed=cols)
    ref = O.evaluate(spec, inp)
    kernels = [c["kernel"] for c in B.Plan(B.Graph.from_spec(spec), "auto").candidates()]
    assert any(",lds" in k for k in kernels), kernels
    note(f"{spec.name}: worst {all_candidates(spec, inp, ref, floors_for(spec, inp, ref), repeat=2, unfused=False)}")


def test_chunks_in_lds_of_several_operands():
    """Two row operands and column vectors: the sum of input and residual, plus a bias, normalised."""
    from workloads import add_bias_layernorm_graph
    spec = add_bias_layernorm_graph(2, 70000, in_dtype="f32", out_dtype="bf16")
    inp = make_inputs(spec, seed=1)
    ref = O.evaluate(spec, inp)
    kernels = [c["kernel"] for c in B.Plan(B.Graph.from_spec(spec), "auto").candidates()]
    assert any(",lds" in k for k in kernels), kernels
    note(f"{spec.name}: worst {all_candidates(spec, inp, ref, floors_for(spec, inp, ref), repeat=2, unfused=False)}")
