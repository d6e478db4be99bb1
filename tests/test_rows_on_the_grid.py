"""Which generated kernels read and write rows of an odd number of 16-bit elements on the tensor's grid of whole steps (the times that
decide stand at the rule, row_on_grid in fs_codegen.cpp)."""
import pytest

from paper_2009_10924_amd import binding as B
from workloads import attention_scores_graph, masked_scores_gate_graph, softmax_graph

pytestmark = pytest.mark.skipif(not B.codegen_available(), reason="the HIP run-time compiler is not installed here")


def _on_grid(spec, block):
    """Of the generated candidates with a workgroup per row (or a group of lanes): how many, and how many of them on the grid."""
    graph = B.Graph.from_spec(spec)
    some = grid = 0
    for c in B.Plan(graph, "auto").candidates():
        if not c["kernel"].startswith("row_generated") or (c["lanes_per_row"] > 64) != block:
            continue
        source = B.Plan(graph, "auto", candidate=c["candidate"]).source()
        some += 1
        grid += "EDGE_FIRST" in source
    return some, grid


@pytest.mark.parametrize("spec,lanes,block", [
    (attention_scores_graph(2, 2, 5, 333, dtype="f16"), True, True),       # one exponential, a stretched mask
    (masked_scores_gate_graph(2, 2, 5, 333, "f16"), False, True),          # a tanh before it
    (softmax_graph(5, 333, "bf16"), False, True),                          # no stretched operand
    (attention_scores_graph(2, 2, 5, 334, dtype="f16"), False, False),     # an even number
    (attention_scores_graph(2, 2, 5, 333, dtype="f32"), False, False)], ids=lambda v: v.name if hasattr(v, "name") else str(v))
def test_rows_on_the_grid(spec, lanes, block):
    some, grid = _on_grid(spec, block=False)
    assert some > 0 and (grid > 0) == lanes
    some, grid = _on_grid(spec, block=True)
    assert (grid > 0) == (block and some > 0)
