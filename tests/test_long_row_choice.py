"""Rows beyond a workgroup's registers: where the chosen form keeps chunks in LDS too, and where it leaves them to the cache
(the times that decide stand at the rule, in fs_rowprog.cpp)."""
import pytest

from paper_2009_10924_amd import binding as B
from workloads import add_bias_layernorm_graph, log_softmax_graph, rmsnorm_graph, softmax_backward_graph, softmax_graph

pytestmark = pytest.mark.skipif(not B.codegen_available(), reason="the HIP run-time compiler is not installed here")


@pytest.mark.parametrize("spec,lds", [
    # a few chunks beyond the registers, many rows: the cache holds them
    (softmax_graph(500, 98304, "f32"), False), (softmax_graph(1500, 98304, "f32"), False), (rmsnorm_graph(500, 98304, dtype="f32"), False),
    (log_softmax_graph(4096, 128256, "bf16"), False),
    # LDS would hold as much as the registers
    (softmax_backward_graph(500, 98304, "bf16"), False), (softmax_backward_graph(1500, 49152, "bf16"), False),
    # many chunks, few rows, no register for more, a row that lies on the grid by it
    (log_softmax_graph(1500, 131072, "f32"), True), (softmax_graph(50, 122868, "f32"), True), (log_softmax_graph(300, 98304, "f32"), True),
    (add_bias_layernorm_graph(500, 70000, in_dtype="bf16", out_dtype="bf16"), True), (softmax_backward_graph(500, 131072, "f32"), True),
    (log_softmax_graph(1500, 128257, "bf16"), True)], ids=lambda v: v.name if hasattr(v, "name") else str(v))
def test_chunks_in_lds_only_where_they_pay(spec, lds):
    kernel = B.Plan(B.Graph.from_spec(spec), "auto").info["kernel"]
    assert "chunks" in kernel and (",lds" in kernel) == lds, kernel
