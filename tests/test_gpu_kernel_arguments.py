"""The hand-written kernels take their shapes, flags and shifts packed into few argument words: every candidate of the
patterns whose words are filled to the edge -- the largest widths of a family and widths beyond a word's field (served by the
kernel for rows of any length), a mask with three leading axes, workgroup rows of 64 to 256 lanes, statistics, one head --
against the float64 oracle."""
import pytest

from oracle import oracle as O
from paper_2009_10924_amd import binding as B
from tests.gpu_util import check, floors_for, run_spec
from workloads import (add_bias_layernorm_graph, attention_scores_graph, bias_gelu_dbias_graph, bias_gelu_graph, layernorm_backward_graph,
                       layernorm_stats_graph, make_inputs, rmsnorm_graph, softmax_backward_graph, softmax_graph, transpose_chain_graph, transpose_graph)

pytestmark = pytest.mark.gpu

SPECS = [
    attention_scores_graph(2, 3, 7, 1024, dtype="f32"), attention_scores_graph(3, 2, 5, 197, dtype="f16"), attention_scores_graph(1, 1, 1, 64, dtype="bf16"),
    softmax_graph(3, 300001, "f32"), softmax_graph(5, 16384, "f16"), softmax_graph(1, 8, "bf16"),
    layernorm_stats_graph(9, 3072), layernorm_stats_graph(33, 64), add_bias_layernorm_graph(7, 4096, in_dtype="bf16", out_dtype="bf16"),
    add_bias_layernorm_graph(64, 768), layernorm_backward_graph(48, 3072, "bf16"), layernorm_backward_graph(41, 768, "f32"), layernorm_backward_graph(64, 64, "f16"),
    rmsnorm_graph(5, 8192), softmax_backward_graph(6, 4096, "f16"), bias_gelu_graph(3, 520), bias_gelu_dbias_graph(67, 1032, "bf16"),
    transpose_chain_graph(1, 7, 5, 256, dtype="f32"), transpose_chain_graph(2, 9, 1, 64, dtype="f16"), transpose_chain_graph(1, 1, 3, 8, dtype="bf16"),
    transpose_graph((3, 5, 7, 40), (2, 0, 1, 3), "f16"),
]


@pytest.mark.parametrize("spec", SPECS, ids=lambda s: s.name)
def test_every_hand_written_candidate(spec):
    inp = make_inputs(spec, seed=2)
    ref = O.evaluate(spec, inp)
    floors = floors_for(spec, inp, ref)
    with B.codegen(False):
        n = B.Plan(B.Graph.from_spec(spec), "auto").info["n_candidates"]
        for i in range(n):
            got, _, info, _ = run_spec(spec, inp, "auto", candidate=i)
            for name, dt in spec.outputs:
                check(got[name], ref[name].reshape(got[name].shape), dt, floors.get(name, 0.0), f"{spec.name} {info['kernel']}/{name}")
