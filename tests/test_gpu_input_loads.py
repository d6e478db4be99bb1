"""Row inputs are read through the caches up to 96 MiB of inputs and past them (with the streaming hint) above: every kernel
that exists in both forms, on the last sizes of the one and the first of the other.  Every output element is compared with
the float64 oracle (inputs repeat a seeded block of rows), transposed bits exactly."""
import pytest

from tests.gpu_util import note
from tests.test_gpu_max_size import _run_rows
from workloads import (add_bias_layernorm_graph, attention_scores_graph, bias_gelu_dbias_graph, bias_gelu_graph, layernorm_backward_graph,
                       layernorm_stats_graph, log_softmax_graph, rmsnorm_backward_graph, rmsnorm_graph, softmax_backward_graph,
                       softmax_graph, transpose_chain_graph, transpose_graph)

pytestmark = pytest.mark.gpu

LIMIT = 96 << 20   # bytes of inputs

# descriptor of k rows (or batch entries), bytes of row inputs per row, rows of the repeated block
KINDS = {
    "softmax, wavefront rows": (lambda k: softmax_graph(k, 1024, "f16"), 2048, 64),
    "softmax, workgroup rows": (lambda k: softmax_graph(k, 3864, "f32"), 15456, 32),
    "masked scores": (lambda k: attention_scores_graph(k, 4, 64, 128), 4 * 64 * 256 + 256, 2),
    "layernorm": (lambda k: add_bias_layernorm_graph(k, 768), 6144, 64),
    "layernorm with statistics": (lambda k: layernorm_stats_graph(k, 1024), 8192, 64),
    "layernorm backward": (lambda k: layernorm_backward_graph(k, 768, "f32"), 6152, 64),
    "layernorm backward, 16 bits": (lambda k: layernorm_backward_graph(k, 1024, "bf16"), 4104, 64),
    "rms norm": (lambda k: rmsnorm_graph(k, 4096), 8192, 64),
    "rms norm, odd width": (lambda k: rmsnorm_graph(k, 523, dtype="f16"), 1046, 64),
    "rms norm backward": (lambda k: rmsnorm_backward_graph(k, 1024, "bf16"), 4100, 64),
    "softmax backward": (lambda k: softmax_backward_graph(k, 512, "bf16"), 2048, 64),
    "bias and gelu": (lambda k: bias_gelu_graph(k, 3072), 6144, 64),
    "bias and gelu with bias gradient": (lambda k: bias_gelu_dbias_graph(k, 1024), 4096, 64),
    "kept chunks": (lambda k: log_softmax_graph(k, 50257, "bf16"), 100514, 8),
    "transpose chain": (lambda k: transpose_chain_graph(k, 64, 12, 64), 64 * 12 * 64 * 4, 2),
}


@pytest.mark.parametrize("side", ["through the caches", "past the caches"])
@pytest.mark.parametrize("dims,perm,dtype", [((197, 768), (0, 2, 1), "bf16"), ((128, 12, 64), (0, 2, 3, 1), "f32"), ((24, 20), (0, 2, 1), "f16")])
def test_transposes_on_both_sides_of_the_input_size_rule(dims, perm, dtype, side):
    import torch
    from paper_2009_10924_amd import binding as B
    size = 4 if dtype == "f32" else 2
    per_batch = size * int(torch.tensor(dims).prod())
    n = LIMIT // per_batch + (0 if side == "through the caches" else 1)
    kind = torch.int32 if size == 4 else torch.int16
    x = torch.arange(n * per_batch // size, dtype=torch.int32, device="cuda").mul_(40503).to(kind).view(n, *dims)
    want = x.permute(perm).contiguous()
    out = torch.zeros_like(want)
    plan = B.Plan(B.Graph.from_spec(transpose_graph((n,) + dims, perm, dtype)), "auto")
    note(f"  {(n,) + dims} {perm} {dtype}, {side}: {plan.info['kernel']}")
    plan.execute_ptrs([x.data_ptr()], [out.data_ptr()], 0, 0, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert torch.equal(out, want)


@pytest.mark.parametrize("side", ["through the caches", "past the caches"])
@pytest.mark.parametrize("kind", sorted(KINDS))
def test_both_sides_of_the_input_size_rule(kind, side):
    make, row_bytes, period = KINDS[kind]
    n = (LIMIT - 65536) // row_bytes if side == "through the caches" else LIMIT // row_bytes + 1
    errs, info = _run_rows(make, n, period)
    note(f"{kind}, {n} rows, {side}: {info['kernel']} worst {errs}")
