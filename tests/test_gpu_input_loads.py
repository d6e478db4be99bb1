"""Row inputs are read through the caches up to 96 MiB of inputs and past them (with the streaming hint) above: the chosen
kernel of every family on the last sizes of the one form and the first of the other, and every hand-written candidate in the
form for large inputs (test_gpu_kernel_arguments.py runs them on small ones).  The plan's listing says which form a launch has.
Every output element is compared with the float64 oracle (inputs repeat a seeded block of rows), transposed bits exactly."""
import pytest

from paper_2009_10924_amd import binding as B
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
@pytest.mark.parametrize("dims,perm,dtype", [((197, 768), (0, 2, 1), "bf16"), ((128, 12, 64), (0, 2, 3, 1), "f32"), ((24, 20), (0, 2, 1), "f16"),
                                             ((24, 20, 40), (0, 3, 2, 1), "f16"), ((20, 6, 28), (0, 3, 2, 1), "f32"),
                                             ((136, 12, 200), (0, 3, 2, 1), "bf16"), ((77, 5, 131), (0, 3, 2, 1), "f32")])
def test_transposes_on_both_sides_of_the_input_size_rule(dims, perm, dtype, side):
    import torch
    size = 4 if dtype == "f32" else 2
    per_batch = size * int(torch.tensor(dims).prod())
    n = LIMIT // per_batch + (0 if side == "through the caches" else 1)
    kind = torch.int32 if size == 4 else torch.int16
    x = torch.arange(n * per_batch // size, dtype=torch.int32, device="cuda").mul_(40503).to(kind).view(n, *dims)
    want = x.permute(perm).contiguous()
    out = torch.zeros_like(want)
    plan = B.Plan(B.Graph.from_spec(transpose_graph((n,) + dims, perm, dtype)), "auto")
    note(f"  {(n,) + dims} {perm} {dtype}, {side}: {plan.info['kernel']}")
    assert ("\n  loads cached\n" if side == "through the caches" else "\n  loads streamed\n") in plan.describe()
    plan.execute_ptrs([x.data_ptr()], [out.data_ptr()], 0, 0, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert torch.equal(out, want)


@pytest.mark.parametrize("side", ["through the caches", "past the caches"])
@pytest.mark.parametrize("kind", sorted(KINDS))
def test_both_sides_of_the_input_size_rule(kind, side):
    make, row_bytes, period = KINDS[kind]
    n = (LIMIT - 65536) // row_bytes if side == "through the caches" else LIMIT // row_bytes + 1
    listing = B.Plan(B.Graph.from_spec(make(n)), "auto").describe()
    assert ("\n  loads cached\n" if side == "through the caches" else "\n  loads streamed\n") in listing, listing
    errs, info = _run_rows(make, n, period)
    note(f"{kind}, {n} rows, {side}: {info['kernel']} worst {errs}")


# shapes with candidates of every hand-written form: lane groups and whole workgroups, with and without masks and statistics, the
# head split through LDS and without
WIDE = {
    "softmax": (lambda k: softmax_graph(k, 1024, "f32"), 4096, 32),
    "masked scores": (lambda k: attention_scores_graph(k, 2, 8, 1024, dtype="f32"), 2 * 8 * 4096 + 4096, 2),
    "layernorm": (lambda k: add_bias_layernorm_graph(k, 1024, in_dtype="bf16", out_dtype="bf16"), 4096, 64),
    "layernorm, wide": (lambda k: add_bias_layernorm_graph(k, 1536), 12288, 32),
    "layernorm with statistics": (lambda k: layernorm_stats_graph(k, 1536), 12288, 32),
    "layernorm backward": (lambda k: layernorm_backward_graph(k, 768, "f16"), 3080, 64),
    "softmax backward": (lambda k: softmax_backward_graph(k, 1024, "f32"), 8192, 32),
    "rms norm": (lambda k: rmsnorm_graph(k, 1024), 2048, 64),
    "bias and gelu": (lambda k: bias_gelu_graph(k, 520), 1040, 64),
    "bias and gelu with bias gradient": (lambda k: bias_gelu_dbias_graph(k, 1032), 4128, 64),
    "transpose chain": (lambda k: transpose_chain_graph(k, 96, 6, 64, dtype="bf16"), 96 * 6 * 64 * 2, 2),
}


@pytest.mark.parametrize("kind", sorted(WIDE))
def test_every_hand_written_candidate_past_the_caches(kind):
    make, row_bytes, period = WIDE[kind]
    n = LIMIT // row_bytes + 1
    graph, seen = B.Graph.from_spec(make(n)), set()
    with B.codegen(False):
        for i in range(B.Plan(graph, "auto").info["n_candidates"]):
            plan = B.Plan(graph, "auto", candidate=i)
            listing = plan.describe()
            if "  loads " not in listing:   # the interpreter has one form
                continue
            assert "\n  loads streamed\n" in listing and "cached" not in listing
            seen.add(plan.info["kernel"].split("<")[0])
            _run_rows(make, n, period, candidate=i)
    note(f"{kind}, {n} rows: {sorted(seen)}")
    if kind.startswith(("softmax", "masked", "layernorm", "rms")) and kind != "layernorm backward":
        assert len(seen) == 2, seen     # lane groups and workgroups
    if kind == "transpose chain":
        assert seen == {"tchain_wave", "tchain_lds"}, seen
