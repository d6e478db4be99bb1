"""Bias + GELU with the bias gradient on ragged shapes whose workgroups walk several row tiles: rows that end inside a tile and
rows that fill it, a last column tile whose surplus lanes repeat its last columns, every dtype (16-bit shapes walk without tests
around their stores, float32 ones with them) and every candidate, against the float64 oracle (inputs repeat a seeded block)."""
import pytest

from paper_2009_10924_amd import binding as B
from tests.gpu_util import note
from tests.test_gpu_max_size import _run_rows
from workloads import bias_gelu_dbias_graph

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,rows,cols", [("f32", 3001, 12292), ("f32", 3072, 12292), ("f32", 3001, 12288), ("f16", 6003, 12296), ("bf16", 6003, 12296),
                                             ("bf16", 6144, 12296), ("f16", 6003, 12288)])
def test_every_candidate_over_several_row_tiles(dtype, rows, cols):
    graph = B.Graph.from_spec(bias_gelu_dbias_graph(rows, cols, dtype))
    col_tiles, rounds = -(-cols // (256 if dtype == "f32" else 512)), []
    with B.codegen(False):
        for i in range(B.Plan(graph, "auto").info["n_candidates"]):
            info = B.Plan(graph, "auto", candidate=i).info
            if not info["kernel"].startswith("bias_gelu_dbias<"):
                continue
            rounds.append(-(-rows // (info["rows_per_block"] * (info["grid"][0] // col_tiles))))
            errs, _ = _run_rows(lambda k: bias_gelu_dbias_graph(k, cols, dtype), rows, 64, candidate=i)
            note(f"{dtype} {rows} x {cols} {info['kernel']}: {rounds[-1]} row tiles per workgroup, worst {errs}")
    assert len(rounds) == 8 and min(rounds) >= 3, rounds
