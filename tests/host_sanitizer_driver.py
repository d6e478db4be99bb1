"""Run as a child process by tests/test_host_sanitizers.py with the sanitizer build of the host core loaded
(FUSION_STITCHING_LIB) and the sanitizer runtime preloaded.  Plans and "executes" the benchmark configurations, the
generic patterns, packs and explored programs through the host stub: every launch is checked (its arguments are taken apart
again as the kernel does it) and counted, none runs, no device pointer is dereferenced.  Any AddressSanitizer /
UndefinedBehaviorSanitizer report aborts the process."""
import ctypes
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

from paper_2009_10924_amd import binding as B                                            # noqa: E402
from workloads import (EXPLORE_CONFIGS, FULL_CONFIGS, GENERIC_CONFIGS, NEXT_CONFIGS, PACK_CONFIGS, bias_gelu_dbias_graph,  # noqa: E402
                       gelu_backward_graph, independent_tiny_patterns_graph, layernorm_backward_bias_graph, layernorm_backward_graph,
                       random_multi_pattern, random_row_pattern, transpose_graph)
from tests.gpu_util import side_by_side                                                  # noqa: E402


def fake(n, base):
    return [base * (i + 1) for i in range(n)]


def run_plan(spec, scheme="auto", **opts):
    plan = B.Plan(B.Graph.from_spec(spec), scheme, **opts)
    ws = plan.info["workspace_bytes"]
    plan.execute_ptrs(fake(len(spec.inputs), 0x10000), fake(len(spec.outputs), 0x1000000), 0x40000000 if ws else 0, ws, 0)
    if 0 < ws <= B.FS_STATIC_SCRATCH_BYTES:
        plan.execute_static_ptrs(fake(len(spec.inputs), 0x10000), fake(len(spec.outputs), 0x1000000), 0)
    plan.describe()
    plan.source()
    return plan


def run_program(spec, **opts):
    prog = B.Program(B.Graph.from_spec(spec), **opts)
    ws = prog.info["workspace_bytes"]
    ins, outs = fake(len(spec.inputs), 0x10000), fake(len(spec.outputs), 0x1000000)
    prog.bind(ins, outs, 0x40000000, ws, 0)()
    for stage in range(prog.info["n_stages"]):
        prog.bind_stage(stage, ins, outs, 0x40000000, ws, 0)()
    prog.describe()
    prog.patterns()
    return prog


def launches_of(lib, call):
    before = lib.fs_stub_launch_count()
    call()
    return lib.fs_stub_launch_count() - before


def one_launch_forms(lib):
    """A small pattern with column sums runs as one launch wherever its kernel can be loaded, also if the plan was made without a device;
    under capture before that, and where an output shares memory with anything, as two."""
    for spec in (layernorm_backward_graph(64, 768, "bf16"), bias_gelu_dbias_graph(64, 768, "bf16")):
        n_in, n_out = len(spec.inputs), len(spec.outputs)
        ins = fake(n_in, 0x100000)
        outs = [0x40000000 + 0x100000 * i for i in range(n_out)]
        lib.fs_stub_state(0, 0)
        plan = B.Plan(B.Graph.from_spec(spec), "auto")
        ws = plan.info["workspace_bytes"]
        assert "at_once " in plan.describe()
        run = lambda i=ins, o=outs: launches_of(lib, lambda: plan.execute_ptrs(i, o, 0x70000000, ws, 0))  # noqa: E731
        lib.fs_stub_state(1, 1)
        assert run() == 2                      # captured before anything could load the kernel
        lib.fs_stub_state(1, 0)
        assert run() == 1 and launches_of(lib, lambda: plan.execute_static_ptrs(ins, outs, 0)) == 1
        lib.fs_stub_state(1, 1)
        assert run() == 1                      # loaded by now
        lib.fs_stub_state(1, 0)
        size = 64 * 768 * 2
        big = [k for k, t in enumerate(spec.inputs) if tuple(t.dims) == (64, 768)][0]
        for at, launches in ((0, 2), (16, 2), (size - 16, 2), (size, 1), (16 - size, 2), (-size, 1)):
            assert run(o=[ins[big] + at] + outs[1:]) == launches, at   # over an input, into it from either side, beside it
        assert run(o=[outs[0], outs[0] + size - 16] + outs[2:]) == 2 and run(o=[outs[0], outs[0] + size] + outs[2:]) == 1


def merged_launches(lib):
    """Two lone transposes run as one launch wherever its kernel can be loaded; captured before that, in the two kernels that are compiled
    in.  A result that lies in another's buffer, or over an input, sends the run step by step."""
    spec = side_by_side([transpose_graph((64, 128, 12, 64), (0, 2, 1, 3), "bf16"), transpose_graph((64, 256, 12, 64), (0, 2, 1, 3), "f32")])
    lib.fs_stub_state(0, 0)
    prog = B.Program(B.Graph.from_spec(spec))
    assert "merged 0 of 1 steps=0,1 " in prog.describe() and prog.info["n_kernels"] == 2
    ins, outs = [0x10000000, 0x20000000], [0x40000000, 0x50000000]
    run = lambda o=outs: launches_of(lib, prog.bind(ins, o, 0x70000000, prog.info["workspace_bytes"], 0))  # noqa: E731
    lib.fs_stub_state(1, 1)
    assert run() == 2
    lib.fs_stub_state(1, 0)
    assert run() == 1
    lib.fs_stub_state(1, 1)
    assert run() == 1
    lib.fs_stub_state(1, 0)
    assert run([ins[1], outs[1]]) == 2 and run([outs[0], outs[0] + 64]) == 2


def main():
    lib = B.load()
    lib.fs_stub_launch_count.restype = ctypes.c_long
    assert "host_san" in B.lib_path()
    assert lib.fs_stub_check_argument_words() == 0      # every field of the kernels' argument words, at its limits and beyond
    for compile_ok in ("", "1"):
        if compile_ok:
            os.environ["FS_STUB_COMPILE_OK"] = "1"      # generated kernels "compile": the generator's whole path runs
            one_launch_forms(lib)
            merged_launches(lib)
        for name, make in list(FULL_CONFIGS.items()) + list(NEXT_CONFIGS.items()) + list(GENERIC_CONFIGS.items()):
            spec = make()
            plan = run_plan(spec)
            n = plan.info["n_candidates"]
            for i in range(n):                          # every enumerated launch shape
                try:
                    run_plan(spec, candidate=i)
                except B.FsError as e:
                    assert e.code == -5, (name, i, e)   # a generated candidate that did not "compile"
            run_plan(spec, "unfused")
        for dims, perm in (((64, 197, 768), (0, 2, 1)), ((4096, 4096), (1, 0)), ((5, 24, 20, 40), (0, 3, 2, 1)), ((9, 136, 12, 200), (0, 2, 3, 1)),
                           ((3, 77, 5, 131), (0, 3, 2, 1)), ((700, 3000), (1, 0)), ((2048, 512), (1, 0))):
            for dt in ("bf16", "f32"):
                run_plan(transpose_graph(dims, perm, dt))
        for r, c, dt in ((64, 128, "f32"), (37, 96, "bf16"), (300, 1001, "f16")):
            run_plan(gelu_backward_graph(r, c - c % 8 if dt != "f32" else c - c % 4, dt))
            run_plan(layernorm_backward_bias_graph(r, 96, dt, sum_dtype="f32"))
        for seed in range(12):
            run_plan(random_row_pattern(seed, 33, 136, ("f32", "f16", "bf16")[seed % 3], n_ops=6 + seed, column_sums=seed % 3))
        members = PACK_CONFIGS["P1"]()
        pack = B.Pack([B.Plan(B.Graph.from_spec(m), "auto") for m in members])
        pack.bind(fake(sum(len(m.inputs) for m in members), 0x10000), fake(sum(len(m.outputs) for m in members), 0x1000000), 0)()
        for name in ("T1", "T2", "T3"):
            spec = EXPLORE_CONFIGS[name]()
            for opts in ({}, {"no_joint_folds": True}, {"no_packing": True, "no_remote_fusion": True}, {"top_k": 1, "beam_width": 1}):
                run_program(spec, **opts)
        run_program(independent_tiny_patterns_graph())
        for seed in range(6):
            run_program(random_multi_pattern(seed, rows=64, cols=128, segments=2 + seed % 3, column_sums=seed % 2, external_links=seed % 2 == 1))
    # error paths must leave nothing behind either
    g = B.Graph.from_spec(FULL_CONFIGS["C4"]())
    for bad in (lambda: B.Plan(g, "lds"), lambda: B.Plan(g, "auto", candidate=999), lambda: run_plan(FULL_CONFIGS["C4"](), "auto", block_threads=96)):
        try:
            bad()
        except B.FsError:
            pass
    launches = lib.fs_stub_launch_count()
    assert launches > 1000, launches
    print(f"host sanitizer driver: {launches} checked launches, no report")


if __name__ == "__main__":
    main()
