"""Host-side checks of the C ABI that need no GPU: the library loads, exports every symbol
the header declares, validates problems and rejects bad arguments before any launch."""
import ctypes
import subprocess
import sys
import re

import pytest

import paper_2508_17756_amd as sg
from synthetic import CONFIGS


def test_library_exports_every_declared_symbol(repo_root):
    header = open(f"{repo_root}/include/supergen_tile.h").read()
    header = re.sub(r"/\*.*?\*/", "", header, flags=re.S)
    names = set(re.findall(r"\b(sg_[a-z_]+)\s*\(", header))
    assert {"sg_tile_attention", "sg_tile_blend", "sg_cache_gate", "sg_denoise_step_tiled"} <= names
    lib = sg.load_library()
    for n in names:
        assert hasattr(lib, n), n
    assert sg.sg_version() == "0.1"
    assert sg.sg_status_string(sg.SG_ERR_WORKSPACE).startswith("workspace")


def test_struct_layout_matches_header():
    assert ctypes.sizeof(sg.sg_problem) == 13 * 4 + 4 + 16 + 8  # 13 int32/float + padding + 2 int64 + 2 int32
    assert sg.sg_problem.grid_stride_token.offset == 56 and sg.sg_problem.shift_h.offset == 72


@pytest.mark.parametrize("name", list(CONFIGS))
def test_benchmark_configs_validate(name):
    assert sg.sg_problem_validate(sg.make_problem(CONFIGS[name])) == sg.SG_OK


@pytest.mark.parametrize("field,value,status", [
    ("T", 0, sg.SG_ERR_INVALID_ARG), ("tile_h", 11, sg.SG_ERR_INVALID_ARG),       # tiles no longer cover H
    ("stride_w", 11, sg.SG_ERR_INVALID_ARG),                                       # gap between tiles
    ("dtype", 5, sg.SG_ERR_INVALID_ARG), ("scale", float("nan"), sg.SG_ERR_INVALID_ARG),
    ("scale", 0.0, sg.SG_ERR_INVALID_ARG), ("grid_stride_token", 60, sg.SG_ERR_INVALID_ARG),
    ("head_dim", 96, sg.SG_ERR_UNSUPPORTED),
    ("shift_h", 16, sg.SG_ERR_INVALID_ARG), ("shift_w", -1, sg.SG_ERR_INVALID_ARG),
])
def test_invalid_problems(field, value, status):
    p = sg.make_problem(CONFIGS["tiny_f32"])
    setattr(p, field, value)
    if field == "head_dim":
        p.grid_stride_token = 96
    assert sg.sg_problem_validate(p) == status


def test_tile_count_limit():
    from synthetic import TileGeometry
    ok = TileGeometry("m", 1, 17, 17, 2, 2, 1, 1, 16, 16, 1, 64, "f32", 0)
    assert sg.sg_problem_validate(sg.make_problem(ok)) == sg.SG_OK                      # 256 tiles
    over = TileGeometry("m", 1, 18, 17, 2, 2, 1, 1, 17, 16, 1, 64, "f32", 0)
    assert sg.sg_problem_validate(sg.make_problem(over)) == sg.SG_ERR_UNSUPPORTED       # 272 tiles


def test_null_and_workspace_checks_need_no_gpu():
    lib = sg.load_library()
    p = sg.make_problem(CONFIGS["tiny_f32"])
    assert sg.sg_problem_validate(p) == 0
    assert lib.sg_problem_validate(None) == sg.SG_ERR_INVALID_ARG
    assert lib.sg_tile_attention(ctypes.byref(p), None, None, None, 0, 0, None, None) == sg.SG_ERR_INVALID_ARG
    assert lib.sg_tile_attention(ctypes.byref(p), 16, 16, 16, 0, 5, 16, None) == sg.SG_ERR_INVALID_ARG
    assert lib.sg_tile_attention(ctypes.byref(p), 16, 16, 8, 0, 0, 16, None) == sg.SG_ERR_INVALID_ARG   # misaligned
    assert lib.sg_tile_blend(ctypes.byref(p), None, None, None) == sg.SG_ERR_INVALID_ARG
    arr = (ctypes.c_void_p * 2)(256, 512)
    assert lib.sg_cache_gate(arr, arr, 256, 2, 64, sg.SG_BF16, 0.05, 256, 256, None, 0, None) == sg.SG_ERR_WORKSPACE
    assert lib.sg_cache_gate(arr, arr, 256, 2, 64, sg.SG_BF16, 0.05, 256, 256, 256, 16, None) == sg.SG_ERR_WORKSPACE
    assert lib.sg_cache_gate(arr, arr, 256, -1, 64, sg.SG_BF16, 0.05, 256, 256, 256, 1 << 20, None) == sg.SG_ERR_INVALID_ARG
    assert lib.sg_cache_gate(arr, arr, 256, 2, 64, 9, 0.05, 256, 256, 256, 1 << 20, None) == sg.SG_ERR_INVALID_ARG
    assert lib.sg_denoise_step_tiled(ctypes.byref(p), None, None) == sg.SG_ERR_INVALID_ARG
    assert sg.sg_workspace_bytes(20) >= 20 * 2 * 8
    # gain / path-length policy entry points
    st = sg.sg_gain_state()
    st.has_prev = st.has_gain = st.gain = st.path_len = 256
    assert lib.sg_gain_gate(arr, arr, None, 2, 64, sg.SG_BF16, 0.05, None, 256, 256, 256, 256, 1 << 20, None) == sg.SG_ERR_INVALID_ARG
    assert lib.sg_gain_gate(arr, arr, ctypes.byref(st), 2, 64, sg.SG_BF16, 0.05, None, 256, 256, 256, None, 0, None) == sg.SG_ERR_WORKSPACE
    assert lib.sg_gain_gate(arr, arr, ctypes.byref(st), 2, 64, sg.SG_BF16, float("nan"), None, 256, 256, 256, 256, 1 << 20, None) == sg.SG_ERR_INVALID_ARG
    assert lib.sg_gain_gate(arr, arr, ctypes.byref(st), 0, 64, sg.SG_BF16, 0.05, None, None, None, None, None, 0, None) == sg.SG_OK
    assert lib.sg_gain_refresh(arr, arr, arr, arr, 256, 256, ctypes.byref(st), 2, 63, sg.SG_BF16, 256, 1 << 20, None) == sg.SG_ERR_INVALID_ARG   # not a multiple of 8
    assert lib.sg_gain_refresh(arr, arr, arr, None, 256, 256, ctypes.byref(st), 2, 64, sg.SG_BF16, 256, 1 << 20, None) == sg.SG_ERR_INVALID_ARG
    assert lib.sg_gain_refresh(arr, arr, arr, arr, 256, 256, ctypes.byref(st), 2, 64, sg.SG_BF16, 256, 16, None) == sg.SG_ERR_WORKSPACE
    assert lib.sg_denoise_step_gain(ctypes.byref(p), None, None) == sg.SG_ERR_INVALID_ARG
    assert lib.sg_tile_similarity(arr, arr, 2, 64, sg.SG_BF16, 256, None, 256, 1 << 20, None) == sg.SG_ERR_INVALID_ARG
    assert lib.sg_tile_similarity(arr, arr, 2, 64, sg.SG_BF16, 256, 256, 256, 16, None) == sg.SG_ERR_WORKSPACE
    assert lib.sg_tile_similarity(None, None, 0, 64, sg.SG_BF16, None, None, None, 0, None) == sg.SG_OK
    # shifted partitions
    ps = sg.make_problem(CONFIGS["tiny_f32"], shift=(3, 5))
    assert sg.sg_problem_validate(ps) == sg.SG_OK
    assert lib.sg_tile_attention(ctypes.byref(ps), 16, 16, 16, 2, 0, 16, None) == sg.SG_ERR_INVALID_ARG
    assert lib.sg_tile_slice(ctypes.byref(ps), arr, 4, 0, 0, 256, None) == sg.SG_ERR_INVALID_ARG
    assert lib.sg_tile_slice(ctypes.byref(ps), arr, 2, 2, 0, 256, None) == sg.SG_ERR_INVALID_ARG
    assert lib.sg_tile_blend_update(ctypes.byref(ps), arr, None, 1.0, 0.1, 256, None) == sg.SG_ERR_INVALID_ARG
    assert lib.sg_tile_blend_update(ctypes.byref(ps), arr, 256, float("nan"), 0.1, 256, None) == sg.SG_ERR_INVALID_ARG


def test_canvas_refine_step_wants_its_own_tile_buffers():
    lib = sg.load_library()
    p = sg.make_problem(CONFIGS["tiny_f32"])            # 4 tiles
    mine = (ctypes.c_void_p * 4)(256, 512, 768, 1024)
    other = (ctypes.c_void_p * 4)(256, 512, 768, 2048)
    io = sg.sg_gain_step_io()
    io.tile_x = other
    assert lib.sg_refine_step_canvas(ctypes.byref(p), 16, 16, 16, mine, ctypes.byref(io), None, None, None) == sg.SG_ERR_INVALID_ARG
    io.tile_x = mine    # the same buffers, but the step's own arguments are incomplete
    assert lib.sg_refine_step_canvas(ctypes.byref(p), 16, 16, 16, mine, ctypes.byref(io), None, None, None) == sg.SG_ERR_INVALID_ARG
    assert lib.sg_refine_step_canvas(ctypes.byref(p), None, 16, 16, mine, ctypes.byref(io), None, None, None) == sg.SG_ERR_INVALID_ARG
    assert lib.sg_refine_step_canvas(ctypes.byref(p), 16, 16, 16, None, ctypes.byref(io), None, None, None) == sg.SG_ERR_INVALID_ARG


def test_plain_c_client_compiles_links_and_agrees_on_layout(repo_root, tmp_path):
    """The header is C: a C99 translation unit with -pedantic -Werror includes it, links against the
    library and calls the host-only entry points; the sizes the C compiler derives are the binding's."""
    import os
    import shutil
    gcc = shutil.which("gcc")
    if gcc is None:
        pytest.skip("no C compiler")
    sg.load_library()
    libdir = f"{repo_root}/paper_2508_17756_amd"
    exe = str(tmp_path / "host_client")
    subprocess.run([gcc, "-std=c99", "-pedantic", "-Wall", "-Wextra", "-Werror", f"-I{repo_root}/include",
                    f"{repo_root}/tests/c_client/host_client.c", "-o", exe, f"-L{libdir}", "-lsupergen_tile",
                    f"-Wl,-rpath,{libdir}"], check=True, capture_output=True, text=True)
    env = dict(os.environ)
    run = subprocess.run([exe], check=True, capture_output=True, text=True, env=env, timeout=120)
    kv = dict(line.split("=", 1) for line in run.stdout.strip().splitlines())
    assert kv["version"] == sg.sg_version()
    assert int(kv["sizeof_problem"]) == ctypes.sizeof(sg.sg_problem)
    assert int(kv["offset_stride_token"]) == sg.sg_problem.grid_stride_token.offset
    assert int(kv["offset_shift_h"]) == sg.sg_problem.shift_h.offset
    assert int(kv["sizeof_step_io"]) == ctypes.sizeof(sg.sg_step_io)
    assert int(kv["sizeof_gain_state"]) == ctypes.sizeof(sg.sg_gain_state)
    assert int(kv["sizeof_gain_step_io"]) == ctypes.sizeof(sg.sg_gain_step_io)
    assert int(kv["sizeof_region_control"]) == ctypes.sizeof(sg.sg_region_control)
    assert int(kv["sizeof_scheduler_update"]) == ctypes.sizeof(sg.sg_scheduler_update)
    assert int(kv["validate"]) == sg.SG_OK and int(kv["validate_gap"]) == sg.SG_ERR_INVALID_ARG
    assert int(kv["workspace_status"]) == sg.SG_OK and int(kv["workspace_bytes"]) == sg.sg_workspace_bytes(20)
    assert int(kv["null_attention"]) == int(kv["null_blend"]) == int(kv["null_step"]) == sg.SG_ERR_INVALID_ARG
    assert kv["status_string"] == "invalid argument"
    assert (int(kv["shift_status"]), int(kv["shift_h"]), int(kv["shift_w"])) == (sg.SG_OK, 5, 5)


def test_bench_refuses_more_than_one_gpu(repo_root):
    """One GPU only: asking the benchmark for more ends with a message, before anything touches a device."""
    run = subprocess.run([sys.executable, f"{repo_root}/bench.py", "--gpus", "2"], capture_output=True, text=True, timeout=120)
    assert run.returncode != 0
    assert "one GPU" in (run.stdout + run.stderr)


def test_shift_schedule_follows_the_oracle_and_rejects_bad_arguments():
    """Algorithm 1 "ShiftThisStep" / "Shift" on the host: the C entry point against the oracle's schedule."""
    import oracle
    lib = sg.load_library()
    for name in ("canvas2k_bf16", "canvas4k_bf16", "tiny_f32"):
        g = CONFIGS[name]
        p = sg.make_problem(g)
        for loop, freq in ((16, 1), (16, 3), (7, 2), (1, 1)):
            for step in range(0, loop * freq + 5):
                dy, dx = sg.sg_shift_schedule(p, step, loop, freq)
                assert (dy, dx) == oracle.shift_schedule(step, g.tile_h, g.tile_w, loop, freq)
                q = sg.make_problem(g, shift=(dy, dx))
                assert lib.sg_problem_validate(ctypes.byref(q)) == sg.SG_OK      # a shift the other calls accept
    p = sg.make_problem(CONFIGS["tiny_f32"])
    dy, dx = ctypes.c_int32(-7), ctypes.c_int32(-7)
    for step, loop, freq in ((-1, 16, 1), (0, 0, 1), (0, 16, 0)):
        assert lib.sg_shift_schedule(ctypes.byref(p), step, loop, freq, ctypes.byref(dy), ctypes.byref(dx)) == sg.SG_ERR_INVALID_ARG
    assert lib.sg_shift_schedule(ctypes.byref(p), 0, 16, 1, None, ctypes.byref(dx)) == sg.SG_ERR_INVALID_ARG
    assert lib.sg_shift_schedule(None, 0, 16, 1, ctypes.byref(dy), ctypes.byref(dx)) == sg.SG_ERR_INVALID_ARG
    assert (dy.value, dx.value) == (-7, -7)                                       # nothing written on failure


def test_partition_tiles_follows_the_oracle_and_leaves_the_problem_alone_on_failure():
    """Algorithm 1 "PartitionTiles" on the host: the C entry point against the oracle, over the benchmark geometries
    and a sweep of small canvases, including every combination that has no exact partition."""
    import oracle
    lib = sg.load_library()
    for g in CONFIGS.values():
        p = sg.make_problem(g)
        want = (p.n_tile_rows, p.n_tile_cols, p.stride_h, p.stride_w)
        p.n_tile_rows = p.n_tile_cols = p.stride_h = p.stride_w = p.tile_h = p.tile_w = 0
        sg.sg_partition_tiles(p, g.tile_h, g.tile_w, g.tile_h - g.stride_h if g.n_tile_rows > 1 else 0,
                              g.tile_w - g.stride_w if g.n_tile_cols > 1 else 0)
        got = (p.n_tile_rows, p.n_tile_cols, p.stride_h, p.stride_w)
        if g.n_tile_rows > 1 and g.n_tile_cols > 1:
            assert got == want
        assert lib.sg_problem_validate(ctypes.byref(p)) == sg.SG_OK
    p = sg.make_problem(CONFIGS["tiny_f32"])
    for H in (7, 12, 16):
        for th in range(0, H + 2):
            for oh in range(-1, th + 1):
                p.H, p.W = H, 24
                before = bytes(p)
                st = lib.sg_partition_tiles(ctypes.byref(p), th, 8, oh, 0)
                try:
                    nr, nc, sh, sw = oracle.partition_tiles(H, 24, th, 8, oh, 0)
                except ValueError:
                    assert st == sg.SG_ERR_INVALID_ARG and bytes(p) == before, (H, th, oh)
                else:
                    assert st == sg.SG_OK and (p.n_tile_rows, p.n_tile_cols, p.stride_h, p.stride_w) == (nr, nc, sh, sw)
    p.H, p.W = 300, 300
    before = bytes(p)
    assert lib.sg_partition_tiles(ctypes.byref(p), 10, 10, 0, 0) == sg.SG_ERR_UNSUPPORTED and bytes(p) == before   # 900 tiles
    assert lib.sg_partition_tiles(None, 10, 10, 0, 0) == sg.SG_ERR_INVALID_ARG


def test_stream_handle_without_the_raw_getters():
    """The binding asks torch for the raw stream of the current device; a torch that lacks those private functions still gives it."""
    from types import SimpleNamespace as NS
    from paper_2508_17756_amd.binding import _stream_getter
    started = []
    cuda = NS(is_initialized=lambda: bool(started), init=lambda: started.append(1),
              current_stream=lambda: NS(cuda_stream=77))
    raw = NS(_cuda_getCurrentRawStream=lambda device: 100 + device, _cuda_getDevice=lambda: 3)
    assert _stream_getter(NS(cuda=cuda, _C=raw))() == 103 and started == [1]
    assert _stream_getter(NS(cuda=cuda, _C=NS()))() == 77
    assert _stream_getter(NS(cuda=cuda, _C=NS(_cuda_getDevice=lambda: 3)))() == 77
