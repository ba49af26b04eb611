"""GPU parity at sizes the fp64 oracle finishes in seconds: every entry point of the C ABI
against the oracle, element by element, on seeded inputs spanning several blocks and ragged
tails."""
import math
from dataclasses import replace

import numpy as np
import pytest
import torch

import oracle
import paper_2508_17756_amd as sg
from synthetic import CONFIGS, TileGeometry, randn_tensor, torch_dtype, scaled_down, eps_table, perturb_
from gpu_util import (to_f64, errors, assert_close, canvas_qkv, gpu_tile_attention,
                      oracle_tile_attention_full, BF16_MAX_ABS, BF16_REL_L2)

pytestmark = pytest.mark.gpu


def _geom(name, T, H, W, th, tw, sh, sw, heads, d, dtype, seed):
    nr = (H - th) // sh + 1 if th < H else 1
    nc = (W - tw) // sw + 1 if tw < W else 1
    return TileGeometry(name, T, H, W, th, tw, sh, sw, nr, nc, heads, d, dtype, seed)


# ------------------------------------------------------------------ attention
def test_attention_tiny_f32_all_tiles():
    g = CONFIGS["tiny_f32"]
    q, k, v = canvas_qkv(g)
    for tr in range(g.n_tile_rows):
        for tc in range(g.n_tile_cols):
            got = gpu_tile_attention(g, q, k, v, tr, tc)
            assert_close(to_f64(got), oracle_tile_attention_full(g, q, k, v, tr, tc), "f32", f"tile {tr},{tc}")


@pytest.mark.parametrize("d", [64, 128])
def test_attention_f32_ragged(d):
    g = _geom("f32r", 2, 9, 11, 9, 11, 9, 11, 3, d, "f32", 11)      # N = 198: 4 workgroups, ragged
    q, k, v = canvas_qkv(g)
    assert_close(to_f64(gpu_tile_attention(g, q, k, v, 0, 0)), oracle_tile_attention_full(g, q, k, v, 0, 0), "f32")


@pytest.mark.parametrize("th,tw", [(1, 1), (3, 11), (7, 10), (3, 43), (8, 16), (13, 20)])
def test_attention_f32_key_split(th, tw):
    # N = 1, 33, 70, 129, 128, 260 tokens: the 4 wavefronts of a workgroup share the keys in chunks of 32,
    # so these leave wavefronts without any key, with a partial chunk, and with unequal chunk counts
    g = _geom("f32s", 1, th, tw, th, tw, th, tw, 2, 64, "f32", 300 + th * tw)
    q, k, v = canvas_qkv(g)
    assert_close(to_f64(gpu_tile_attention(g, q, k, v, 0, 0)), oracle_tile_attention_full(g, q, k, v, 0, 0), "f32")


@pytest.mark.parametrize("d,heads,th,tw", [(64, 9, 25, 40), (64, 9, 23, 43), (128, 3, 16, 17), (128, 1, 5, 51), (128, 1, 8, 32),
                                             (64, 32, 31, 33), (64, 32, 10, 103), (128, 16, 10, 103)])
@pytest.mark.parametrize("view", [False, True], ids=["packed", "wrapped"])
def test_attention_f32_growing_scores(d, heads, th, tw, view):
    """Scores that grow along the key axis, so that the softmax reference has to move past its slack in every share of the
    keys; 9 heads of about 1,000 tokens take 64 queries per workgroup (head_dim 64), those of 255, 256 and 272 32; 255, 256, 272, 989 and
    1,000 tokens end in partial and whole 32-key blocks; 16 and 32 heads of 1,023 and 1,030 tokens go to the kernel on the bf16
    instruction.  (Four shares of the keys: test_gpu_attention_routes.py.)  The logits reach 12: their rounding, a few times 12 * 2^-24,
    is the relative error of the probabilities (the bound below leaves a factor of three)."""
    g = _geom("f32g", 1, 2 * th, 2 * tw, th, tw, th, tw, heads, d, "f32", 900 + th) if view else _geom(
        "f32g", 1, th, tw, th, tw, th, tw, heads, d, "f32", 900 + th)
    shift = (th // 2, tw // 3) if view else (0, 0)
    tr, tc = (1, 1) if view else (0, 0)
    q, k, v = canvas_qkv(g)
    u = torch.nn.functional.normalize(randn_tensor((d,), "f32", 5).cuda(), dim=0)
    rise = torch.linspace(0.0, 1.0, g.H * g.W, device="cuda").reshape(1, 1, g.H, g.W, 1)
    q = 0.3 * q + 8.0 * u
    k = 0.3 * k + (12.0 * math.sqrt(d) / 8.0) * rise * u
    out = torch.empty(g.tile_shape, dtype=torch.float32, device="cuda")
    sg.sg_tile_attention(sg.make_problem(g, shift=shift), q, k, v, tr, tc, out)
    win = [oracle.slice_tile_shifted(to_f64(t), g, tr, tc, *shift).reshape(heads, -1, d) for t in (q, k, v)]
    ref = np.stack([oracle.attention(win[0][a], win[1][a], win[2][a], g.scale) for a in range(heads)]).reshape(g.tile_shape)
    assert errors(to_f64(out), ref)[1] <= 1e-5


@pytest.mark.parametrize("d", [64, 128])
def test_attention_f32_scores_near_the_largest_number(d):
    """One key whose scores reach 1e38: a query with a positive score attends to it alone, one with a negative score to the
    others; nothing overflows (the logits of the others are of order one)."""
    g = _geom("f32b", 1, 10, 20, 10, 20, 10, 20, 1, d, "f32", 61)
    q, k, v = canvas_qkv(g)
    k.view(-1, d)[77] = 0.0
    k.view(-1, d)[77, 5] = 3e38
    out = gpu_tile_attention(g, q, k, v, 0, 0)
    assert torch.isfinite(out).all()
    assert errors(to_f64(out), oracle_tile_attention_full(g, q, k, v, 0, 0))[1] <= 1e-5


BF16_CASES = [
    # name, T, H, W, th, tw, sh, sw, heads: packed tiles (linear addressing) and canvas views
    ("packed_n576", 3, 12, 16, 12, 16, 12, 16, 2),      # 576 = 2*256 + 64, 9 full key blocks
    ("packed_n429", 3, 11, 13, 11, 13, 11, 13, 2),      # ragged: 429 = 256 + 173 ; 6*64 + 45
    ("packed_n273", 3, 7, 13, 7, 13, 7, 13, 3),         # key tail 17 < 32: second half block all masked
    ("packed_n40", 1, 5, 8, 5, 8, 5, 8, 1),             # fewer keys than one block
    ("view_2x2", 3, 16, 22, 10, 14, 6, 8, 2),           # overlapping tiles read in place, N = 420
    ("view_3x3", 2, 20, 40, 12, 24, 4, 8, 2),           # N = 576, triple row coverage; tile width 24: scalar walk, several row wraps per stage
    ("view_w72", 2, 8, 136, 6, 72, 2, 64, 2),           # N = 864, tile width 72 >= one stage: scalar walk, at most one wrap per stage
    ("view_w8", 3, 40, 12, 32, 8, 8, 4, 1),             # N = 768, tile width 8: eight row wraps per stage, frame wraps
    ("view_w3", 7, 9, 5, 5, 3, 4, 2, 2),                # N = 105, tile width 3: narrower than a run of 8 tokens, which are looked up one by one
    ("view_w1", 9, 4, 3, 4, 1, 4, 1, 1),                # N = 36, tile width 1: every token is its own tile row
]


@pytest.mark.parametrize("case", BF16_CASES, ids=[c[0] for c in BF16_CASES])
def test_attention_bf16_small(case):
    name, T, H, W, th, tw, sh, sw, heads = case
    g = _geom(name, T, H, W, th, tw, sh, sw, heads, 128, "bf16", 21)
    q, k, v = canvas_qkv(g)
    for tr, tc in {(0, 0), (g.n_tile_rows - 1, g.n_tile_cols - 1), (g.n_tile_rows - 1, 0)}:
        got = gpu_tile_attention(g, q, k, v, tr, tc)
        ma, rl = assert_close(to_f64(got), oracle_tile_attention_full(g, q, k, v, tr, tc), "bf16", f"{name} {tr},{tc}")
        print(f"{name} tile({tr},{tc}) max_abs={ma:.2e} rel_l2={rl:.2e}")


@pytest.mark.parametrize("case", BF16_CASES, ids=[c[0] for c in BF16_CASES])
def test_attention_bf16_head_dim_64(case):
    """head_dim 64 (the head width of CogVideoX-1.5, Section 8 "Workloads") in bf16: the same cases, packed through
    the streaming kernel; in place up to 448 tokens through the register-staged one."""
    name, T, H, W, th, tw, sh, sw, heads = case
    g = _geom(name, T, H, W, th, tw, sh, sw, heads, 64, "bf16", 23)
    q, k, v = canvas_qkv(g)
    for tr, tc in {(0, 0), (g.n_tile_rows - 1, g.n_tile_cols - 1)}:
        got = gpu_tile_attention(g, q, k, v, tr, tc)
        assert_close(to_f64(got), oracle_tile_attention_full(g, q, k, v, tr, tc), "bf16", f"{name} {tr},{tc}")


@pytest.mark.parametrize("heads,th,tw", [(2, 16, 28), (2, 20, 23), (64, 14, 33), (65, 14, 33), (25, 24, 50), (26, 24, 50), (26, 25, 49),
                                         (32, 24, 40), (33, 24, 40), (33, 31, 31)])
def test_attention_bf16_head_dim_64_windows_around_the_kernels_sizes(heads, th, tw):
    """Windows of head_dim 64 on either side of the rule that picks the kernel: 448 and 460 tokens with few workgroups; 462 tokens with 128
    and 130 of them on 256 compute units, 960 with 128 and 132, 961 with 132; behind it 1,200 with 125 and 130, 1,225 with 130."""
    g = _geom("rule", 1, 2 * th, 2 * tw, th, tw, th, tw, heads, 64, "bf16", 29 + heads)
    q, k, v = canvas_qkv(g)
    out = gpu_tile_attention(g, q, k, v, 1, 0)
    for a in (0, heads - 1):
        win = [oracle.slice_tile(to_f64(t[a:a + 1]), g, 1, 0).reshape(-1, 64) for t in (q, k, v)]
        assert_close(to_f64(out[a]).reshape(-1, 64), oracle.attention(*win, g.scale), "bf16", a)


@pytest.mark.parametrize("shape", [(3, 20, 25), (2, 33, 37), (4, 16, 32)], ids=["n1500", "n2442", "n2048"])
def test_attention_bf16_head_dim_64_long_packed(shape):
    """Packed head_dim-64 tiles of many stages of the streaming kernel (128 keys, two keys per LDS slot): 11.7 and exactly 16 in
    its form for few stages, 19.1 in the one with a steady loop."""
    T, H, W = shape
    g = _geom("d64long", T, H, W, H, W, H, W, 2, 64, "bf16", 27)
    q, k, v = canvas_qkv(g)
    got = gpu_tile_attention(g, q, k, v, 0, 0)
    assert_close(to_f64(got), oracle_tile_attention_full(g, q, k, v, 0, 0), "bf16")


def test_step_bf16_head_dim_64():
    g = _geom("d64step", 2, 14, 20, 8, 12, 6, 8, 3, 64, "bf16", 25)
    q, k, v = canvas_qkv(g)
    outs = [torch.empty(g.tile_shape, dtype=torch.bfloat16, device="cuda") for _ in range(g.n_tiles)]
    canvas = torch.empty(g.grid_shape, dtype=torch.bfloat16, device="cuda")
    sg.sg_denoise_step_tiled(sg.make_problem(g), canvas, outs, q=q, k=k, v=v)
    ref = [oracle_tile_attention_full(g, q, k, v, tr, tc) for tr in range(g.n_tile_rows) for tc in range(g.n_tile_cols)]
    assert_close(to_f64(canvas), oracle.blend(ref, g), "bf16")


@pytest.mark.parametrize("dtype,d,tw", [("bf16", 128, 10), ("bf16", 128, 16), ("bf16", 64, 10), ("f32", 64, 10), ("f32", 128, 10)])
def test_attention_token_major_layout(dtype, d, tw):
    """[T][H][W][heads][d] canvas through the stride fields, every kernel (tile width 16: scalar walk)."""
    g = _geom("tokmaj", 2, 12, tw + 8, 8, tw, 4, 8, 3, d, dtype, 31)
    qkv_hm = canvas_qkv(g)
    qkv_tm = [t.permute(1, 2, 3, 0, 4).contiguous() for t in qkv_hm]
    out = torch.empty(g.tile_shape, dtype=torch_dtype(dtype), device="cuda")
    sg.sg_tile_attention(sg.make_problem(g, token_major=True), *qkv_tm, 1, 1, out)
    assert_close(to_f64(out), oracle_tile_attention_full(g, *qkv_hm, 1, 1), dtype)


def _strided(canvases, g, stride):
    """The canvases (one head) in one buffer, their tokens `stride` elements apart and side by side in every token."""
    buf = torch.empty(g.grid_tokens * stride, dtype=canvases[0].dtype, device="cuda")
    out = [buf[i * g.head_dim:] for i in range(3)]
    for o, t in zip(out, canvases):
        o.as_strided((g.grid_tokens, g.head_dim), (stride, 1)).copy_(t.reshape(g.grid_tokens, g.head_dim))
    return out


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("tw", [20, 24, 13], ids=["broken_runs", "unbroken_runs", "narrow"])
@pytest.mark.parametrize("shift", [(0, 0), (5, 7)], ids=["fixed", "wrapped"])
def test_attention_bf16_wide_token_stride_takes_general_addressing(shift, tw, d):
    """A canvas whose per-head extent exceeds 4 GiB (token stride of 2^21 elements), tiles of 624 to 1,152 tokens, which head_dim 64 takes to the
    streaming kernel too.  Windows whose runs of tokens break (head_dim 128: width 20 and 13, or wrapping; head_dim 64, runs of 16:
    any) look every such run's tokens up with 64-bit addresses; whole runs, and unbroken windows of head_dim 128 and width 24, go by
    a wave-uniform 64-bit pointer.  13 tokens are fewer than a run of head_dim 64.  Same numbers as the oracle every time."""
    g = _geom("wide", 3, 32, 2 * tw, 16, tw, 16, tw, 1, d, "bf16", 71)
    dense = canvas_qkv(g)
    wide = _strided(dense, g, 1 << 21)
    p = sg.make_problem(g, shift=shift)
    p.grid_stride_token = 1 << 21
    p.grid_stride_head = d                        # one head; any positive multiple of 8
    assert sg.sg_problem_validate(p) == sg.SG_OK
    out = torch.empty(g.tile_shape, dtype=torch.bfloat16, device="cuda")
    sg.sg_tile_attention(p, *wide, 1, 1, out)
    win = [oracle.slice_tile_shifted(to_f64(t), g, 1, 1, *shift).reshape(-1, d) for t in dense]
    assert_close(to_f64(out), oracle.attention(*win, g.scale).reshape(g.tile_shape), "bf16")


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("packed", [True, False], ids=["packed", "window"])
def test_attention_bf16_tokens_too_far_apart_for_lane_offsets(packed, d):
    """A token stride of 2^26 elements: the 16 tokens of a run span more than 4 GiB, so a lane's offset inside it leaves 32 bits.  A tile
    that is the whole canvas is then read as a window of itself, and every token is looked up."""
    g = _geom("far", 1, 10, 13, 10, 13, 10, 13, 1, d, "bf16", 73) if packed else _geom("far", 1, 10, 26, 10, 13, 10, 13, 1, d, "bf16", 73)
    dense = canvas_qkv(g)
    p = sg.make_problem(g)
    p.grid_stride_token = 1 << 26
    p.grid_stride_head = d
    out = torch.empty(g.tile_shape, dtype=torch.bfloat16, device="cuda")
    sg.sg_tile_attention(p, *_strided(dense, g, 1 << 26), 0, g.n_tile_cols - 1, out)
    assert_close(to_f64(out), oracle_tile_attention_full(g, *dense, 0, g.n_tile_cols - 1), "bf16")


@pytest.mark.parametrize("T,th,tw", [(9, 10, 8), (1, 1, 704), (5, 1, 136), (3, 20, 16), (2, 9, 56), (1, 11, 64), (3, 5, 72), (2, 3, 128),
                                     (3, 20, 9), (2, 8, 63), (1, 13, 65)])
@pytest.mark.parametrize("where", ["fixed", "inside", "wrapped"])
def test_attention_bf16_windows_equal_the_packed_tile_bit_for_bit(T, th, tw, where):
    """Windows of head_dim 128 through the loaders for unbroken runs (widths that are multiples of 8, at and below and above a
    stage of 64, one to many tile rows and frames per stage) and for broken ones (other widths, wrapping windows) carry out the
    arithmetic of the packed tile.  The rest of the canvas is NaN: nothing outside the window is read."""
    g = _geom("walk", T, 2 * th, 2 * tw, th, tw, th, tw, 3, 128, "bf16", 37 + tw)
    shift = {"fixed": (0, 0), "inside": (th // 3, 5), "wrapped": (2 * th - (th + 1) // 2, 2 * tw - 3)}[where]
    tile = [randn_tensor(g.tile_shape, "bf16", g.seed + i).cuda() for i in range(3)]
    canvas = []
    for t in tile:
        c = torch.full(g.grid_shape, float("nan"), dtype=torch.bfloat16, device="cuda")
        c[:, :, :th, :tw] = t
        canvas.append(torch.roll(c, shift, dims=(2, 3)))
    got, want = torch.empty_like(tile[0]), torch.empty_like(tile[0])
    sg.sg_tile_attention(sg.make_problem(g, shift=shift), *canvas, 0, 0, got)
    sg.sg_tile_attention(sg.make_problem(_geom("walk", T, th, tw, th, tw, th, tw, 3, 128, "bf16", 0)), *tile, 0, 0, want)
    assert torch.isfinite(want.float()).all() and torch.equal(got, want)


def test_attention_bf16_large_logits_and_constant_v():
    """Scores far from N(0,1): softmax concentrates; constant V must come back exactly-ish."""
    g = _geom("sharp", 2, 10, 16, 10, 16, 10, 16, 2, 128, "bf16", 41)
    q, k, v = canvas_qkv(g)
    q = (q.float() * 4).to(torch.bfloat16)
    got = gpu_tile_attention(g, q, k, v, 0, 0)
    assert_close(to_f64(got), oracle_tile_attention_full(g, q, k, v, 0, 0), "bf16")
    vc = torch.full_like(v, 0.75)
    got = gpu_tile_attention(g, q, k, vc, 0, 0)
    assert float((got.float() - 0.75).abs().max()) <= 0.75 * 2 ** -7


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("sigma", [1.0, 1.5, 2.0])
def test_attention_bf16_wider_inputs_keep_the_tolerance(sigma, d):
    """Q and K ~ N(0, sigma^2) with uncorrelated keys: the kernel multiplies Q by scale * log2(e) and rounds it to bf16
    once more before the score products, an error that grows with |q| |k| and does not cancel in the normalisation.
    At sigma = 2 the logits reach about +-15; the result must still be within the bf16 tolerance of the oracle."""
    g = _geom("wide", 6, 12, 16, 12, 16, 12, 16, 2, d, "bf16", 47)       # N = 1152: 18 key stages
    q, k, v = canvas_qkv(g)
    q = (q.float() * sigma).to(torch.bfloat16)
    k = (k.float() * sigma).to(torch.bfloat16)
    got = gpu_tile_attention(g, q, k, v, 0, 0)
    ref = oracle_tile_attention_full(g, q, k, v, 0, 0)
    ma, rl = errors(to_f64(got), ref)
    print(f"sigma={sigma} d={d}: max_abs={ma:.3e} rel_l2={rl:.3e} max|ref|={np.abs(ref).max():.2f}")
    # the softmax concentrates, outputs reach several units: the absolute bound of the N(0,1) workloads (2e-2, there 3
    # times the largest output) scales with the output's magnitude, the relative L2 bound is the stated one
    assert rl <= BF16_REL_L2 and ma <= BF16_MAX_ABS * max(1.0, float(np.abs(ref).max())), (ma, rl)


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("frames", [2, 11], ids=["n384", "n2112"])
@pytest.mark.parametrize("order", ["ascending", "descending", "spike"])
def test_attention_bf16_softmax_reference_moves(order, frames, d):
    """Scores that keep growing along the key axis (the running reference must move again and again),
    that start at their maximum, or that hold one huge outlier: same numbers as the two-pass oracle.
    N = 384 stays in the kernel's first stages, N = 2112 moves the reference inside its steady loop."""
    g = _geom("adv", frames, 12, 16, 12, 16, 12, 16, 2, d, "bf16", 43)
    q, k, v = canvas_qkv(g)
    N = g.tile_tokens
    u = torch.nn.functional.normalize(randn_tensor((d,), "f32", 5).cuda(), dim=0)
    ramp = torch.linspace(0.0, 1.0, N, device="cuda")
    if order == "descending":
        ramp = ramp.flip(0)
    if order == "spike":
        ramp = torch.zeros(N, device="cuda")
        ramp[N // 2 + 7] = 1.0
    # q along u with length 30; keys get up to 40 u: logits (scale 1/sqrt(d)) span ~0 .. 106 (150 at head_dim 64), far beyond 2^16
    q = (q.float() * 0.3 + 30.0 * u).to(torch.bfloat16)
    k = (k.float() * 0.3 + (40.0 * ramp).reshape(1, g.T, g.tile_h, g.tile_w, 1) * u).to(torch.bfloat16)
    got = gpu_tile_attention(g, q, k, v, 0, 0)
    assert torch.isfinite(got.float()).all()
    assert_close(to_f64(got), oracle_tile_attention_full(g, q, k, v, 0, 0), "bf16", order)


# ------------------------------------------------------------------ blend
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", ["tiny2x2", "triple3x2", "placement", "cover5x4", "oddplanes", "single"])
def test_blend_small(dtype, shape):
    d = 64 if dtype == "f32" else 128
    g = {"tiny2x2": replace(CONFIGS["tiny_f32"], dtype=dtype, head_dim=d),
         "triple3x2": _geom("tr", 2, 9, 7, 5, 4, 2, 3, 3, d, dtype, 51),
         "placement": _geom("pl", 2, 8, 6, 4, 3, 4, 3, 2, d, dtype, 52),
         "cover5x4": _geom("c54", 1, 15, 13, 9, 7, 2, 2, 3, d, dtype, 54),      # up to 5 x 4 tiles per token
         "oddplanes": _geom("odd", 3, 16, 22, 10, 14, 6, 8, 1, d, dtype, 55),   # 3 (head, frame) planes
         "single": _geom("one", 3, 5, 9, 5, 9, 5, 9, 3, d, dtype, 56)}[shape]   # one tile = the canvas
    tiles = [randn_tensor(g.tile_shape, dtype, 600 + i).cuda() for i in range(g.n_tiles)]
    out = torch.full(g.grid_shape, float("nan"), dtype=torch_dtype(dtype), device="cuda")
    sg.sg_tile_blend(sg.make_problem(g), tiles, out)
    ref = oracle.blend([to_f64(t) for t in tiles], g)
    assert_close(to_f64(out), ref, dtype, shape)
    if shape == "placement":      # o = 0: pure placement, bit exact
        assert np.array_equal(to_f64(out)[:, :, 0:4, 0:3, :], to_f64(tiles[0]))


def test_blend_and_step_at_the_maximum_tile_count():
    """256 tiles (16 x 16 of 2 x 2 tokens, stride 1): the most the ABI carries per canvas."""
    g = _geom("max", 1, 17, 17, 2, 2, 1, 1, 1, 64, "f32", 57)
    assert g.n_tiles == 256
    q, k, v = canvas_qkv(g)
    tiles = [torch.empty(g.tile_shape, dtype=torch.float32, device="cuda") for _ in range(g.n_tiles)]
    canvas = torch.empty(g.grid_shape, dtype=torch.float32, device="cuda")
    sg.sg_denoise_step_tiled(sg.make_problem(g), canvas, tiles, q=q, k=k, v=v)
    outs = [oracle_tile_attention_full(g, q, k, v, tr, tc) for tr in range(16) for tc in range(16)]
    for i in (0, 17, 255):
        assert_close(to_f64(tiles[i]), outs[i], "f32", f"tile {i}")
    assert_close(to_f64(canvas), oracle.blend(outs, g), "f32")


def test_blend_token_major_canvas():
    g = _geom("tm", 2, 9, 7, 5, 4, 2, 3, 3, 128, "bf16", 53)
    tiles = [randn_tensor(g.tile_shape, "bf16", 700 + i).cuda() for i in range(g.n_tiles)]
    out = torch.empty((g.T, g.H, g.W, g.heads, g.head_dim), dtype=torch.bfloat16, device="cuda")
    sg.sg_tile_blend(sg.make_problem(g, token_major=True), tiles, out)
    ref = oracle.blend([to_f64(t) for t in tiles], g)
    assert_close(to_f64(out.permute(3, 0, 1, 2, 4)), ref, "bf16")


# ------------------------------------------------------------------ gate
def _gate(x_cur, x_cached, has_cache, thr):
    n = len(x_cur)
    hc = torch.tensor(has_cache, dtype=torch.uint8, device="cuda")
    scores = torch.full((max(n, 1),), -1.0, dtype=torch.float32, device="cuda")
    rec = torch.full((max(n, 1),), 7, dtype=torch.uint8, device="cuda")
    ws = torch.empty(sg.sg_workspace_bytes(n), dtype=torch.uint8, device="cuda")
    sg.sg_cache_gate(x_cur, x_cached, hc, thr, scores, rec, ws)
    torch.cuda.synchronize()
    return scores.cpu().numpy()[:n], rec.cpu().numpy()[:n].astype(bool)


def _check_gate(x_cur, x_cached, has_cache, thr):
    s, r = _gate(x_cur, x_cached, has_cache, thr)
    so, ro = oracle.cache_gate([to_f64(t) for t in x_cur], [to_f64(t) for t in x_cached], has_cache,
                               float(np.float32(thr)))
    for i in range(len(x_cur)):
        if np.isinf(so[i]):
            assert np.isinf(s[i]) and r[i]
            continue
        assert abs(s[i] - so[i]) <= 2e-6 * max(1.0, so[i]), (i, s[i], so[i])
        if abs(so[i] - float(np.float32(thr))) > 1e-4:       # decisions bit exact outside the band
            assert r[i] == ro[i], (i, s[i], so[i])
    return s, r


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("elems", [8, 1000, 4099, 3 * 2 * 3 * 10 * 10 * 64, 1 << 20])
def test_gate_small(dtype, elems):
    n = 5
    cached = [randn_tensor((elems,), dtype, 800 + i).cuda() for i in range(n)]
    eps = [0.0, 0.01, 0.1, 0.06, 0.04]
    cur = [perturb_(c.clone(), e, 900 + i) for i, (c, e) in enumerate(zip(cached, eps))]
    s, r = _check_gate(cur, cached, [1, 1, 1, 1, 0], 0.05)
    assert s[0] == 0.0 and not r[0] and r[4]


def test_gate_edge_cases():
    x = randn_tensor((4096,), "bf16", 1).cuda()
    z = torch.zeros_like(x)
    s, r = _check_gate([x, x, z], [z, x, z], [1, 1, 1], 0.05)
    assert np.isinf(s[0]) and r[0] and not r[1] and r[2]        # zero cache -> +inf -> recompute
    # exact tie: x_cur = (1 + 1/16) x_cached on exactly representable data, threshold 1/16
    xc = (torch.arange(4096, device="cuda") % 7 + 1).float()
    s, r = _gate([xc * 1.0625, xc * 1.03125], [xc, xc], [1, 1], 0.0625)
    assert s[0] == 0.0625 and r[0] and s[1] == 0.03125 and not r[1]
    # negative threshold: everything recomputes; zero tiles: no-op
    s, r = _gate([x], [x], [1], -1.0)
    assert r[0]
    _gate([], [], [], 0.05)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("where,bad", [("cur", float("nan")), ("cached", float("nan")), ("cur", float("inf")),
                                       ("cached", float("inf"))])
def test_gate_nan_or_inf_input_recomputes(dtype, where, bad):
    """A NaN or Inf anywhere in a tile's input or cache must not leave the stale cache in use (Equation 7 reuses
    only strictly below the threshold); the oracle takes the same decisions."""
    n = 3
    cached = [randn_tensor((8192 + 24,), dtype, 1300 + i).cuda() for i in range(n)]
    cur = [perturb_(c.clone(), 0.01, 1400 + i) for i, c in enumerate(cached)]      # all three would reuse
    (cur if where == "cur" else cached)[1][4321] = bad
    s, r = _gate(cur, cached, [1] * n, 0.05)
    so, ro = oracle.cache_gate([to_f64(t) for t in cur], [to_f64(t) for t in cached], [1] * n, float(np.float32(0.05)))
    assert list(r.astype(bool)) == list(ro) == [False, True, False]
    assert not (s[1] < 0.05) and not (so[1] < 0.05)
    assert abs(s[0] - so[0]) <= 2e-6 and abs(s[2] - so[2]) <= 2e-6


def test_gate_many_tiles():
    n = 70                                            # more than one launch's worth of pointers
    cached = [randn_tensor((2048,), "bf16", 1000 + i).cuda() for i in range(n)]
    cur = [perturb_(c.clone(), 0.1 if i % 3 == 0 else 0.01, 2000 + i) for i, c in enumerate(cached)]
    s, r = _check_gate(cur, cached, [1] * n, 0.05)
    assert list(r) == [i % 3 == 0 for i in range(n)]


# ------------------------------------------------------------------ tiled step
def test_step_canvas_mode_tiny_f32():
    g = CONFIGS["tiny_f32"]
    q, k, v = canvas_qkv(g)
    cache_out = [torch.empty(g.tile_shape, dtype=torch.float32, device="cuda") for _ in range(g.n_tiles)]
    canvas = torch.empty(g.grid_shape, dtype=torch.float32, device="cuda")
    sg.sg_denoise_step_tiled(sg.make_problem(g), canvas, cache_out, q=q, k=k, v=v)
    outs = [oracle_tile_attention_full(g, q, k, v, tr, tc) for tr in range(2) for tc in range(2)]
    assert_close(to_f64(canvas), oracle.blend(outs, g), "f32")


@pytest.mark.parametrize("d", [128, 64])
def test_step_cached_mode_bf16_three_steps(d):
    g = _geom("stepc", 2, 14, 20, 8, 12, 6, 8, 2, d, "bf16", 61)         # 2x2 tiles, N = 192
    n = g.n_tiles
    canvas_in = canvas_qkv(g)
    tile_x = []
    for tr in range(g.n_tile_rows):
        for tc in range(g.n_tile_cols):
            r0, c0 = tr * g.stride_h, tc * g.stride_w
            tile_x.append(torch.stack([t[:, :, r0:r0 + g.tile_h, c0:c0 + g.tile_w, :] for t in canvas_in]).contiguous())
    cache_x = [torch.zeros_like(t) for t in tile_x]
    cache_out = [torch.zeros(g.tile_shape, dtype=torch.bfloat16, device="cuda") for _ in range(n)]
    has_cache = torch.zeros(n, dtype=torch.uint8, device="cuda")
    scores = torch.empty(n, dtype=torch.float32, device="cuda")
    rec = torch.empty(n, dtype=torch.uint8, device="cuda")
    ws = torch.empty(sg.sg_workspace_bytes(n), dtype=torch.uint8, device="cuda")
    canvas = torch.empty(g.grid_shape, dtype=torch.bfloat16, device="cuda")
    p = sg.make_problem(g)
    state = oracle.StepState(n)
    eps = [[0, 0, 0, 0], [0.01, 0.1, 0.01, 0.1], [0.01, 0.01, 0.1, 0.01]]
    expect = [[True] * 4, [False, True, False, True], [False, False, True, False]]
    for step in range(3):
        if step:
            for i in range(n):
                perturb_(tile_x[i], eps[step][i], 3000 + 10 * step + i)
        sg.sg_denoise_step_tiled(p, canvas, cache_out, tile_x=tile_x, cache_x=cache_x, has_cache=has_cache,
                                 threshold=0.05, scores=scores, recompute=rec, workspace=ws)
        torch.cuda.synchronize()
        ref_canvas, ref_s, ref_r = oracle.denoise_step_tiled(
            [tuple(to_f64(t[j]) for j in range(3)) for t in tile_x], g, g.scale, state, float(np.float32(0.05)))
        assert list(rec.cpu().numpy().astype(bool)) == list(ref_r) == expect[step]
        got_s = scores.cpu().numpy()
        for i in range(n):
            assert (np.isinf(ref_s[i]) and np.isinf(got_s[i])) or abs(got_s[i] - ref_s[i]) < 2e-6
        assert has_cache.cpu().numpy().all()
        assert_close(to_f64(canvas), ref_canvas, "bf16", f"step {step}")
        for i in range(n):                       # cache holds exactly the last recomputed input
            assert np.array_equal(to_f64(cache_x[i]).ravel(), state.cache_x[i])


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("heads,N", [(1, 100), (2, 129), (25, 1124), (26, 1124), (40, 1030), (56, 1030), (52, 1281)])
def test_attention_bf16_whole_and_halved_rounds(heads, N, d):
    """Query blocks dealt whole and, in a last round that fills at most half of the compute units, as halves: 1 to 130 workgroups
    (halved up to 128 on 256 compute units), 200 (whole), 280 and 312 (a whole round, and 24 / 56 halved), with last blocks of 1,
    6 and 100 rows, so that second halves are empty; every row of the first, the middle and the last head."""
    g = _geom("hv", 1, 1, N, 1, N, 1, N, heads, d, "bf16", 4000 + heads)
    q, k, v = canvas_qkv(g)
    out = torch.full(g.tile_shape, float("nan"), dtype=torch.bfloat16, device="cuda")
    sg.sg_tile_attention(sg.make_problem(g), q, k, v, 0, 0, out)
    assert torch.isfinite(out.float()).all()
    for a in sorted({0, heads // 2, heads - 1}):
        one = [to_f64(t[a]).reshape(N, d) for t in (q, k, v)]
        assert_close(to_f64(out[a]).reshape(N, d), oracle.attention(*one, g.scale), "bf16", a)


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("T,th,tw", [(1, 5, 8), (1, 1, 255), (1, 16, 16), (1, 1, 257), (3, 20, 25), (5, 13, 21), (9, 16, 17), (11, 16, 29)])
def test_step_refreshes_the_cache_while_it_attends(T, th, tw, d):
    """The cache refresh that rides on the attention launch, bit for bit: one to twenty query blocks, whose stages lie in the
    first iterations, the steady loop and the last ones; ragged and whole last stages (N = 40 ... 5,104); the tile that is
    reused keeps its cache."""
    g = _geom("rf", T, 2 * th, tw, th, tw, th, tw, 2, d, "bf16", 77 + tw)
    x = [randn_tensor((3,) + g.tile_shape, "bf16", g.seed + i).cuda() for i in range(2)]
    cache = [torch.full_like(x[0], 3.0), x[1].clone()]          # tile 0 has drifted, tile 1 has not
    has = torch.tensor([1, 1], dtype=torch.uint8, device="cuda")
    out = [torch.full(g.tile_shape, 7.0, dtype=torch.bfloat16, device="cuda") for _ in range(2)]
    cache[1].view(-1)[0] += 1.0                                 # ... measurably: a refresh of tile 1 would show
    kept = cache[1].clone()
    canvas = torch.empty(g.grid_shape, dtype=torch.bfloat16, device="cuda")
    scores, rec = torch.empty(2, device="cuda"), torch.empty(2, dtype=torch.uint8, device="cuda")
    ws = torch.empty(sg.sg_workspace_bytes(2), dtype=torch.uint8, device="cuda")
    for step in range(2):
        if step == 1:
            has.zero_()
        sg.sg_denoise_step_tiled(sg.make_problem(g), canvas, out, tile_x=x, cache_x=cache, has_cache=has, threshold=0.5,
                                 scores=scores, recompute=rec, workspace=ws)
        assert rec.tolist() == ([1, 0] if step == 0 else [1, 1])
        assert torch.equal(cache[0], x[0]) and has.tolist() == [1, 1]
        assert torch.equal(cache[1], kept if step == 0 else x[1])
    one = g.single_tile()
    assert torch.equal(out[0], gpu_tile_attention(one, x[0][0], x[0][1], x[0][2], 0, 0))


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_step_cached_mode_many_tiles_one_launch_skips_on_the_device(dtype):
    """40 packed tiles (more than one launch's table of 32) through the cached step: the attention launches number
    only the tiles the gate flags, whichever they are.  Reused tiles must keep their cached output bit for bit,
    recomputed ones must match the oracle; the flagged sets straddle the two launches unevenly."""
    d = 128 if dtype == "bf16" else 64
    g = _geom("many", 1, 18, 23, 6, 5, 3, 2, 2, d, dtype, 67)            # 5 x 10 = 50 tiles, N = 30 (one ragged block)
    n = g.n_tiles
    assert n == 50
    td = torch_dtype(dtype)
    tile_x = [randn_tensor((3,) + g.tile_shape, dtype, 4000 + i).cuda() for i in range(n)]
    cache_x = [torch.zeros_like(t) for t in tile_x]
    cache_out = [torch.zeros(g.tile_shape, dtype=td, device="cuda") for _ in range(n)]
    has_cache = torch.zeros(n, dtype=torch.uint8, device="cuda")
    scores = torch.empty(n, dtype=torch.float32, device="cuda")
    rec = torch.empty(n, dtype=torch.uint8, device="cuda")
    ws = torch.empty(sg.sg_workspace_bytes(n), dtype=torch.uint8, device="cuda")
    canvas = torch.empty(g.grid_shape, dtype=td, device="cuda")
    p = sg.make_problem(g)
    patterns = [None,
                [i in (0, 31, 32, 49) for i in range(n)],                 # first and last slot of both launches
                [i >= 33 for i in range(n)],                              # first launch entirely skipped
                [False] * n]                                              # nothing runs
    for step, pat in enumerate(patterns):
        if pat is not None:
            for i in range(n):
                perturb_(tile_x[i], 0.1 if pat[i] else 0.001, 5000 + 100 * step + i)
        before = [t.clone() for t in cache_out]
        sg.sg_denoise_step_tiled(p, canvas, cache_out, tile_x=tile_x, cache_x=cache_x, has_cache=has_cache,
                                 threshold=0.05, scores=scores, recompute=rec, workspace=ws)
        torch.cuda.synchronize()
        want = [True] * n if pat is None else pat
        assert list(rec.cpu().numpy().astype(bool)) == want, step
        for i in range(n):
            if not want[i]:
                assert torch.equal(cache_out[i], before[i]), (step, i)
            elif i in (0, 31, 32, 33, 49):
                Q, K, V = (to_f64(tile_x[i][j]) for j in range(3))
                ref = np.stack([oracle.attention(Q[a].reshape(-1, d), K[a].reshape(-1, d), V[a].reshape(-1, d), g.scale)
                                for a in range(g.heads)]).reshape(g.tile_shape)
                assert_close(to_f64(cache_out[i]), ref, dtype, f"step {step} tile {i}")
        assert_close(to_f64(canvas), oracle.blend([to_f64(t) for t in cache_out], g), dtype, f"canvas step {step}")


# ------------------------------------------------------------------ error paths reach no kernel
def test_bad_arguments_are_rejected():
    g = CONFIGS["tiny_f32"]
    q, k, v = canvas_qkv(g)
    out = torch.empty(g.tile_shape, dtype=torch.float32, device="cuda")
    with pytest.raises(sg.SgError) as e:
        sg.sg_tile_attention(sg.make_problem(g), q, k, v, 2, 0, out)
    assert e.value.status == sg.SG_ERR_INVALID_ARG
    with pytest.raises(sg.SgError) as e:
        sg.sg_tile_attention(sg.make_problem(g), q, k, None, 0, 0, out)
    assert e.value.status == sg.SG_ERR_INVALID_ARG


def _random_geometries(count, seed):
    rng = np.random.default_rng(seed)
    out = []
    while len(out) < count:
        T = int(rng.integers(1, 4))
        th, tw = int(rng.integers(2, 14)), int(rng.choice([3, 5, 8, 8, 12, 16, 16, 24, 7, 10]))
        sh, sw = int(rng.integers(1, th + 1)), int(rng.integers(1, tw + 1))
        nr, nc = int(rng.integers(1, 4)), int(rng.integers(1, 4))
        H, W = (nr - 1) * sh + th, (nc - 1) * sw + tw
        if T * th * tw > 900 or T * H * W > 6000:
            continue
        heads = int(rng.integers(1, 4))
        out.append((T, H, W, th, tw, sh, sw, nr, nc, heads, bool(rng.integers(0, 2))))
    return out


@pytest.mark.parametrize("geom", _random_geometries(36, 2024), ids=lambda t: "T%d_%dx%d_tile%dx%d_s%dx%d_%dx%d_h%d_%s" % (
    t[0], t[1], t[2], t[3], t[4], t[5], t[6], t[7], t[8], t[9], "tm" if t[10] else "hm"))
def test_attention_bf16_random_geometries(geom):
    """Seeded random tilings (tile widths that are and are not multiples of 8, single tiles, token-major
    canvases, key counts below and above one stage): the last tile and a random one against the oracle."""
    T, H, W, th, tw, sh, sw, nr, nc, heads, token_major = geom
    g = TileGeometry("rnd", T, H, W, th, tw, sh, sw, nr, nc, heads, 128, "bf16", 300 + T * 7 + H * 13 + W)
    qkv = canvas_qkv(g)
    dev = [t.permute(1, 2, 3, 0, 4).contiguous() for t in qkv] if token_major else qkv
    p = sg.make_problem(g, token_major=token_major)
    for tr, tc in {(nr - 1, nc - 1), ((g.seed * 3) % nr, (g.seed * 5) % nc)}:
        out = torch.full(g.tile_shape, float("nan"), dtype=torch.bfloat16, device="cuda")
        sg.sg_tile_attention(p, *dev, tr, tc, out)
        assert_close(to_f64(out), oracle_tile_attention_full(g, *qkv, tr, tc), "bf16", f"{geom} tile {tr},{tc}")
