"""bf16 attention of few stages (64 keys, head_dim 64: 128): up to 24 of them every iteration is the same code, the first and the last
included, and there is one copy of it per slot of the ring of four; beyond, a steady loop of groups of four begins at the second."""
import math

import pytest
import torch

import paper_2508_17756_amd as sg
from synthetic import TileGeometry
from gpu_util import assert_close
from test_gpu_extremes import _attend_window

pytestmark = pytest.mark.gpu

HEADS = 2


def _inputs(n, d):
    gen = torch.Generator().manual_seed(1000 * d + n)
    return [torch.randn(HEADS, n, d, generator=gen).to(torch.bfloat16) for _ in range(3)]


def _exact(q, k, v):
    out = torch.empty(q.shape, dtype=torch.float64)
    for a in range(q.shape[0]):
        out[a] = torch.softmax(q[a].double() @ k[a].double().T / math.sqrt(q.shape[2]), dim=1) @ v[a].double()
    return out


# Stages of 64 | 128 keys
SIZES = [
    (1, 7, 9),      # 63: 1 | 1
    (1, 8, 16),     # 128: 2 | 1, whole
    (1, 3, 43),     # 129: 3 | 2, the last with one key
    (1, 16, 16),    # 256: 4 | 2, whole
    (1, 1, 257),    # 257: 5 | 3, the last with one key
    (1, 16, 33),    # 528: 9 | 5
    (2, 23, 32),    # 1,472: 23 | 12
    (1, 48, 32),    # 1,536: 24 | 12, the last of the short form for head_dim 128
    (1, 53, 29),    # 1,537: 25 | 13
    (1, 32, 64),    # 2,048: 32 | 16, the last of the short form for packed tiles of head_dim 64 without a refresh
    (1, 3, 683),    # 2,049: 33 | 17, the last with one key
    (2, 32, 48),    # 3,072: 48 | 24, the last of the short form for head_dim 64
    (1, 7, 439),    # 3,073: 49 | 25
    # the other form: 1 iteration, groups of four of the steady loop, 4 to 7 iterations
    (1, 50, 32),    # 1,600: 25, whole
    (1, 52, 32),    # 1,664: 26, whole
    (1, 54, 32),    # 1,728: 27, whole
    (7, 13, 19),    # 1,729: 28, the last with one key
    (1, 56, 32),    # 1,792: 28, whole
    (1, 100, 32),   # 3,200: 50 | 25, whole
    (3, 11, 97),    # 3,201: 51 | 26, the last with one key
    (1, 112, 32),   # 3,584: 56 | 28, whole
]


@pytest.mark.parametrize("where", ["packed", "fixed", "wrapped"])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("T,th,tw", SIZES)
def test_sizes(T, th, tw, d, where):
    n = T * th * tw
    q, k, v = _inputs(n, d)
    got = _attend_window("bf16", d, HEADS, T, th, tw, q, k, v, wrapped=where == "wrapped" and th > 2, packed=where == "packed")
    assert_close(got.double().numpy(), _exact(q, k, v).numpy(), "bf16", "%d tokens x %d" % (n, d))


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("T,th,tw", SIZES)
def test_the_cache_refresh_copies_the_input(T, th, tw, d):
    g = TileGeometry("refresh", T, th, 2 * tw, th, tw, th, tw, 1, 2, HEADS, d, "bf16", 0)
    n = T * th * tw
    x = [torch.stack([t.reshape((HEADS, T, th, tw, d)) for t in _inputs(n, d)]).cuda() * f for f in (1.0, 0.5)]
    cache_x = [torch.full_like(t, 7.0) for t in x]
    out = [torch.zeros((HEADS, T, th, tw, d), dtype=torch.bfloat16, device="cuda") for _ in x]
    has_cache = torch.tensor([0, 1], dtype=torch.uint8, device="cuda")
    cache_x[1].copy_(x[1])   # nothing has changed: reused
    scores, recompute = torch.zeros(2, device="cuda"), torch.zeros(2, dtype=torch.uint8, device="cuda")
    canvas = torch.empty(g.grid_shape, dtype=torch.bfloat16, device="cuda")
    ws = torch.empty(sg.sg_workspace_bytes(2), dtype=torch.uint8, device="cuda")
    sg.sg_denoise_step_tiled(sg.make_problem(g), canvas, out, tile_x=x, cache_x=cache_x, has_cache=has_cache, threshold=0.05, scores=scores,
                             recompute=recompute, workspace=ws)
    assert recompute.tolist() == [1, 0] and has_cache.tolist() == [1, 1]
    assert torch.equal(cache_x[0], x[0]) and torch.equal(cache_x[1], x[1])
    assert not out[1].any()
    assert_close(out[0].cpu().double().reshape(HEADS, n, d).numpy(), _exact(*x[0].cpu().reshape(3, HEADS, n, d)).numpy(), "bf16")


@pytest.mark.parametrize("where", ["fixed", "wrapped"])
@pytest.mark.parametrize("d,T,th,tw,stride", [
    (128, 2, 40, 21, 1 << 19),   # 1,680 tokens: 27 stages, runs of 8 tokens broken
    (128, 2, 35, 24, 1 << 19),   # 1,680, unbroken unless the window wraps
    (64, 4, 37, 21, 1 << 18),    # 3,108: 25 stages, runs of 16 broken
    (64, 5, 50, 13, 1 << 18),    # 3,250: 26, narrower than a run
    (64, 4, 25, 32, 1 << 18),    # 3,200: 25 whole, unbroken unless the window wraps
])
def test_windows_of_heads_beyond_4_gib_in_the_other_form(d, T, th, tw, stride, where):
    """More than 24 stages of a head that spans 4 GiB or more: broken runs are looked up with 64-bit addresses."""
    n = T * th * tw
    q, k, v = (x[:1] for x in _inputs(n, d))
    got = _attend_window("bf16", d, 1, T, th, tw, q, k, v, wrapped=where == "wrapped", token_stride=stride)
    assert_close(got.double().numpy(), _exact(q, k, v).numpy(), "bf16", "%d tokens x %d" % (n, d))
