"""Attention at the ends of the value range: one dominating key, the largest finite values, infinities, NaN."""
import math

import pytest
import torch

import paper_2508_17756_amd as sg
from synthetic import TileGeometry, torch_dtype

pytestmark = pytest.mark.gpu

LOG2E = math.log2(math.e)


def _attend_window(dtype, d, heads, T, th, tw, q, k, v, wrapped=False, packed=False, token_stride=0):
    """Attention of tile (0, 0) of a canvas of 2 x 2 tiles (packed: of one), whose tokens are q, k, v [heads][N][d]; wrapped:
    shifted so far that the window crosses both canvas edges.  With a token stride the three canvases lie in one
    buffer of tokens that far apart, their heads side by side in every token."""
    rows, cols = (1, 1) if packed else (2, 2)
    g = TileGeometry("ends", T, rows * th, cols * tw, th, tw, th, tw, rows, cols, heads, d, dtype, 0)
    shift = (2 * th - 3, 2 * tw - 5) if wrapped else (0, 0)
    canvases = []
    for x in (q, k, v):
        c = torch.zeros(g.grid_shape, dtype=torch_dtype(dtype))
        c[:, :, :th, :tw] = x.reshape(heads, T, th, tw, d).to(c.dtype)
        canvases.append(torch.roll(c, shift, dims=(2, 3)).cuda())
    out = torch.empty(g.tile_shape, dtype=torch_dtype(dtype), device="cuda")
    p = sg.make_problem(g, shift=shift)
    if token_stride:
        buf = torch.empty(g.grid_tokens * token_stride, dtype=out.dtype, device="cuda")
        p.grid_stride_token, p.grid_stride_head = token_stride, d
        for i, c in enumerate(canvases):
            canvases[i] = buf[i * heads * d:]
            view = canvases[i].as_strided((heads, g.grid_tokens, d), (d, token_stride, 1))
            view.copy_(c.reshape(heads, g.grid_tokens, d))
    sg.sg_tile_attention(p, *canvases, 0, 0, out)
    return out.cpu().reshape(heads, -1, d)


def _dominated(d, n, key):
    """Queries 0 .. n-1 whose score of `key` is 14 to 15.9 in the log2 domain, that of key 0 is 0 and the others' is below -40: the
    softmax is 1 - 2^-14 or more at `key`, whatever the other keys hold."""
    q, k = torch.zeros(1, n, d), torch.zeros(1, n, d)
    step = 0.5                                             # bf16 holds these
    first = math.ceil(14.0 * math.sqrt(d) / LOG2E / step)
    last = math.floor(15.9 * math.sqrt(d) / LOG2E / step)
    q[0, :, 0] = step * (first + torch.arange(n) % (last - first + 1))
    q[0, :, 1] = 255.0
    k[0, :, 1] = -1.0 * math.sqrt(d / 64)
    k[0, 0] = 0.0
    k[0, key] = 0.0
    k[0, key, 0] = 1.0
    return q, k


def _check_dominated(d, T, th, tw, key, **where):
    n = T * th * tw
    q, k = _dominated(d, n, key)
    v = torch.zeros(1, n, d)
    v[0, key] = torch.where(torch.arange(d) % 2 == 0, 1.0, 3e38)
    got = _attend_window("bf16", d, 1, T, th, tw, q, k, v, **where).double()[0]
    p = torch.softmax((q[0].double() @ k[0].double().T) / math.sqrt(d), dim=1)[:, key]
    assert float((got[:, 0::2] - p[:, None]).abs().max()) <= 2 ** -9
    assert bool(torch.isfinite(got).all())
    big = float(torch.tensor(3e38).bfloat16())
    assert float((got[:, 1::2] / big - p[:, None]).abs().max()) <= 2 ** -8     # one bf16 unit: 3e38 is rounded as well


@pytest.mark.parametrize("wrapped", [False, True], ids=["fixed", "wrapped"])
@pytest.mark.parametrize("T,th,tw,key", [(1, 15, 20, 299), (2, 12, 21, 200), (2, 12, 21, 503), (5, 20, 25, 1300)])
def test_head_dim_64_windows_hold_the_dominating_probability_exactly(T, th, tw, key, wrapped):
    """The probability of a dominating key far above the first stage's maximum is 1: its output is its value, rounded to bf16 once
    (half a unit in the last place, 2^-9 below 1, and the 2^-14 of key 0).  A probability that is itself rounded to bf16 would add
    up to as much again.  For the same reason the largest finite value comes back finite.  300 tokens take the short kernel."""
    _check_dominated(64, T, th, tw, key, wrapped=wrapped)


@pytest.mark.parametrize("tw,wrapped", [(21, False), (21, True), (24, True)], ids=["w21", "w21_wrapped", "w24_wrapped"])
def test_windows_of_heads_beyond_4_gib_hold_the_dominating_probability_exactly(tw, wrapped):
    """The same of head_dim 128 where a head spans 4 GiB or more and the window wraps or is no multiple of 8 tokens wide."""
    _check_dominated(128, 2, 10, tw, 2 * 10 * tw - 1, wrapped=wrapped, token_stride=1 << 21)


def _infinite_last_value(dtype, d, heads, T, th, tw, **where):
    n = T * th * tw
    gen = torch.Generator().manual_seed(n + d)
    q, k, v = (torch.randn(heads, n, d, generator=gen) for _ in range(3))
    v[:, n - 1, 3] = math.inf
    got = _attend_window(dtype, d, heads, T, th, tw, q, k, v, **where)
    assert bool((got[:, :, 3] == math.inf).all())
    got[:, :, 3] = 0.0
    assert bool(torch.isfinite(got).all())


@pytest.mark.parametrize("wrapped", [False, True], ids=["fixed", "wrapped"])
@pytest.mark.parametrize("T,th,tw", [(1, 16, 36), (1, 20, 23), (1, 16, 32), (2, 17, 40), (5, 20, 25)])
def test_head_dim_64_windows_take_an_infinite_last_value(T, th, tw, wrapped):
    """576, 460, 512, 1,360, 2,500 tokens: the keys that fill up the last stage stand in for the last one and must not turn its
    infinity into 0 * inf."""
    _infinite_last_value("bf16", 64, 2, T, th, tw, wrapped=wrapped)


@pytest.mark.parametrize("dtype,d,packed,shape", [("bf16", 64, False, (1, 15, 20)), ("bf16", 64, False, (3, 20, 23)), ("bf16", 64, True, (3, 20, 23)),
                                                  ("bf16", 128, False, (3, 20, 24)), ("bf16", 128, False, (3, 20, 23)),
                                                  ("bf16", 128, True, (3, 20, 23)), ("f32", 64, False, (3, 20, 23)), ("f32", 128, True, (3, 20, 23))])
@pytest.mark.parametrize("where,token", [("q", 77), ("k", 0), ("k", 299), ("v", 5), ("v", 260)])
def test_nan_reaches_what_depends_on_it_and_nothing_else(dtype, d, packed, shape, where, token):
    """A NaN in a query reaches that query's output, one in a key every output, one in a value its channel of every output; in the
    first stage of keys, where the softmax reference is set, and behind it.  Every kernel."""
    T, th, tw = shape
    n = T * th * tw
    gen = torch.Generator().manual_seed(n + d)
    x = {name: torch.randn(2, n, d, generator=gen) for name in "qkv"}
    x[where][1, token, 9] = math.nan
    got = _attend_window(dtype, d, 2, T, th, tw, x["q"], x["k"], x["v"], packed=packed).isnan()
    want = torch.zeros(2, n, d, dtype=torch.bool)
    if where == "q":
        want[1, token] = True
    elif where == "k":
        want[1] = True
    else:
        want[1, :, 9] = True
    assert torch.equal(got, want)


def _fma(a, b, c):
    """fp32 fused multiply-add: product and sum in fp64, rounded once (the sum's second rounding is 2^-29 of the first)."""
    return (a.double() * b.double() + c.double()).float()


def _fp32_attention(q, k, v, scale):
    """Attention in fp32 with the score's channels in four interleaved chains of fused multiply-adds and the values added in runs of
    32 keys: the error that fp32 on the vector ALU has."""
    qs, n, d = q * torch.tensor(scale, dtype=torch.float32), q.shape[1], q.shape[2]
    chains = [torch.zeros(q.shape[0], n, n) for _ in range(4)]
    for c in range(d):
        chains[c % 4] = _fma(qs[:, :, None, c], k[:, None, :, c], chains[c % 4])
    s = (chains[0] + chains[1]) + (chains[2] + chains[3])
    p = torch.exp2((s - s.max(2, keepdim=True).values) * LOG2E)
    out, total = torch.zeros_like(q), torch.zeros(q.shape[0], n, 1)
    for j0 in range(0, n, 32):
        o = torch.zeros_like(q)
        for j in range(j0, min(j0 + 32, n)):
            o = _fma(p[:, :, j:j + 1], v[:, None, j], o)
        out, total = out + o, total + p[:, :, j0:j0 + 32].sum(2, keepdim=True)
    return out / total


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("th,tw", [(3, 11), (9, 9), (10, 15)])
def test_fp32_attention_is_as_close_to_fp64_as_plain_fp32(th, tw, d):
    """Tiles of 33, 81, 150 tokens, where the rounding of the scores is most of the error: no further from fp64 than plain fp32 (5 % for
    the spread of 12 heads' worth of roundings)."""
    n, heads = th * tw, 12
    gen = torch.Generator().manual_seed(n + d)
    q, k, v = (torch.randn(heads, n, d, generator=gen) for _ in range(3))
    scale = 1.0 / math.sqrt(d)
    ref = torch.softmax(q.double() @ k.double().transpose(1, 2) * scale, dim=2) @ v.double()
    got = _attend_window("f32", d, heads, 1, th, tw, q, k, v, packed=True).double()
    plain = _fp32_attention(q, k, v, scale).double()
    assert float((got - ref).norm()) <= 1.05 * float((plain - ref).norm())


# 1 head: eight shares of the keys, 400 tokens are 13 blocks of 32 keys, dealt to the shares in turn; 48 heads: the kernel on the bf16 instruction, but
# four shares for heads beyond 4 GiB and eight up to 64 tokens.
@pytest.mark.parametrize("heads", [1, 48])
@pytest.mark.parametrize("d", [64, 128])
def test_fp32_attention_takes_values_up_to_the_largest_number(d, heads):
    """Scores that rise by 4.9 from a share's first block of keys to its second or third: no probability may exceed 1, or
    3e38 times it would overflow."""
    n, key = 400, 261                                       # block 8, that of share 0 in either split
    q, k, v = torch.zeros(heads, n, d), torch.zeros(heads, n, d), torch.zeros(heads, n, d)
    q[:, :, 0] = math.sqrt(d)
    k[:, key, 0] = 4.9
    v[:, key] = 3e38
    got = _attend_window("f32", d, heads, 1, 16, 25, q, k, v, packed=True).double()
    want = 3e38 * math.exp(4.9) / (math.exp(4.9) + n - 1)
    assert float((got / want - 1.0).abs().max()) <= 1e-5


@pytest.mark.parametrize("key", [1, 40, 261])
@pytest.mark.parametrize("heads", [1, 48])
@pytest.mark.parametrize("d", [64, 128])
def test_fp32_attention_counts_probabilities_below_the_normal_range(d, heads, key):
    """A key 90 below the maximum has probability 8e-40: times 3e38 it is 0.25, in the block of the maximum, another share of the keys and
    a later block of the same share.  The rounding of the exponent (130 +- 2^-17) and of the probability (2^-150) allow 7e-6."""
    n = 400
    q, k, v = torch.zeros(heads, n, d), torch.zeros(heads, n, d), torch.zeros(heads, n, d)
    q[:, :, 0] = math.sqrt(d)
    k[:, :, 0] = -200.0
    k[:, 0, 0] = 0.0
    k[:, key, 0] = -90.0
    v[:, key] = 3e38
    got = _attend_window("f32", d, heads, 1, 16, 25, q, k, v, packed=True).double()
    assert float((got / (3e38 * math.exp(-90.0)) - 1.0).abs().max()) <= 1.2e-5


@pytest.mark.parametrize("block", [0, 1, 4, 11, 12])
@pytest.mark.parametrize("heads", [1, 48])
@pytest.mark.parametrize("d", [64, 128])
def test_fp32_attention_ignores_a_block_of_scores_at_minus_infinity(d, heads, block):
    """Keys whose scores overflow to -inf have probability 0, also where they are all that a share of the keys has seen so far."""
    n = 400
    gen = torch.Generator().manual_seed(n + d)
    q, k, v = (torch.randn(heads, n, d, generator=gen) for _ in range(3))
    q[:, :, 7] = 1e20
    k[:, :, 7] = 0.0
    gone = slice(32 * block, min(32 * block + 32, n))
    k[:, gone, 7] = -1e20
    got = _attend_window("f32", d, heads, 1, 16, 25, q, k, v, packed=True).double()
    s = q.double() @ k.double().transpose(1, 2) / math.sqrt(d)
    s[:, :, gone] = -math.inf
    ref = torch.softmax(s, dim=2) @ v.double()
    assert float((got - ref).norm() / ref.norm()) <= 1e-5


@pytest.mark.parametrize("heads", [1, 48])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("T,th,tw", [(1, 1, 7), (1, 3, 11), (1, 16, 25), (1, 16, 26)])
def test_fp32_attention_takes_an_infinite_last_value(T, th, tw, d, heads):
    """7, 33, 400 and 416 tokens: the keys that fill up the last block of 32 stand in for the last one."""
    _infinite_last_value("f32", d, heads, T, th, tw)


@pytest.mark.parametrize("heads", [1, 48])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("wrapped", [False, True], ids=["fixed", "wrapped"])
@pytest.mark.parametrize("stride", [1 << 19, 1 << 20], ids=["3gib", "6gib"])
def test_fp32_attention_of_heads_of_gibibytes(stride, wrapped, d, heads):
    """Byte offsets inside a head that take all 32 bits (48 heads: in the kernel on the bf16 instruction), and that leave them, with either
    split of the keys."""
    n = 400
    gen = torch.Generator().manual_seed(n + d)
    q, k, v = (torch.randn(heads, n, d, generator=gen) for _ in range(3))
    got = _attend_window("f32", d, heads, 1, 16, 25, q, k, v, wrapped=wrapped, token_stride=stride).double()
    ref = torch.softmax(q.double() @ k.double().transpose(1, 2) / math.sqrt(d), dim=2) @ v.double()
    assert float((got - ref).norm() / ref.norm()) <= 1e-6           # measured 2.3e-7
    _infinite_last_value("f32", d, heads, 1, 16, 25, wrapped=wrapped, token_stride=stride)
