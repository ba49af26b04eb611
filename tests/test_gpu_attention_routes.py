"""Which attention kernel a call takes, by the names of the launches of a trace, and the fp32 kernels that only steps reach: the split kernel over
several tiles and under run flags, the kernels with four shares of the keys."""
import math
import re

import pytest
import torch

import paper_2508_17756_amd as sg
from synthetic import TileGeometry, randn_tensor, torch_dtype
from test_gpu_f32_split import TOLERANCE

pytestmark = pytest.mark.gpu

LOG2E = math.log2(math.e)
CUS = 256   # the sizes below are chosen for this many compute units


@pytest.fixture(scope="module", autouse=True)
def _device():
    if torch.cuda.get_device_properties(0).multi_processor_count != CUS:
        pytest.skip("the sizes are those of a device with %d compute units" % CUS)


def _attention_kernels(call):
    """Names and template arguments of the attention kernels that a call launches."""
    from torch.profiler import ProfilerActivity, profile
    call()
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as trace:
        call()
        torch.cuda.synchronize()
    names = [e.key for e in trace.key_averages()]
    found = [re.search(r"(attention_\w+_kernel)(?:<([^>]*)>)?", n) for n in names]
    found = [(m.group(1), (m.group(2) or "").replace(" ", "")) for m in found if m]
    if not found and not any("sg::" in n for n in names):
        pytest.skip("no trace of kernels on this device")
    return sorted(found)


def _row(n_tiles, heads, T, th, tw, d, dtype, rows=1):
    return TileGeometry("row", T, rows * th, n_tiles // rows * tw, th, tw, th, tw, rows, n_tiles // rows, heads, d, dtype, 0)


class GatedStep:
    """A cached step of n tiles of one row, tile_x [n][3][heads][N][d] on the CPU: the tiles of `reused` have their own input cached."""

    def __init__(self, heads, T, th, tw, d, dtype, tile_x, reused):
        n = len(tile_x)
        self.g = g = _row(n, heads, T, th, tw, d, dtype)
        self.p = sg.make_problem(g)
        self.x = [x.reshape((3,) + g.tile_shape).to(torch_dtype(dtype)).cuda() for x in tile_x]
        self.reused = reused
        self.cache_x = [torch.full_like(x, 7.0) for x in self.x]
        self.out = [torch.full(g.tile_shape, 3.0, dtype=torch_dtype(dtype), device="cuda") for _ in range(n)]
        self.has_cache = torch.zeros(n, dtype=torch.uint8, device="cuda")
        self.scores = torch.zeros(n, device="cuda")
        self.recompute = torch.zeros(n, dtype=torch.uint8, device="cuda")
        self.canvas = torch.empty(g.grid_shape, dtype=torch_dtype(dtype), device="cuda")
        self.ws = torch.empty(sg.sg_workspace_bytes(n), dtype=torch.uint8, device="cuda")

    def __call__(self):
        self.has_cache.zero_()
        for i in self.reused:
            self.has_cache[i] = 1
            self.cache_x[i].copy_(self.x[i])
        sg.sg_denoise_step_tiled(self.p, self.canvas, self.out, tile_x=self.x, cache_x=self.cache_x, has_cache=self.has_cache, threshold=0.05,
                                 scores=self.scores, recompute=self.recompute, workspace=self.ws)

    def results(self):
        """Outputs [heads][N][d] of the tiles that ran; the others kept theirs."""
        self()
        n = len(self.x)
        assert self.recompute.tolist() == [int(i not in self.reused) for i in range(n)]
        for i in range(n):
            assert torch.equal(self.cache_x[i], self.x[i]) or self.x[i].isnan().any()
            if i in self.reused:
                assert bool((self.out[i] == 3.0).all())
        return [o.cpu().reshape(self.g.heads, -1, self.g.head_dim) for o in self.out]


class Window:
    """One tile read in place from a canvas of 2 x 2 tiles; a canvas of one tile where packed."""

    def __init__(self, heads, T, th, tw, d, dtype, shift=(0, 0), packed=False, token_stride=0):
        rows, cols = (1, 1) if packed else (2, 2)
        self.g = g = TileGeometry("one", T, rows * th, cols * tw, th, tw, th, tw, rows, cols, heads, d, dtype, 0)
        self.p = sg.make_problem(g, shift=shift)
        if token_stride:
            self.p.grid_stride_token, self.p.grid_stride_head = token_stride, d
            buf = torch.empty(g.grid_tokens * token_stride + 3 * heads * d, dtype=torch_dtype(dtype), device="cuda")
            self.qkv = [buf[i * heads * d:] for i in range(3)]
            for t in self.qkv:
                t.as_strided((heads, g.grid_tokens, d), (d, token_stride, 1)).normal_()
        else:
            self.qkv = [randn_tensor(g.grid_shape, dtype, 5 + i).cuda() for i in range(3)]
        self.out = torch.empty(g.tile_shape, dtype=torch_dtype(dtype), device="cuda")

    def __call__(self):
        sg.sg_tile_attention(self.p, *self.qkv, 0, 0, self.out)


def _gated(n, heads, T, th, tw, d, dtype):
    gen = torch.Generator().manual_seed(n + heads)
    x = [torch.randn(3, heads, T * th * tw, d, generator=gen) for _ in range(n)]
    return GatedStep(heads, T, th, tw, d, dtype, x, reused=[])


SPLIT, F32, BF16, STAGED = "attention_f32_split_kernel", "attention_f32_kernel", "attention_bf16_kernel", "attention_bf16_short_kernel"

# fp32: <head_dim, window> of the split kernel; <head_dim, blocks of 32 queries, shares of the keys, window, wide offsets> of the other
F32_ROUTES = [
    ("tiny", lambda: Window(2, 3, 10, 10, 64, "f32"), [(F32, "64,1,8,1,false")]),
    ("split_packed_64", lambda: Window(200, 1, 5, 13, 64, "f32", packed=True), [(SPLIT, "64,0")]),
    ("split_window_64", lambda: Window(30, 2, 17, 20, 64, "f32", shift=(3, 5)), [(SPLIT, "64,1")]),
    ("split_packed_128", lambda: Window(51, 7, 10, 10, 128, "f32", packed=True), [(SPLIT, "128,0")]),
    ("split_window_128", lambda: Window(120, 1, 3, 43, 128, "f32"), [(SPLIT, "128,1")]),
    ("split_wide_strides", lambda: Window(48, 1, 16, 25, 128, "f32", token_stride=1 << 19), [(SPLIT, "128,1")]),
    ("beyond_4_gib", lambda: Window(48, 1, 16, 25, 128, "f32", token_stride=1 << 20), [(F32, "128,1,4,1,true")]),
    ("split_gated_64", lambda: _gated(4, 250, 1, 9, 11, 64, "f32"), [(SPLIT, "64,0")]),
    ("split_gated_128", lambda: _gated(4, 250, 1, 9, 11, 128, "f32"), [(SPLIT, "128,0")]),
    ("gated_64_queries", lambda: _gated(9, 12, 1, 16, 25, 64, "f32"), [(F32, "64,2,4,0,false")]),
    ("gated_32_queries_64", lambda: _gated(8, 5, 1, 16, 25, 64, "f32"), [(F32, "64,1,4,0,false")]),
    ("gated_32_queries_128", lambda: _gated(9, 12, 1, 16, 25, 128, "f32"), [(F32, "128,1,4,0,false")]),
    ("window_64_queries", lambda: Window(512, 1, 7, 9, 64, "f32"), [(F32, "64,2,4,1,false")]),
    ("window_32_queries_64", lambda: Window(600, 1, 7, 9, 64, "f32"), [(F32, "64,1,4,1,false")]),
    ("window_32_queries_128", lambda: Window(600, 1, 7, 9, 128, "f32"), [(F32, "128,1,4,1,false")]),
]

# bf16: <head_dim, packed 0 | planned 1 | walked 2, scaled behind the product, refresh, few stages>
BF16_ROUTES = [
    ("packed_128", lambda: Window(2, 1, 48, 32, 128, "bf16", packed=True), [(BF16, "128,0,false,false,true")]),
    ("packed_128_long", lambda: Window(2, 1, 53, 29, 128, "bf16", packed=True), [(BF16, "128,0,false,false,false")]),
    ("walked", lambda: Window(2, 1, 48, 32, 128, "bf16"), [(BF16, "128,2,false,false,true")]),
    ("walked_long", lambda: Window(2, 1, 56, 32, 128, "bf16"), [(BF16, "128,2,false,false,false")]),
    ("planned", lambda: Window(2, 1, 48, 32, 128, "bf16", shift=(50, 3)), [(BF16, "128,1,false,false,true")]),
    ("planned_long", lambda: Window(2, 1, 56, 32, 128, "bf16", shift=(60, 3)), [(BF16, "128,1,false,false,false")]),
    ("planned_wide", lambda: Window(1, 2, 10, 21, 128, "bf16", token_stride=1 << 21), [(BF16, "128,1,true,false,true")]),
    ("planned_wide_long", lambda: Window(1, 4, 20, 21, 128, "bf16", token_stride=1 << 19), [(BF16, "128,1,true,false,false")]),
    ("refresh_128", lambda: _gated(2, 2, 1, 48, 32, 128, "bf16"), [(BF16, "128,0,false,true,true")]),
    ("refresh_128_long", lambda: _gated(2, 2, 1, 53, 29, 128, "bf16"), [(BF16, "128,0,false,true,false")]),
    ("packed_64", lambda: Window(2, 1, 32, 64, 64, "bf16", packed=True), [(BF16, "64,0,false,false,true")]),
    ("packed_64_long", lambda: Window(2, 1, 3, 683, 64, "bf16", packed=True), [(BF16, "64,0,false,false,false")]),
    ("refresh_64", lambda: _gated(2, 2, 2, 32, 48, 64, "bf16"), [(BF16, "64,0,false,true,true")]),
    ("refresh_64_long", lambda: _gated(2, 2, 1, 7, 439, 64, "bf16"), [(BF16, "64,0,false,true,false")]),
    ("window_64", lambda: Window(2, 2, 32, 48, 64, "bf16"), [(BF16, "64,1,true,false,true")]),
    ("window_64_long", lambda: Window(2, 1, 7, 439, 64, "bf16"), [(BF16, "64,1,true,false,false")]),
]


@pytest.mark.parametrize("name,call,kernels", F32_ROUTES + BF16_ROUTES, ids=[r[0] for r in F32_ROUTES + BF16_ROUTES])
def test_a_call_takes_its_kernel(name, call, kernels):
    assert _attention_kernels(call()) == kernels


@pytest.mark.parametrize("heads,tokens,kernel", [(2, 448, STAGED), (2, 464, BF16), (65, 960, STAGED), (32, 960, BF16), (65, 976, BF16)])
def test_windows_of_head_dim_64_with_few_keys(heads, tokens, kernel):
    """Up to 448 tokens the register-staged kernel, up to 960 where there are workgroups for more than half of the compute units."""
    assert [n for n, _ in _attention_kernels(Window(heads, 1, 16, tokens // 16, 64, "bf16"))] == [kernel]


@pytest.mark.parametrize("d,heads,th,tw,kernel", [
    (64, 200, 5, 13, SPLIT), (64, 342, 5, 13, F32), (64, 769, 5, 13, F32), (64, 512, 3, 43, F32), (64, 512, 8, 12, F32), (64, 257, 8, 25, F32),
    (64, 257, 1, 97, F32), (64, 640, 1, 97, SPLIT), (64, 385, 7, 23, SPLIT), (64, 192, 16, 16, SPLIT), (64, 129, 16, 16, F32),
    (128, 200, 5, 13, SPLIT), (128, 769, 5, 13, F32), (128, 257, 8, 16, F32), (128, 769, 1, 97, SPLIT), (128, 359, 3, 43, SPLIT)])
def test_fp32_calls_of_several_rounds_of_short_tiles(d, heads, th, tw, kernel):
    """One round of 128-query workgroups goes to the split kernel; several of up to 256 tokens only where they hide its start and end."""
    w = Window(heads, 1, th, tw, d, "f32", packed=True)
    assert [n for n, _ in _attention_kernels(w)] == [kernel]
    assert _rel(w.out.cpu().reshape(heads, -1, d), _exact([t.cpu().reshape(heads, -1, d) for t in w.qkv], _fp32_scale(d))) <= TOLERANCE


def _exact(x, scale):
    q, k, v = (t.double() for t in x)
    out = torch.empty(q.shape, dtype=torch.float64)
    for a in range(q.shape[0]):
        out[a] = torch.softmax(q[a] @ k[a].T * scale, dim=1) @ v[a]
    return out


def _rel(got, want):
    return float(((got.double() - want).flatten(1).norm(dim=1) / want.flatten(1).norm(dim=1)).max())


def _fp32_scale(d):
    return float(torch.tensor(1.0 / math.sqrt(d)))


# ---- the split kernel over several tiles and under run flags
@pytest.mark.parametrize("reused", [[], [1], [0, 3]], ids=["all", "one_reused", "two_reused"])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("th,tw", [(9, 11), (8, 16)])
def test_split_kernel_attends_the_active_tiles(th, tw, d, reused):
    """Tile 2 holds values that the parts do not (one head of it), beside tiles of ordinary numbers; reused tiles are skipped."""
    heads = 250
    gen = torch.Generator().manual_seed(d + th)
    x = [torch.randn(3, heads, th * tw, d, generator=gen) for _ in range(4)]
    x[2][2, 7] *= 2.0 ** 100
    step = GatedStep(heads, 1, th, tw, d, "f32", x, reused)
    got = step.results()
    for i in range(4):
        if i not in reused:
            assert _rel(got[i], _exact(x[i], _fp32_scale(d))) <= TOLERANCE
    assert _attention_kernels(step) == [(SPLIT, "%d,0" % d)]


@pytest.mark.parametrize("shift", [(0, 0), (5, 9)], ids=["fixed", "wrapped"])
@pytest.mark.parametrize("d", [64, 128])
def test_split_kernel_attends_overlapping_tiles_of_a_canvas(d, shift):
    """2 x 3 tiles of 1 x 13 x 10 tokens that share rows and columns, 21 heads: one launch, two workgroups a head, the second with two
    queries; a value that the parts do not hold lies in some of the windows only."""
    heads = 21
    g = TileGeometry("over", 1, 20, 24, 13, 10, 7, 7, 2, 3, heads, d, "f32", 0)
    qkv = [randn_tensor(g.grid_shape, "f32", 40 + i) for i in range(3)]
    qkv[2][5, 0, 9, 16, 3] = 2.0 ** 90
    dev = [t.cuda() for t in qkv]
    out = [torch.empty(g.tile_shape, device="cuda") for _ in range(g.n_tiles)]
    canvas = torch.empty(g.grid_shape, device="cuda")
    p = sg.make_problem(g, shift=shift)

    def step():
        sg.sg_denoise_step_tiled(p, canvas, out, q=dev[0], k=dev[1], v=dev[2])

    step()
    for i in range(g.n_tiles):
        y0, x0 = i // 3 * 7 + shift[0], i % 3 * 7 + shift[1]
        ys, xs = [(y0 + y) % 20 for y in range(13)], [(x0 + c) % 24 for c in range(10)]
        x = [t[:, :, ys][:, :, :, xs].reshape(heads, -1, d) for t in qkv]
        assert _rel(out[i].cpu().reshape(heads, -1, d), _exact(x, _fp32_scale(d))) <= TOLERANCE, i
    assert _attention_kernels(step) == [(SPLIT, "%d,1" % d)]


# ---- four shares of the keys: 400 tokens are 13 blocks of 32 keys, dealt to the shares in turn
def _growing(x, d):
    u = torch.nn.functional.normalize(randn_tensor((d,), "f32", 5), dim=0)
    x[0].mul_(0.3).add_(8.0 * u)
    x[1].mul_(0.3).add_((12.0 * math.sqrt(d) / 8.0) * torch.linspace(0.0, 1.0, x.shape[2])[:, None] * u)


def _large_values(x, d):
    """Scores that rise by 4.9 at key 261, in block 8 of share 0."""
    x.zero_()
    x[0, :, :, 0] = math.sqrt(d)
    x[1, :, 261, 0] = 4.9
    x[2, :, 261] = 3e38


def _small_probability(x, d):
    x.zero_()
    x[0, :, :, 0] = math.sqrt(d)
    x[1, :, :, 0] = -200.0
    x[1, :, 0, 0] = 0.0
    x[1, :, 261, 0] = -90.0
    x[2, :, 261] = 3e38


def _block_at_minus_infinity(x, d):
    x[0, :, :, 7] = 1e20
    x[1, :, :, 7] = 0.0
    x[1, :, 128:160, 7] = -1e20


def _infinite_last_value(x, d):
    x[2, :, -1, 3] = math.inf


def _nan(x, d):
    x[0, 0, 11, 0] = x[1, 1, 399, 1] = x[2, 2, 2, 9] = math.nan


CONTENTS = [_growing, _large_values, _small_probability, _block_at_minus_infinity, _infinite_last_value, _nan]


@pytest.mark.parametrize("d,heads,n,kernel", [(64, 12, 9, "64,2,4,0,false"), (64, 5, 8, "64,1,4,0,false"), (128, 12, 9, "128,1,4,0,false")])
def test_four_shares_of_the_keys(d, heads, n, kernel):
    """What the kernels with eight shares are tested for at one head: scores that grow from block to block, values up to the largest number,
    probabilities below the normal range, a block of scores at -inf, an infinite last value, NaN; one tile of each, a plain one, the others reused."""
    T, th, tw = 1, 16, 25
    gen = torch.Generator().manual_seed(d + n)
    x = [torch.randn(3, heads, th * tw, d, generator=gen) for _ in range(n)]
    for i, put in enumerate(CONTENTS):
        put(x[i], d)
    step = GatedStep(heads, T, th, tw, d, "f32", x, reused=list(range(7, n)))
    got = step.results()
    scale = _fp32_scale(d)
    assert _rel(got[6], _exact(x[6], scale)) <= 1e-6
    # the logits reach 12, and their rounding, a few times 12 * 2^-24, is the relative error of the probabilities
    assert _rel(got[0], _exact(x[0], scale)) <= 1e-5
    want = 3e38 * math.exp(4.9) / (math.exp(4.9) + th * tw - 1)
    assert float((got[1].double() / want - 1.0).abs().max()) <= 1e-5
    # the rounding of the exponent (130 +- 2^-17) and of the probability (2^-150) allow 7e-6
    assert float((got[2].double() / (3e38 * math.exp(-90.0)) - 1.0).abs().max()) <= 1.2e-5
    q, k, v = (t.double() for t in x[3])
    s = q @ k.transpose(1, 2).contiguous() / math.sqrt(d)
    s[:, :, 128:160] = -math.inf
    assert _rel(got[3], torch.softmax(s, dim=2) @ v) <= 1e-5
    assert bool((got[4][:, :, 3] == math.inf).all())
    got[4][:, :, 3] = 0.0
    assert bool(torch.isfinite(got[4]).all())
    nans = torch.zeros(heads, th * tw, d, dtype=torch.bool)
    nans[0, 11] = True
    nans[1] = True
    nans[2, :, 9] = True
    assert torch.equal(got[5].isnan(), nans)
    assert _attention_kernels(step) == [(F32, kernel)]


@pytest.mark.parametrize("d,heads", [(64, 512), (64, 600), (128, 600)])
@pytest.mark.parametrize("shift", [(0, 0), (11, 13)], ids=["fixed", "wrapped"])
def test_four_shares_of_the_keys_in_windows(d, heads, shift):
    """63 tokens, two blocks of keys: two of the four shares have none; the last value is infinite in channel 3 of head 9."""
    w = Window(heads, 1, 7, 9, d, "f32", shift=shift)
    ys, xs = [(shift[0] + y) % 14 for y in range(7)], [(shift[1] + c) % 18 for c in range(9)]
    w.qkv[2][9, 0, ys[-1], xs[-1], 3] = math.inf
    w()
    x = [t.cpu()[:, :, ys][:, :, :, xs].reshape(heads, -1, d) for t in w.qkv]
    got = w.out.cpu().reshape(heads, -1, d)
    assert bool((got[9, :, 3] == math.inf).all())
    got[9, :, 3] = 0.0
    x[2][9, -1, 3] = 0.0
    want = _exact(x, _fp32_scale(d))
    want[9, :, 3] = 0.0
    assert _rel(got, want) <= 1e-6
