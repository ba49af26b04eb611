"""GPU parity of the region-aware threshold control (sg_tile_std, sg_region_thresholds) against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2508_17756_amd as sg
from synthetic import randn_tensor, torch_dtype, perturb_
from gpu_util import to_f64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("elems", [8, 4096 + 8, 2 * 3 * 10 * 10 * 64, 1 << 21])
def test_tile_std_small(dtype, elems):
    n = 5
    scale = [1.0, 0.01, 3.0, 1.0, 0.0]
    shift = [0.0, 0.0, -2.0, 50.0, 1.5]          # tile 3: mean far from zero; tile 4: constant
    x = [(randn_tensor((elems,), "f32", 40 + i) * scale[i] + shift[i]).to(torch_dtype(dtype)).cuda() for i in range(n)]
    out = torch.full((n,), -1.0, dtype=torch.float32, device="cuda")
    ws = torch.empty(sg.sg_workspace_bytes(n), dtype=torch.uint8, device="cuda")
    sg.sg_tile_std(x, out, ws)
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    for i in range(n):
        ref = oracle.tile_std(to_f64(x[i]))
        assert abs(got[i] - ref) <= 2e-5 * max(ref, 1e-3), (i, got[i], ref)
    assert got[4] == 0.0


@pytest.mark.parametrize("mode", ["MaxMin", "TopSelect"])
def test_region_thresholds_follow_algorithm_2(mode):
    """Eight steps, thresholds adjusted every third step: the device tracker and policy against the
    oracle's, both fed the same stored per-step standard deviations."""
    n, tau, alpha, every = 7, 0.05, 0.4, 3
    code = sg.SG_REGION_MAXMIN if mode == "MaxMin" else sg.SG_REGION_TOPSELECT
    rng = np.random.default_rng(7)
    track_mean = torch.full((n,), 123.0, dtype=torch.float64, device="cuda")     # garbage: the first update overwrites it
    track_count = torch.zeros(1, dtype=torch.int32, device="cuda")
    thr = torch.full((n,), -1.0, dtype=torch.float32, device="cuda")
    sigma = torch.full((n,), -1.0, dtype=torch.float32, device="cuda")
    tr = oracle.StdTracker(n)
    ref_thr = np.full(n, float(np.float32(tau)))
    for s in range(1, 9):
        stds = torch.tensor(rng.random(n) + 0.1, dtype=torch.float32)
        if s == 5:
            stds[2] = stds[4]                                                     # a tie on this step's values
        adjust = s % every == 0
        sg.sg_region_thresholds(stds.cuda(), track_mean, track_count, tau, alpha, code, adjust, thr, sigma=sigma)
        torch.cuda.synchronize()
        tr.update(stds.numpy().astype(np.float64))
        if adjust:
            ref_thr = oracle.region_thresholds(tr.normalized(), float(np.float32(tau)), float(np.float32(alpha)), mode)
            np.testing.assert_allclose(sigma.cpu().numpy(), tr.normalized(), rtol=0, atol=1e-6)
        np.testing.assert_array_equal(track_mean.cpu().numpy(), tr.mean)          # same fp64 recurrence
        np.testing.assert_allclose(thr.cpu().numpy(), ref_thr, rtol=1e-6)
        assert int(track_count.item()) == s


def test_region_thresholds_edge_cases():
    def run(stds, mode, adjust=True, tau=1.0, alpha=0.2):
        n = len(stds)
        tm = torch.zeros(n, dtype=torch.float64, device="cuda")
        tc = torch.zeros(1, dtype=torch.int32, device="cuda")
        thr = torch.full((n,), -1.0, dtype=torch.float32, device="cuda")
        sg.sg_region_thresholds(torch.tensor(stds, dtype=torch.float32, device="cuda"), tm, tc, tau, alpha, mode, adjust, thr)
        torch.cuda.synchronize()
        return thr.cpu().numpy()
    np.testing.assert_allclose(run([0.5, 0.9, 0.9, 0.1, 0.1], sg.SG_REGION_MAXMIN), [1, 1.2, 1, 0.9, 1], rtol=1e-6)
    np.testing.assert_allclose(run([0.5, 0.9, 0.9, 0.1, 0.1], sg.SG_REGION_TOPSELECT), [1, 1.2, 1.1, 1, 1], rtol=1e-6)
    np.testing.assert_allclose(run([0.3, 0.3], sg.SG_REGION_MAXMIN), [0.9, 1.0], rtol=1e-6)     # all equal
    np.testing.assert_allclose(run([0.3], sg.SG_REGION_TOPSELECT), [1.2], rtol=1e-6)            # one tile
    np.testing.assert_allclose(run([0.3, 0.7, 0.1], sg.SG_REGION_MAXMIN, adjust=False), [1, 1, 1], rtol=1e-6)
    big = list(np.linspace(0.1, 0.9, 300))                                                        # more tiles than threads
    got = run(big, sg.SG_REGION_TOPSELECT)
    assert got[299] == np.float32(1.2) and got[298] == np.float32(1.1) and (got[:298] == 1.0).all()


def test_std_tracker_drives_the_gain_gate_thresholds():
    """The thresholds produced here are what sg_gain_gate consumes: a tile whose threshold was raised
    reuses where its neighbour with the same score recomputes."""
    n, elems = 3, 4096
    prev = [randn_tensor((elems,), "bf16", 70 + i).cuda() for i in range(n)]
    cur = [(p.float() * 1.0625).to(torch.bfloat16) for p in prev]                 # every tile: d = 1/16 up to bf16 rounding
    state = sg.GainState(n)
    state.has_prev.fill_(1)
    state.has_gain.fill_(1)
    state.gain.fill_(1.0)
    tm = torch.zeros(n, dtype=torch.float64, device="cuda")
    tc = torch.zeros(1, dtype=torch.int32, device="cuda")
    thr = torch.empty(n, dtype=torch.float32, device="cuda")
    sg.sg_region_thresholds(torch.tensor([0.2, 0.8, 0.5], device="cuda"), tm, tc, 0.05, 0.4, sg.SG_REGION_MAXMIN, True, thr)
    step = torch.empty(n, dtype=torch.float32, device="cuda")
    scores = torch.empty(n, dtype=torch.float32, device="cuda")
    rec = torch.empty(n, dtype=torch.uint8, device="cuda")
    ws = torch.empty(sg.sg_workspace_bytes(n), dtype=torch.uint8, device="cuda")
    sg.sg_gain_gate(cur, prev, state, 0.05, step, scores, rec, ws, tile_thresholds=thr)
    torch.cuda.synchronize()
    assert all(abs(v - 0.0625) < 1e-3 for v in scores.cpu().tolist())             # thresholds 0.04, 0.07, 0.05
    assert rec.cpu().tolist() == [1, 0, 1]


# ------------------------------------------------------------------ similarity pair of Equation 3
def _similarity(x_new, x_old):
    n = len(x_new)
    l1 = torch.full((max(n, 1),), -5.0, dtype=torch.float32, device="cuda")
    cs = torch.full((max(n, 1),), -5.0, dtype=torch.float32, device="cuda")
    ws = torch.empty(sg.sg_workspace_bytes(n), dtype=torch.uint8, device="cuda")
    sg.sg_tile_similarity(x_new, x_old, l1, cs, ws)
    torch.cuda.synchronize()
    return l1.cpu().numpy()[:n], cs.cpu().numpy()[:n]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("elems", [8, 1000, 4099, 3 * 2 * 3 * 10 * 10 * 64, (1 << 20) + 3])
def test_similarity_against_the_oracle(dtype, elems):
    """Relative L1 distance and cosine similarity (Equation 3) of five tile pairs: identical, barely moved, moved,
    opposite, unrelated; element counts that are ragged against the 16-byte vectors and against the workgroups."""
    n = 5
    old = [randn_tensor((elems,), dtype, 2100 + i).cuda() for i in range(n)]
    new = [old[0].clone(), perturb_(old[1].clone(), 0.01, 2201), perturb_(old[2].clone(), 0.5, 2202), -old[3],
           randn_tensor((elems,), dtype, 2204).cuda()]
    l1, cs = _similarity(new, old)
    for i in range(n):
        ref_l1, ref_cs = oracle.similarity(to_f64(new[i]), to_f64(old[i]))
        assert abs(l1[i] - ref_l1) <= 2e-6 * max(1.0, ref_l1), (i, l1[i], ref_l1)
        assert abs(cs[i] - ref_cs) <= 3e-6, (i, cs[i], ref_cs)
    assert l1[0] == 0.0 and abs(cs[0] - 1.0) <= 3e-6 and abs(cs[3] + 1.0) <= 3e-6 and abs(l1[3] - 2.0) <= 4e-6


def test_similarity_zero_tensors_many_tiles_and_arguments():
    x = randn_tensor((4096,), "bf16", 2300).cuda()
    z = torch.zeros_like(x)
    l1, cs = _similarity([x, z, z], [z, x, z])
    assert np.isinf(l1[0]) and cs[0] == 0.0 and l1[1] == 1.0 and cs[1] == 0.0 and np.isinf(l1[2]) and cs[2] == 0.0
    n = 70                                                           # more than one launch's table of pointers
    old = [randn_tensor((2048,), "bf16", 2400 + i).cuda() for i in range(n)]
    new = [perturb_(t.clone(), 0.05 * (1 + i % 4), 2500 + i) for i, t in enumerate(old)]
    l1, cs = _similarity(new, old)
    for i in (0, 1, 63, 64, 69):
        ref_l1, ref_cs = oracle.similarity(to_f64(new[i]), to_f64(old[i]))
        assert abs(l1[i] - ref_l1) <= 2e-6 * max(1.0, ref_l1) and abs(cs[i] - ref_cs) <= 3e-6, i
    _similarity([], [])
    with pytest.raises(sg.SgError) as e:
        sg.sg_tile_similarity([x], [x], torch.empty(1, device="cuda"), torch.empty(1, device="cuda"),
                              torch.empty(16, dtype=torch.uint8, device="cuda"))
    assert e.value.status == sg.SG_ERR_WORKSPACE


def _probes(n, width, seed):
    """Zeros but for integers 8 .. 15 in vectors where a pass may go wrong: both ends of every run of 256 (threads; unrolled steps and
    chunks end there too), of every workgroup's slab under either rule of cutting, when walked and when three tiles share the device, a few
    hundred more, the last vector and every element of the tail behind it.  Element 0 stays 0: the deviation's pivot."""
    vecs = n // width
    at = set(range(0, vecs, 256)) | set(range(255, vecs, 256)) | {vecs - 1}
    for blocks in {-(-vecs // 4096), -(-vecs // 2048), 256, 85}:
        slab = -(-vecs // blocks)
        at |= {v for b in range(blocks + 1) for v in (b * slab - 1, b * slab) if 0 <= v < vecs}
    rng = np.random.default_rng(seed)
    at = np.array(sorted(at | set(rng.integers(0, vecs, 300).tolist())))
    where = np.concatenate([at * width + 1 + rng.integers(0, width - 1, at.size), np.arange(vecs * width, n)])
    x = torch.zeros(n, dtype=torch.float32)
    x[torch.from_numpy(where)] = torch.from_numpy(rng.integers(8, 16, where.size).astype(np.float32))
    return x.cuda()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("count", [1, 3])
@pytest.mark.parametrize("vecs", [5, 1000, 2047, 2048, 2049, 4095, 4096, 4097, 3 * 4096, 255 * 2048, 255 * 2048 + 1, 256 * 2048 + 7,
                                  255 * 4096, 255 * 4096 + 1, 256 * 4096 + 7])
def test_passes_over_tiles_cut_side_by_side_or_walked(dtype, vecs, count):
    """Both grids of the streaming passes around the sizes where they change (4,096 vectors per workgroup, 2,048 in the gain refresh, a
    device of 256 compute units), over one tile and three, which share the compute units: every element is counted exactly once.  Each sum is carried by a few thousand
    probes (at most 11,000, of 8 to 15, on a background of zeros), so that one lost or repeated changes the results, which are ratios
    and square roots of the sums, by 1e-5 of themselves or more.  All terms are small integers: the sums are exact, the results
    rounded once (2^-24)."""
    width = 8 if dtype == "bf16" else 4
    dt = torch_dtype(dtype)
    n = (vecs * width + 7) // 8 * 8
    ws = torch.empty(sg.sg_workspace_bytes(count), dtype=torch.uint8, device="cuda").fill_(255)
    f = lambda: torch.full((count,), float("nan"), device="cuda")
    has = torch.ones(count, dtype=torch.uint8, device="cuda")

    def near(got, want, what):
        assert abs(float(got) - want) <= 2e-6 * want, (what, float(got), want)

    # change: probes that differ from a background of ones; level: all ones away from a background of probes
    for kind in ("change", "level"):
        for tail in (0, 3):                                  # gate and similarity also take a ragged end
            probes = [_probes(n + tail, width, 17 * i + vecs) for i in range(count)]
            olds = [torch.ones_like(p).to(dt) if kind == "change" else p.to(dt) for p in probes]
            tiles = [(p + 1).to(dt) for p in probes]
            l1, cs, scores, rec = f(), f(), f(), torch.empty(count, dtype=torch.uint8, device="cuda")
            sg.sg_tile_similarity(tiles, olds, l1, cs, ws)
            sg.sg_cache_gate(tiles, olds, has, 0.5, scores, rec, ws)
            for i, (x, y) in enumerate(zip(tiles, olds)):
                x, y = x.double(), y.double()
                want = float((x - y).abs().sum() / y.abs().sum())
                near(l1[i], want, ("l1", kind, tail, i))
                near(scores[i], want, ("gate", kind, tail, i))
                if kind == "level":
                    near(cs[i], float((x * y).sum() / (x.norm() * y.norm())), ("cosine", tail, i))
        probes = [_probes(n, width, 17 * i + vecs) for i in range(count)]
        olds = [torch.ones_like(p).to(dt) if kind == "change" else p.to(dt) for p in probes]
        tiles = [(p + 1).to(dt) for p in probes]
        std = f()
        sg.sg_tile_std([p.to(dt) for p in probes], std, ws)
        state = sg.GainState(count)
        state.has_prev.fill_(1)
        out = [t.clone() for t in tiles]
        delta = [torch.full((n,), 9.0, device="cuda") for _ in tiles]
        recompute = torch.tensor([1, 0, 1][:count], dtype=torch.uint8, device="cuda")
        change = torch.full((count,), 0.25, device="cuda")
        sg.sg_gain_refresh(out, olds, olds, delta, recompute, change, state, ws)
        for i, (x, y) in enumerate(zip(tiles, olds)):
            near(std[i], float(probes[i].double().std(unbiased=False)), ("std", i))
            if recompute[i]:
                assert torch.equal(delta[i], x.float() - y.float()) and torch.equal(out[i], x)
                near(state.gain[i], float((x.double() - y.double()).abs().sum() / y.double().abs().sum()) / 0.25, ("gain", kind, i))
            else:
                assert torch.equal(delta[i], torch.full((n,), 9.0, device="cuda"))
                assert torch.equal(out[i], (y.float() + 9.0).to(dt))


def test_sums_of_small_tiles_are_rounded_once():
    """bf16 tiles of 64 KiB to 4 MiB: standard deviation and cosine are fp64 sums of fp32 sums of 8 elements each, whose roundings
    average out, so each is the exact value rounded once: half a unit in the last place of values just above and just
    below 1 (2^-24 and 2^-25), a fifth more for the sums."""
    for vecs in (1 << 12, 1 << 14, 1 << 16, 1 << 18):
        old = [randn_tensor((8 * vecs,), "bf16", 3000 + i).cuda() for i in range(12)]
        new = [perturb_(x.clone(), 0.1, 3100 + i) for i, x in enumerate(old)]
        ws = torch.empty(sg.sg_workspace_bytes(12), dtype=torch.uint8, device="cuda")
        std, l1, cs = (torch.empty(12, device="cuda") for _ in range(3))
        sg.sg_tile_std(new, std, ws)
        sg.sg_tile_similarity(new, old, l1, cs, ws)
        for i in range(12):
            a, b = new[i].double(), old[i].double()
            want_std, want_cos = float(a.std(unbiased=False)), float((a * b).sum() / (a.norm() * b.norm()))
            assert 0.98 < want_std < 1.03 and 0.99 < want_cos < 1.0
            assert abs(float(std[i]) - want_std) <= 1.2 * 2 ** -24, (vecs, i)
            assert abs(float(cs[i]) - want_cos) <= 1.2 * 2 ** -25, (vecs, i)
