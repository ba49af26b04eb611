"""fp32 attention on the bf16 matrix instruction (three bf16 parts of every number): taken where the rounds of 128-query workgroups over the
device are short against those of 32-query ones, here with 200 heads of few tokens."""
import math

import pytest
import torch

from test_gpu_extremes import _attend_window

pytestmark = pytest.mark.gpu

HEADS = 200    # 256 compute units: one round of 128-query workgroups, three of 32-query ones, up to 128 tokens


def _inputs(heads, n, d):
    gen = torch.Generator().manual_seed(1000 * d + n)
    return [torch.randn(heads, n, d, generator=gen) for _ in range(3)]


def _exact(q, k, v):
    out = torch.empty(q.shape, dtype=torch.float64)
    for a in range(q.shape[0]):
        # the scale as the library gets it, rounded to fp32
        w = torch.softmax(q[a].double() @ k[a].double().T * float(torch.tensor(1.0 / math.sqrt(q.shape[2]))), dim=1)
        out[a] = w @ v[a].double()
    return out


def _rel(got, want):
    """Largest relative 2-norm error of a head."""
    return float(((got.double() - want).flatten(1).norm(dim=1) / want.flatten(1).norm(dim=1)).max())


# Every fp32 sum of products of first parts is rounded d/16 (scores) or n/16 (outputs) times by at most half a unit, 2^-24: as a
# random walk of uniform errors sqrt((8 + n/16) / 3) 2^-24, under 3e-7 at 700 tokens; what the parts leave out of every product (2^-24 at most,
# 2^-27.4 in the mean square), products of scores' errors with the scores (up to 5) and the exponential's own 2^-22 double that.
TOLERANCE = 6e-7


@pytest.mark.parametrize("where", ["packed", "fixed", "wrapped"])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("heads,T,th,tw", [
    (HEADS, 1, 5, 13),      # 65: three stages of 32 keys or two of 64, the last with one key
    (HEADS, 1, 8, 12),      # 96: whole stages of 32 keys
    (HEADS, 1, 8, 16),      # 128: whole stages, whole workgroup
    (120, 1, 3, 43),        # 129: a second workgroup with one query
    (40, 2, 16, 16),        # 512: 16 or 8 whole stages
    (40, 3, 9, 19),         # 513: the range is looked at again behind 16 stages, with one stage left
    (30, 2, 17, 20),        # 680: behind 16 stages in the middle
    (51, 7, 10, 10),        # 700
])
def test_sizes(heads, T, th, tw, d, where):
    n = T * th * tw
    q, k, v = _inputs(heads, n, d)
    got = _attend_window("f32", d, heads, T, th, tw, q, k, v, wrapped=where == "wrapped", packed=where == "packed")
    assert _rel(got, _exact(q, k, v)) <= TOLERANCE


def _put(x, head, tokens, factor):
    x[head, tokens] = x[head, tokens] * factor


# head 7 holds numbers that the parts do not; its neighbours do not
OUT = {
    "large_values": lambda q, k, v: _put(v, 7, slice(None), 2.0 ** 100),
    "one_large_value_in_the_last_stage": lambda q, k, v: _put(v, 7, -1, 2.0 ** 64),
    "tiny_values": lambda q, k, v: _put(v, 7, slice(None), 2.0 ** -112),
    "one_tiny_value": lambda q, k, v: _put(v, 7, 40, 2.0 ** -112),
    "large_keys": lambda q, k, v: (_put(k, 7, slice(None), 2.0 ** 62), _put(q, 7, slice(None), 2.0 ** -62)),
    "large_queries": lambda q, k, v: (_put(q, 7, slice(None), 2.0 ** 70), _put(k, 7, slice(None), 2.0 ** -70)),
    "one_large_query": lambda q, k, v: (_put(q, 7, -1, 2.0 ** 70), _put(k, 7, slice(None), 2.0 ** -69)),
    "zero_values": lambda q, k, v: _put(v, 7, slice(0, 50), 0.0),
}


@pytest.mark.parametrize("name", sorted(OUT))
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("heads,T,th,tw", [(HEADS, 1, 5, 13), (30, 2, 17, 20)])
def test_numbers_that_the_parts_do_not_hold(heads, T, th, tw, d, name):
    n = T * th * tw
    q, k, v = _inputs(heads, n, d)
    OUT[name](q, k, v)
    got = _attend_window("f32", d, heads, T, th, tw, q, k, v)
    assert _rel(got, _exact(q, k, v)) <= TOLERANCE


@pytest.mark.parametrize("name", ["large_keys", "large_values", "one_large_value_in_the_last_stage"])
@pytest.mark.parametrize("where", ["packed", "fixed", "wrapped"])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("heads,T,th,tw", [(120, 1, 3, 43), (51, 7, 10, 10)])
def test_numbers_that_the_parts_do_not_hold_in_packed_and_wrapped_tiles(heads, T, th, tw, d, where, name):
    """129 tokens: one query in the last workgroup, of whose four blocks of 32 only the first is done over; 700: 60 in three blocks."""
    q, k, v = _inputs(heads, T * th * tw, d)
    OUT[name](q, k, v)
    got = _attend_window("f32", d, heads, T, th, tw, q, k, v, wrapped=where == "wrapped", packed=where == "packed")
    assert _rel(got, _exact(q, k, v)) <= TOLERANCE


# The ends of the range that the parts hold: 2^-100 <= |v| < 2^60 for values that are not 0, scaled queries and keys below 2^60
IN = {
    "smallest_values": lambda q, k, v: v[7].copy_(torch.sign(v[7]) * (1.0 + v[7].abs().fmod(1.0)) * 2.0 ** -100),
    "largest_values": lambda q, k, v: v[7].copy_(torch.sign(v[7]) * (1.0 + v[7].abs().fmod(1.0)) * 2.0 ** 58),
    "large_keys": lambda q, k, v: (_put(k, 7, slice(None), 2.0 ** 57), _put(q, 7, slice(None), 2.0 ** -57)),
    "large_queries": lambda q, k, v: (_put(q, 7, slice(None), 2.0 ** 59), _put(k, 7, slice(None), 2.0 ** -59)),
}


@pytest.mark.parametrize("name", sorted(IN))
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("heads,T,th,tw", [(HEADS, 1, 5, 13), (30, 2, 17, 20)])
def test_the_ends_of_the_range_that_the_parts_hold(heads, T, th, tw, d, name):
    q, k, v = _inputs(heads, T * th * tw, d)
    IN[name](q, k, v)
    got = _attend_window("f32", d, heads, T, th, tw, q, k, v)
    assert _rel(got, _exact(q, k, v)) <= TOLERANCE


@pytest.mark.parametrize("d", [64, 128])
def test_probabilities_below_the_smallest_normal_number_count(d):
    """Key 0 has a score 133 below the others' in the log2 domain, and values of 2^100: the products, 2^-33, are all that channel 0 holds."""
    n = 96
    q, k, v = _inputs(HEADS, n, d)
    q[7], k[7] = 0.0, 0.0
    q[7, :, 0] = 1.0
    k[7, 0, 0] = -133.0 / math.log2(math.e) * math.sqrt(d)
    v[7, 1:, 0] = 0.0
    v[7, 0] = 2.0 ** 100
    want = _exact(q, k, v)
    got = _attend_window("f32", d, HEADS, 1, 8, 12, q, k, v)
    # the probability is a multiple of 2^-149: half a unit at 2^-140 is 2^-10
    assert float((got[7, :, 0].double() / want[7, :, 0] - 1.0).abs().max()) <= 2.0 ** -9
    got[7], want[7] = 1.0, 1.0
    assert _rel(got, want) <= TOLERANCE


@pytest.mark.parametrize("log2p", [-112, -125, -133, -140])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("heads,T,th,tw,key", [(HEADS, 1, 5, 13, 0), (HEADS, 1, 5, 13, 64), (30, 2, 17, 20, 0), (30, 2, 17, 20, 679)])
def test_small_probabilities_are_all_that_a_channel_holds(heads, T, th, tw, key, d, log2p):
    """Channel 0 is 0 but for one key, whose probability is 2^log2p of the others' and whose value is an ordinary number.  The probability is a
    multiple of 2^-149; the roundings of the scaled query, the score, the exponent, log2(e) and the exponential's argument are 2^-24
    of |log2p| each."""
    n = T * th * tw
    q, k, v = _inputs(heads, n, d)
    q[7], k[7] = 0.0, 0.0
    q[7, :, 0] = 1.0
    k[7, key, 0] = log2p / math.log2(math.e) * math.sqrt(d)
    v[7, :, 0] = 0.0
    v[7, key, 0] = 2.0 ** 20
    want = _exact(q, k, v)
    got = _attend_window("f32", d, heads, T, th, tw, q, k, v)
    assert float((got[7, :, 0].double() / want[7, :, 0] - 1.0).abs().max()) <= 2.0 ** (-150 - log2p) - log2p * 5 * math.log(2.0) * 2.0 ** -24
    got[7, :, 0], want[7, :, 0] = 1.0, 1.0
    assert _rel(got, want) <= TOLERANCE


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("heads,T,th,tw", [(HEADS, 1, 5, 13), (30, 2, 17, 20)])
def test_infinities_and_nan(heads, T, th, tw, d):
    """An infinite value reaches its channel of every output, also as the last one, for which the keys that fill up the last stage stand
    in; a NaN in a query reaches that query, in a key every output, in a value its channel."""
    n = T * th * tw
    q, k, v = _inputs(heads, n, d)
    v[3, n - 1, 5] = math.inf
    q[4, 11, 0] = math.nan
    k[5, n - 1, 1] = math.nan
    v[6, 2, 9] = math.nan
    got = _attend_window("f32", d, heads, T, th, tw, q, k, v)
    assert bool((got[3, :, 5] == math.inf).all())
    want = torch.zeros(heads, n, d, dtype=torch.bool)
    want[4, 11] = True
    want[5] = True
    want[6, :, 9] = True
    assert torch.equal(got.isnan(), want)
    got[3, :, 5] = 0.0
    assert bool(torch.isfinite(got[~want]).all())


def _near_one(shape, gen):
    """Numbers of [1, 1 + 2^-7), all 24 bits in use: what a first part that is cut off leaves of them is largest there."""
    return 1.0 + torch.rand(shape, generator=gen, dtype=torch.float64).mul(2.0 ** -7).float()


def single_score_products(d, n):
    """Q and K have one channel.  Key 0 has score 0, key j one of -32 to -32.6 in the log2 domain, channel j of the output its probability.
    Returns q, k, v and the scores [head][query][key] of the fp32 factors that are multiplied."""
    gen = torch.Generator().manual_seed(d + n)
    factor = float(torch.tensor(1.0 / math.sqrt(d))) * 1.4426950408889634
    q, k, v = (torch.zeros(HEADS, n, d) for _ in range(3))
    q[:, :, 0] = (_near_one((HEADS, n), gen).double() / factor).float()
    k[:, 1:, 0] = -32.0 * _near_one((HEADS, n - 1), gen)
    v[:, :d] = torch.eye(d)
    scaled = (q[:, :, 0].double() * factor).float()
    return q, k, v, scaled[:, :, None].double() * k[:, None, 1:d, 0].double()


def check_single_score_products(out, scores):
    """Of the product two thirds of a unit of 2^-24 are rounded off in the sum of its parts (|score| above 32), one at most is left out;
    2^-23 of the exponential and twice 2^-24 of the normalisation are 2^-26 of a score of 32."""
    got = torch.log2(out[:, :, 1:].double() / out[:, :, :1].double())
    assert float((got / scores - 1.0).abs().max()) <= 2.3 * 2.0 ** -24


def single_value_products(d, n):
    """Key j has a probability just above one half of that of key 0, and two channels, 2 j with value 1 and 2 j + 1 with a generic one."""
    gen = torch.Generator().manual_seed(d + n)
    q, k, v = (torch.zeros(HEADS, n, d) for _ in range(3))
    q[:, :, 0] = math.sqrt(d) / 1.4426950408889634
    q[:, :, 0] *= 1.0 + torch.rand((HEADS, n), generator=gen) * 2.0 ** -10
    k[:, 1:, 0] = -0.998 + 0.008 * torch.rand((HEADS, n - 1), generator=gen)
    generic = _near_one((HEADS, d // 2), gen)
    for j in range(1, d // 2):
        v[:, j, 2 * j], v[:, j, 2 * j + 1] = 1.0, generic[:, j]
    return q, k, v, generic


def check_single_value_products(out, generic):
    """One unit of 2^-24 at most is left out of the product of the generic value, one rounded off in the sum of its parts, one in either
    channel's normalisation; the probability itself is the same in both channels."""
    got = out[:, :, 3::2].double() / out[:, :, 2::2].double()
    assert float((got / generic[:, None, 1:].double() - 1.0).abs().max()) <= 4.05 * 2.0 ** -24


@pytest.mark.parametrize("d", [64, 128])
def test_a_product_alone(d):
    """No sum of many products hides what the parts leave out of one: below 2^-24 of it, where the first part is rounded (2^-22 where it is
    cut off)."""
    T, th, tw = 1, 8, 16
    q, k, v, scores = single_score_products(d, th * tw)
    check_single_score_products(_attend_window("f32", d, HEADS, T, th, tw, q, k, v), scores)
    q, k, v, generic = single_value_products(d, th * tw)
    check_single_value_products(_attend_window("f32", d, HEADS, T, th, tw, q, k, v), generic)


# The number of [1, 2) of whose square the parts leave out most, 2^-24.01 (2^-22.02 of the second's, if the first part were cut off)
REPEATED = [1.0038986206054688, 1.0077972412109375]


@pytest.mark.parametrize("number", REPEATED)
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("heads,T,th,tw", [(HEADS, 1, 5, 13), (51, 7, 10, 10)])
def test_numbers_of_one_mantissa(heads, T, th, tw, d, number):
    """What is left out of every product is the same share of it and does not average out."""
    n = T * th * tw
    gen = torch.Generator().manual_seed(n + d)
    q, k, v = (number * torch.exp2(torch.randint(-2, 2, (heads, n, d), generator=gen).float()) *
               (2.0 * torch.randint(0, 2, (heads, n, d), generator=gen) - 1.0) for _ in range(3))
    got = _attend_window("f32", d, heads, T, th, tw, q, k, v)
    assert _rel(got, _exact(q, k, v)) <= TOLERANCE
