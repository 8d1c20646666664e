"""Windowed scores whose blocks are held as exponentials relative to the running maximum of their row: ranges of several
steps of which later ones lie past the last key, rows whose maximum moves from step to step, rows that are not finite, a
scale of zero."""
import pytest

from paper_2506_03762_amd import binding as B
from tests.test_gpu_unseen_keys import _inputs, _scores

pytestmark = pytest.mark.gpu

SHAPES = [
    # KV heads, group, window, n, d: ranges of two and four steps (200 and 188 keys in the last), of one, two tiles
    (8, 1, 60, 24776, 128), (24, 1, 30, 12476, 64), (5, 1, 33, 2113, 128), (2, 1, 100, 300, 64), (3, 1, 200, 700, 128),
]


def _exact(p, q, k):
    import torch
    hkv, group, window, n = p.n_kv_heads, p.n_q_heads // p.n_kv_heads, p.window, p.seq_len
    seen = torch.arange(n, device="cuda")[None] <= torch.arange(n - window, n, device="cuda")[:, None]
    out = torch.zeros((1, hkv, n), dtype=torch.float64, device="cuda")
    for h in range(hkv * group):
        x = (q[0, h, n - window:].double() @ k[0, h // group].double().T) * p.fixed_scale
        out[0, h // group] += torch.softmax(x.masked_fill(~seen, float("-inf")), -1).sum(0)
    return out


@pytest.mark.parametrize("rising", [False, True])
@pytest.mark.parametrize("shape", SHAPES)
def test_against_float64(shape, rising):
    import torch
    p, q, k, v = _inputs(shape, shape[4] ** -0.5)
    if rising:  # (longer keys, larger maxima, from block to block)
        k *= torch.linspace(0.5, 3.0, shape[3], device="cuda")[:, None].to(k.dtype)
    want, got = _exact(p, q, k), _scores(p, q, k, v).double()
    # Per term: the exponent's two roundings and the normaliser's three, each of a number below 128 (2^-17 at most, times ln 2),
    # two exponentials and a product (2^-23 each), the products' sums of 128 terms (2^-24 of 128 at most)
    assert ((got - want).abs() <= (5 * 2.0 ** -18 + 2.0 ** -17) * want + 1e-30).all()


@pytest.mark.parametrize("bad", [float("nan"), float("inf"), float("-inf")])
@pytest.mark.parametrize("shape", SHAPES[:2])
def test_a_row_that_is_not_finite(shape, bad):
    import torch
    p, q, k, v = _inputs(shape, shape[4] ** -0.5)
    k[..., 0] = k[..., 0].abs() + 0.5
    want = _scores(p, q, k, v)
    at = p.seq_len - shape[2] // 2
    if bad < 0:  # (every product -inf)
        q[:, :, at, 0] = bad
    else:
        q[:, :, at] = bad
    got = _scores(p, q, k, v)
    assert not torch.isfinite(got[..., :at + 1]).any()
    assert got[..., at + 1:].equal(want[..., at + 1:])


@pytest.mark.parametrize("shape", SHAPES[:2])
def test_a_scale_of_zero(shape):
    import torch
    p, q, k, v = _inputs(shape, 0.0)
    q *= 2.0 ** 57   # (products of some 2^118)
    k *= 2.0 ** 57
    hkv, group, window, n, d = shape
    rows = torch.arange(n - window, n, dtype=torch.float64)
    seen = (rows[:, None] >= torch.arange(n)[None]).double()
    want = (group * seen / (rows[:, None] + 1)).sum(0)
    got = _scores(p, q, k, v).double().cpu()
    # a normaliser of log2 n with 19 bits behind the point, sums of up to 60 equal terms
    assert ((got - want).abs() <= 1e-5 * want).all()


ROUNDS = [
    # more workgroups than the chip holds at once: KV heads, group, window, n, d
    (40, 1, 30, 15990, 64), (20, 2, 15, 32100, 128), (50, 1, 96, 3001, 128), (28, 1, 128, 5000, 64), (70, 1, 64, 4100, 64),
    (3, 1, 128, 16849, 128),  # (one round, many ranges)
    (1, 1, 128, 25601, 128), (2, 1, 70, 12500, 64),  # (and few workgroups)
    # many ranges of a problem in several rounds
    (6, 1, 100, 46001, 128), (16, 1, 64, 49300, 128), (2, 1, 40, 143400, 128), (4, 1, 128, 48600, 64), (8, 1, 50, 58000, 64),
]


@pytest.mark.parametrize("shape", ROUNDS)
def test_several_rounds(shape):
    p, q, k, v = _inputs(shape, shape[4] ** -0.5)
    want, got = _exact(p, q, k), _scores(p, q, k, v)
    assert ((got.double() - want).abs() <= (5 * 2.0 ** -18 + 2.0 ** -17) * want + 1e-30).all()
    # a workgroup that looks once and does whatever is not there yet
    assert B.load().aha_exchange_looks(0) == B.AHA_OK
    try:
        alone = _scores(p, q, k, v)
    finally:
        B.load().aha_exchange_looks(4000)
    assert alone.equal(got)


BESIDE_VALUES = [
    # up to 32 rows beside value rows, d = 128: ranges of four steps, ranges of two in several rounds
    (2, 1, 32, 140001, 128), (9, 1, 2, 32848, 128), (33, 8, 1, 8848, 128), (5, 1, 5, 103215, 128),
    # more rows: many ranges, in one round and in several
    (1, 1, 128, 25601, 128), (6, 1, 100, 46001, 128), (9, 1, 64, 58000, 128), (8, 1, 64, 71500, 64),
]


@pytest.mark.parametrize("shape", BESIDE_VALUES)
def test_beside_value_rows(shape):
    import torch
    p, q, k, v = _inputs(shape, shape[4] ** -0.5)
    want = _exact(p, q, k)
    p.value_prior, n = 1, p.seq_len
    half = (p.pool_kernel - 1) // 2
    past = torch.nn.functional.pad((v.double() ** 2).sum(-1).cumsum(-1), (1, 0))
    first, last = (torch.arange(n, device="cuda") - half).clamp(min=0), (torch.arange(n, device="cuda") + half + 1).clamp(max=n)
    gamma = (past[..., last] - past[..., first]) / (last - first)
    want *= gamma / gamma.amax(-1, keepdim=True)
    got = _scores(p, q, k, v)
    # (as above, and twice, for the key's own prior and the largest: sums of 128 squares, of the pool's seven and two more roundings)
    assert ((got.double() - want).abs() <= (5 * 2.0 ** -18 + 2.0 ** -17 + 2 * (2.0 ** -17 + 9 * 2.0 ** -24)) * want + 1e-30).all()
    # a workgroup that looks once and does whatever is not there yet
    assert B.load().aha_exchange_looks(0) == B.AHA_OK
    try:
        alone = _scores(p, q, k, v)
    finally:
        B.load().aha_exchange_looks(4000)
    assert alone.equal(got)
