"""Keys that a row does not see get nothing from it, whatever its logits are: query rows that are not finite, and a scale of
zero, which weighs all seen keys alike however large their products.  Every way the windowed bf16 scores are formed: held in
ranges of one and several steps and in two tiles, swept twice, keys shared, two launches and several tiles."""
import pytest

from paper_2506_03762_amd import binding as B

pytestmark = pytest.mark.gpu

SHAPES = [
    # KV heads, group, window, n, d
    (2, 1, 64, 600, 128), (2, 2, 60, 333, 64), (4, 1, 100, 700, 128), (3, 1, 200, 700, 128),  # held, one step
    (64, 1, 60, 7000, 64), (64, 1, 128, 3000, 64),                                           # several steps; swept twice
    (33, 1, 256, 2113, 128), (3, 1, 500, 3001, 128), (3, 1, 300, 1500, 64), (2, 1, 600, 1300, 128),
]


def _inputs(shape, scale):
    import torch
    hkv, group, window, n, d = shape
    gen = torch.Generator(device="cuda").manual_seed(n)
    q, k, v = (torch.randn((1, h, n, d), generator=gen, device="cuda", dtype=torch.bfloat16) for h in (hkv * group, hkv, hkv))
    p = B.Params(batch=1, n_q_heads=hkv * group, n_kv_heads=hkv, head_dim=d, seq_len=n, window=window, budget=n // 9, recent=0,
                 scale_mode=B.AHA_SCALE_FIXED, fixed_scale=scale, value_prior=0).with_strides(q, k, v)
    return p, q, k, v


def _scores(p, q, k, v):
    import torch
    scores = torch.full((1, p.n_kv_heads, p.seq_len), -1.0, device="cuda")
    ws = B.alloc_workspace(p)
    ws.fill_(0xA5)
    B.aha_prefill_scores(p, q, k, v, scores, ws)
    return scores


@pytest.mark.parametrize("bad", [float("nan"), float("inf"), float("-inf")])
@pytest.mark.parametrize("shape", SHAPES)
def test_a_row_that_is_not_finite(shape, bad):
    import torch
    p, q, k, v = _inputs(shape, shape[4] ** -0.5)
    k[..., 0] = k[..., 0].abs() + 0.5
    want = _scores(p, q, k, v)
    at = p.seq_len - 40
    if bad < 0:  # (every product -inf)
        q[:, ::shape[1], at, 0] = bad
    else:
        q[:, ::shape[1], at] = bad
    got = _scores(p, q, k, v)
    assert not torch.isfinite(got[..., :at + 1]).any()
    # (the last bits may differ: a row without a finite sum takes the other rows of its wave the exact way; sums by atomics)
    torch.testing.assert_close(got[..., at + 1:], want[..., at + 1:], rtol=1e-5, atol=0)


@pytest.mark.parametrize("shape", SHAPES)
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
    # a normaliser of log2 n with 20 bits behind the point, sums of up to 600 equal terms
    assert ((got - want).abs() <= 1e-5 * want).all()
