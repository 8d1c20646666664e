"""Window attention where a workgroup's eight waves share the keys: fewer key steps than stages in
flight, ragged last steps, row counts that fill neither the last block nor the last workgroup."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,hkv", [(64, 2), (128, 2), (128, 12)])
@pytest.mark.parametrize("group,window", [(5, 29), (8, 32), (3, 90), (7, 64)])  # 5, 8, 9 and 14 blocks of 32 rows
@pytest.mark.parametrize("n", [97, 128, 193, 1000, 4099])
def test_against_float64(d, hkv, group, window, n):
    import torch
    from paper_2506_03762_amd import binding as B
    batch = 2
    gen = torch.Generator(device="cuda").manual_seed(n + d + group)
    q, k, v = (torch.randn((batch, n, h, d), generator=gen, device="cuda", dtype=torch.bfloat16).transpose(1, 2)
               for h in (hkv * group, hkv, hkv))  # token-major
    k[:, :, 0] *= 3
    p = B.Params(batch=batch, n_q_heads=hkv * group, n_kv_heads=hkv, head_dim=d, seq_len=n, window=window,
                 budget=min(n, 40), recent=8, dtype=B.AHA_BF16).with_strides(q, k, v)
    out = torch.full((batch, hkv * group, window, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    lse = torch.full((batch, hkv * group, window), float("nan"), device="cuda")
    ws = torch.full((B.window_attention_workspace_bytes(p),), 0xA5, dtype=torch.uint8, device="cuda")
    B.aha_prefill_window_attention(p, q, k, v, out, lse, ws)
    Q, K, V = (t.double().cpu() for t in (q, k, v))
    K, V = (t.repeat_interleave(group, 1) for t in (K, V))
    s = Q[:, :, n - window:] @ K.transpose(2, 3) / math.sqrt(d)
    s.masked_fill_(torch.arange(n)[None] > torch.arange(n - window, n)[:, None], -math.inf)
    ref_lse = torch.logsumexp(s, -1)
    ref = (torch.softmax(s, -1) @ V).numpy()
    got = out.double().cpu().numpy()
    rms = np.sqrt((ref ** 2).mean(-1, keepdims=True))
    # output and probabilities rounded to bf16: at most 2^-8 and 2^-9 of the value
    assert (np.abs(got - ref) <= 2.0 ** -8 * 1.01 * np.abs(ref) + 2.0 ** -8 * 3 * rms).all()
    np.testing.assert_allclose(lse.double().cpu().numpy(), ref_lse.numpy(), rtol=1e-5, atol=1e-4)


@pytest.mark.parametrize("hkv,group,n,low,high,nparts", [
    (8, 5, 16000, 15491, 15754, 32),   # one range of about eight steps of 64 keys: low in its first, high in its fifth
    (32, 8, 1000, 770, 840, 8),        # two steps per range
])
def test_a_dominant_key_is_weighted_exactly(hkv, group, n, low, high, nparts):
    """Two keys carry each row's weight, `high` 98 to 99 % of it, and `low` comes first, 70 to 90 times
    (2^6 to 2^6.5) lighter: the output is `high`'s value row and a hundredth of `low`'s, rounded
    once to bf16.  A weight of 2^6.3 in bf16 would add up to 2^-8 of the value to that half unit."""
    import torch
    from paper_2506_03762_amd import binding as B
    d, window = 128, 32
    gen = torch.Generator(device="cuda").manual_seed(n)
    q = torch.zeros((1, hkv * group, n, d), device="cuda", dtype=torch.bfloat16)
    k = torch.zeros((1, hkv, n, d), device="cuda", dtype=torch.bfloat16)
    v = torch.randn((1, hkv, n, d), generator=gen, device="cuda", dtype=torch.bfloat16)
    q[..., 0] = 0.95 + 0.1 * torch.rand((1, hkv * group, n), generator=gen, device="cuda")
    k[:, :, low, 0], k[:, :, high, 0] = 157, 206      # log2 of the weights: 20 and 26.3, the others' 0
    p = B.Params(batch=1, n_q_heads=hkv * group, n_kv_heads=hkv, head_dim=d, seq_len=n, window=window,
                 budget=40, recent=8, dtype=B.AHA_BF16).with_strides(q, k, v)
    # (the form whose waves share the keys: `nparts` key ranges of group blocks of 32 rows)
    assert B.window_attention_workspace_bytes(p) == hkv * nparts * group * 32 * (d + 2) * 4
    out = torch.full((1, hkv * group, window, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    ws = torch.empty((B.window_attention_workspace_bytes(p),), dtype=torch.uint8, device="cuda")
    B.aha_prefill_window_attention(p, q, k, v, out, None, ws)
    Q, K, V = (t.double().cpu() for t in (q[:, :, n - window:], k, v))
    K, V = (t.repeat_interleave(group, 1) for t in (K, V))
    s = Q @ K.transpose(2, 3) / math.sqrt(d)
    s.masked_fill_(torch.arange(n)[None] > torch.arange(n - window, n)[:, None], -math.inf)
    w = torch.softmax(s, -1)
    assert ((w[..., high] > 0.97) & (w[..., high] < 0.992)).all()
    ref = (w @ V).numpy()
    half_unit = 2.0 ** (np.floor(np.log2(np.abs(ref))) - 8)
    # the weights other than high's, at most 3 % in all, rounded to bf16: 2^-8 each, values up to 5
    assert (np.abs(out.double().cpu().numpy() - ref) <= half_unit * 1.001 + 2.0 ** -8 * 0.03 * 5).all()


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
@pytest.mark.parametrize("hkv,group,n,window,back,size", [
    (24, 1, 3000, 256, 1, 31948800), (24, 1, 3000, 256, 130, 31948800),  # eight blocks of one head
    (2, 2, 9000, 200, 1, 20334080),                                      # thirteen blocks, two heads in one of them
    (8, 1, 20000, 160, 70, 21299200),                                    # five blocks: waves without rows
])
def test_a_value_row_that_is_not_finite(hkv, group, n, window, back, size, bad):
    """Blocks of 32 rows that end before the bad row's step of 64 keys do not see it."""
    import torch
    from paper_2506_03762_amd import binding as B
    d = 128
    gen = torch.Generator(device="cuda").manual_seed(n)
    q, k, v = (torch.randn((1, h, n, d), generator=gen, device="cuda", dtype=torch.bfloat16) for h in (hkv * group, hkv, hkv))
    p = B.Params(batch=1, n_q_heads=hkv * group, n_kv_heads=hkv, head_dim=d, seq_len=n, window=window,
                 budget=40, recent=8, dtype=B.AHA_BF16).with_strides(q, k, v)
    assert B.window_attention_workspace_bytes(p) == size  # (the form whose waves share the keys)

    def attention():
        out = torch.full((1, hkv * group, window, d), float("nan"), dtype=torch.bfloat16, device="cuda")
        ws = torch.full((B.window_attention_workspace_bytes(p),), 0xA5, dtype=torch.uint8, device="cuda")
        B.aha_prefill_window_attention(p, q, k, v, out, None, ws)
        return out.reshape(hkv, group * window, d)

    want = attention()
    v[:, :, n - back] = bad
    got = attention()
    pos = torch.arange(group * window) % window + n - window
    last = torch.stack([b.max() for b in pos.split(32)]).repeat_interleave(32)[:len(pos)]
    unseen = (last < (n - back) // 64 * 64).cuda()
    assert unseen.any()
    assert torch.equal(got[:, unseen], want[:, unseen])
    assert not torch.isfinite(got[:, (pos >= n - back).cuda()]).any()
