"""Window attention where a workgroup's eight waves share the keys: fewer key steps than stages in
flight, ragged last steps, row counts that fill neither the last block nor the last workgroup."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("group,window", [(5, 29), (8, 32), (3, 90), (7, 64)])  # 5, 8, 9 and 14 blocks of 32 rows
@pytest.mark.parametrize("n", [97, 128, 193, 1000, 4099])
def test_against_float64(d, group, window, n):
    import torch
    from paper_2506_03762_amd import binding as B
    hkv, batch = 2, 2
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
