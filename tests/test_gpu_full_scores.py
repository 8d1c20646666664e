"""bf16 scores of more rows than one tile holds (plain accumulation and wide windows): ends of tiles, of steps and of query
heads, both scale modes, the value prior, given normalisers, and logits that outgrow the first keys' by far."""
import numpy as np
import pytest

import oracle
from paper_2506_03762_amd import binding as B
from paper_2506_03762_amd import synth
from tests import harness as H
from tests.harness import Opts

SHAPES = [
    # batch, KV heads, group, window, n, d
    (1, 2, 1, 513, 513, 128), (1, 1, 1, 1025, 1025, 64),      # one row more than the tiles; a single key in the last step
    (1, 2, 3, 333, 333, 128), (2, 1, 5, 257, 320, 64),        # ends of heads inside a tile
    (1, 3, 7, 100, 1111, 128), (1, 1, 6, 87, 700, 64),        # rows of two heads in one wave
    (1, 1, 2, 2500, 2500, 128), (1, 4, 2, 640, 4000, 64),     # several tiles and parts, odd and even counts
    (1, 2, 3, 50, 900, 128), (1, 1, 5, 40, 600, 64),          # 129 to 224 rows with a wide pool: tiles of 128 rows
]


def _case(shape, prior, fixed, grow=False):
    batch, hkv, group, window, n, d = shape
    w = synth.scaled(synth.C2, name="full", batch=batch, n_q_heads=hkv * group, n_kv_heads=hkv, head_dim=d, seq_len=n,
                     window=window, budget=max(1, n // 9), recent=min(20, n // 9))
    wide = group * window <= 224
    opts = Opts(value_prior=prior or wide, pool=19 if wide else 7, scale_mode=oracle.SCALE_FIXED if fixed else oracle.SCALE_ADAPTIVE,
                fixed_scale=d ** -0.5 if fixed else 0.0)
    q, k, v = synth.make_prefill(w)
    if grow:  # some late keys far along the queries: 2^100 and more times the first ones' weight
        k = k.copy()
        k[:, :, n // 2::97] = q[:, ::group, n - 1:n] * 8.0
    return w, opts, (q, k, v)


def _close(got, ref, rtol):
    # fp32 sums of exact products: logits of x carry x * 1e-6 or so, the relative error of their exponentials
    np.testing.assert_allclose(got, ref, rtol=rtol, atol=rtol * 1e-3 * ref.mean())


@pytest.mark.gpu
@pytest.mark.parametrize("prior,fixed", [(False, True), (True, True), (False, False), (True, False)])
@pytest.mark.parametrize("shape", SHAPES)
def test_scores(shape, prior, fixed):
    w, opts, inputs = _case(shape, prior, fixed)
    _close(H.run_prefill_gpu(w, opts, inputs).scores, H.run_prefill_oracle(w, opts, inputs).scores, 2e-4)


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [SHAPES[0], SHAPES[6]])
def test_late_keys_that_outweigh_the_first(shape):
    w, opts, inputs = _case(shape, False, True, grow=True)
    # (logits of several hundred: 2e-3)
    _close(H.run_prefill_gpu(w, opts, inputs).scores, H.run_prefill_oracle(w, opts, inputs).scores, 2e-3)


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [SHAPES[2], SHAPES[4], SHAPES[7]])
def test_given_normalisers(shape):
    import torch
    w, opts, inputs = _case(shape, True, False)
    p = H.gpu_params(w, opts)
    q, k, v = (H.to_device(a, w.dtype) for a in inputs)
    lse = torch.empty((w.batch, w.n_q_heads, w.window), dtype=torch.float32, device="cuda")
    B.aha_prefill_row_stats(p.with_strides(q, k, v), q, k, lse, None, B.alloc_workspace(p))
    got = H.run_scores_from_lse_gpu(w, opts, inputs, lse.cpu().numpy())
    _close(got, H.run_prefill_oracle(w, opts, inputs).scores, 2e-4)


@pytest.mark.gpu
def test_given_normalisers_are_taken_as_they_are():
    """Keys of zeros: a row adds exp(-lse).  Normalisers whose logarithms to base 2 lie around 1, of which one place is lost if
    1 is added and subtracted on the way."""
    import torch
    n, window = 1000, 600
    p, q, k, v, scores, ws = _random(2, 1, window, n, 128)
    k.zero_()
    gen = torch.Generator(device="cuda").manual_seed(3)
    lse = 0.69 + 0.01 * torch.rand((1, 2, window), generator=gen, device="cuda")
    B.aha_prefill_scores_lse(p, q, k, v, lse, scores, ws)
    added = torch.exp(-lse.double())
    want = torch.cat([added.sum(-1, keepdim=True).expand(1, 2, n - window), added.flip(-1).cumsum(-1).flip(-1)], -1)
    error = scores.double() / want - 1
    # a sum of several hundred fp32 terms ends rounded at 2^-24 of itself, 3.5e-8 on average; 5.0e-8 to 5.8e-8 with the place lost
    assert error.pow(2).mean().sqrt() < 4.4e-8


def _time(calls):
    """Median us of each call, timed in turn."""
    import torch
    times = [[] for _ in calls]
    for i in range(24):
        for call, t in zip(calls, times):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            for _ in range(4):
                call()
            b.record()
            torch.cuda.synchronize()
            t.append(a.elapsed_time(b) * 250)
    return [sorted(t[4:])[10] for t in times]


def _random(hkv, group, window, n, d):
    import torch
    q, k, v = (torch.randn((1, h, n, d), device="cuda", dtype=torch.bfloat16) for h in (hkv * group, hkv, hkv))
    p = B.Params(batch=1, n_q_heads=hkv * group, n_kv_heads=hkv, head_dim=d, seq_len=n, window=window, budget=64, recent=8,
                 scale_mode=oracle.SCALE_FIXED, fixed_scale=d ** -0.5, value_prior=0).with_strides(q, k, v)
    return p, q, k, v, torch.empty((1, hkv, n), dtype=torch.float32, device="cuda"), B.alloc_workspace(p)


@pytest.mark.gpu
def test_time_of_given_normalisers():
    """Rows that are no multiple of a wave's: us with the end of one head and the start of the next in a wave 141, against 96 of
    4992 rows; 97 with whole waves to a head."""
    import torch
    calls = []
    for n in (5000, 4992):
        p, q, k, v, scores, ws = _random(4, 7, n, n, 64)
        lse = torch.full((1, 28, n), 9.0, device="cuda")
        calls.append(lambda p=p, q=q, k=k, v=v, lse=lse, s=scores, ws=ws: B.aha_prefill_scores_lse(p, q, k, v, lse, s, ws))
    t = _time(calls)
    assert t[0] < 1.15 * t[1], t


@pytest.mark.gpu
def test_time_of_rows_that_fill_no_tile():
    """Windows of 3 x 400 rows fill 5 tiles, 6 with whole waves to a head: us in six 205 against 160 of 3 x 384 rows, in five 165."""
    calls = []
    for window in (400, 384):
        args = _random(16, 3, window, 12822, 128)
        calls.append(lambda args=args: B.aha_prefill_scores(*args))
    t = _time(calls)
    assert t[0] < 1.15 * t[1], t


@pytest.mark.gpu
@pytest.mark.parametrize("given", [False, True])
@pytest.mark.parametrize("shape", [SHAPES[0], SHAPES[3], SHAPES[4], SHAPES[5], SHAPES[7], SHAPES[8], SHAPES[9]])
def test_token_major(shape, given):
    """Neighbouring tokens of a head lie a row of all heads apart: as from heads that lie together (sums by atomics)."""
    import torch
    batch, hkv, group, window, n, d = shape
    gen = torch.Generator(device="cuda").manual_seed(n)
    heads = [torch.randn((batch, h, n, d), generator=gen, device="cuda", dtype=torch.bfloat16) for h in (hkv * group, hkv, hkv)]
    tokens = [t.transpose(1, 2).contiguous().transpose(1, 2) for t in heads]
    got = []
    for q, k, v in (heads, tokens):
        p = B.Params(batch=batch, n_q_heads=hkv * group, n_kv_heads=hkv, head_dim=d, seq_len=n, window=window, budget=n // 9,
                     recent=0, pool_kernel=19 if group * window <= 224 else 7).with_strides(q, k, v)
        ws = B.alloc_workspace(p)
        ws.fill_(0xA5)
        scores = torch.full((batch, hkv, n), float("nan"), device="cuda")
        if given:
            lse = torch.full((batch, hkv * group, window), 7.0, device="cuda")
            B.aha_prefill_scores_lse(p, q, k, v, lse, scores, ws)
        else:
            B.aha_prefill_scores(p, q, k, v, scores, ws)
        got.append(scores)
    torch.testing.assert_close(got[1], got[0], rtol=1e-5, atol=0)
