"""Windowed bf16 scores whose waves share the keys: full tiles of 256 and 512 rows that are swept twice.  Ends of ranges and of
steps, ranges that LDS does not keep, rows past the last one, and a workgroup that does missing parts itself."""
import numpy as np
import pytest

import oracle
from paper_2506_03762_amd import binding as B
from paper_2506_03762_amd import synth
from tests import harness as H
from tests.harness import Opts

SHAPES = [
    # batch, KV heads, group, window, n, d
    (1, 33, 4, 64, 2113, 128), (1, 8, 8, 32, 8321, 128),    # one key more than a range; several ranges
    (2, 40, 7, 30, 1000, 128),                               # 210 rows
    (1, 64, 8, 32, 8300, 128),                               # ranges longer than the LDS keeps
    (1, 3, 8, 64, 3001, 128), (1, 2, 7, 57, 515, 128),      # two tiles, 399 rows
    (1, 5, 8, 64, 2817, 64), (1, 70, 4, 125, 1800, 64),
]


@pytest.mark.gpu
@pytest.mark.parametrize("prior,fixed", [(True, False), (False, True), (True, True)])
@pytest.mark.parametrize("shape", SHAPES)
def test_scores_and_missing_parts(shape, prior, fixed):
    batch, hkv, group, window, n, d = shape
    w = synth.scaled(synth.C2, name="share", batch=batch, n_q_heads=hkv * group, n_kv_heads=hkv, head_dim=d, seq_len=n,
                     window=window, budget=n // 12, recent=20)
    opts = Opts(value_prior=prior, pool=17 if n % 2 else 7, scale_mode=oracle.SCALE_FIXED if fixed else oracle.SCALE_ADAPTIVE,
                fixed_scale=d ** -0.5 if fixed else 0.0)
    inputs = synth.make_prefill(w)
    got, ref = H.run_prefill_gpu(w, opts, inputs).scores, H.run_prefill_oracle(w, opts, inputs).scores
    # (fp32 sums of exact products: logits of a few tens carry 1e-5, which is the relative error of their exponentials)
    np.testing.assert_allclose(got, ref, rtol=2e-4, atol=2e-4 * 1e-3 * ref.mean())
    assert B.load().aha_exchange_looks(0) == B.AHA_OK
    try:
        alone = H.run_prefill_gpu(w, opts, inputs).scores
    finally:
        B.load().aha_exchange_looks(4000)
    assert np.array_equal(alone, got)


def _scores(p, q, k, v):
    import torch
    p = p.with_strides(q, k, v)
    ws = B.alloc_workspace(p)
    ws.fill_(0xA5)
    scores = torch.full((p.batch, p.n_kv_heads, p.seq_len), float("nan"), device="cuda")
    B.aha_prefill_scores(p, q, k, v, scores, ws)
    return scores


def _random(batch, hkv, group, window, n, d, pool=7):
    import torch
    gen = torch.Generator(device="cuda").manual_seed(n)
    q, k, v = (torch.randn((batch, h, n, d), generator=gen, device="cuda", dtype=torch.bfloat16) for h in (hkv * group, hkv, hkv))
    p = B.Params(batch=batch, n_q_heads=hkv * group, n_kv_heads=hkv, head_dim=d, seq_len=n, window=window, budget=n // 12,
                 recent=8, pool_kernel=pool)
    return p, q, k, v


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [SHAPES[0], SHAPES[2], SHAPES[3], SHAPES[4], SHAPES[6]])
def test_token_major(shape):
    """Neighbouring tokens of a head lie a row of all heads apart: the same bits as from heads that lie together."""
    p, *heads = _random(*shape, pool=17)
    tokens = [t.transpose(1, 2).contiguous().transpose(1, 2) for t in heads]
    assert all(t.stride(2) == t.shape[1] * t.shape[3] for t in tokens)
    assert _scores(p, *tokens).equal(_scores(p, *heads))


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [SHAPES[0], SHAPES[3], SHAPES[4], SHAPES[6]])
def test_graph_replays(shape):
    """A replay reuses the call's tag: both kinds of words of the one before must be gone."""
    import torch
    p, q, k, v = _random(*shape)
    p = p.with_strides(q, k, v)
    sets = [(q.clone(), k.clone(), v.clone()), (q.flip(2), k.roll(5, 2), 2 * v.flip(2))]
    ws = B.alloc_workspace(p)
    ws.fill_(0xA5)
    scores = torch.empty((p.batch, p.n_kv_heads, p.seq_len), device="cuda")
    want = []
    for s in sets:
        B.aha_prefill_scores(p, *s, scores, ws)
        want.append(scores.clone())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        B.aha_prefill_scores(p, q, k, v, scores, ws)
    for i in (1, 0, 0, 1):
        for dst, src in zip((q, k, v), sets[i]):
            dst.copy_(src)
        scores.fill_(-1.0)
        graph.replay()
        torch.cuda.synchronize()
        assert scores.equal(want[i])
        B.aha_prefill_scores(p, *sets[1], scores, ws)  # other work of the same workspace in between


@pytest.mark.gpu
@pytest.mark.parametrize("d,n", [(64, 6000), (128, 3500)])
def test_value_rows_past_the_caches(d, n):
    """From 80 MB of keys and values on the value rows are read past the caches: against the halves of the heads, which are
    below (their ranges differ: last bits, rescaled by the largest prior of the same head)."""
    import torch
    p, q, k, v = _random(1, 64, 8, 64, n, d)
    assert 4 * 64 * n * d > 80e6 > 4 * 32 * n * d
    whole = _scores(p, q, k, v)
    p.n_q_heads, p.n_kv_heads = 256, 32
    halves = torch.cat([_scores(p, q[:, i * 8:i * 8 + 256], k[:, i:i + 32], v[:, i:i + 32]) for i in (0, 32)], 1)
    torch.testing.assert_close(whole, halves, rtol=2e-5, atol=0)
