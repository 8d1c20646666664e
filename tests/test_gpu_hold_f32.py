"""fp32 scores in one launch: one to six blocks of rows, ragged last ranges, rows and keys, a wide pool, missing parts, replays,
rows that are not finite, and a workspace that holds two launches only."""
import numpy as np
import pytest

from paper_2506_03762_amd import binding as B
from paper_2506_03762_amd import synth
from tests import harness as H
from tests.harness import Opts
from tests.test_score_routes import _call, _one_launch, _params

SHAPES = [
    # batch, KV heads, group, window, n, d
    (1, 2, 1, 32, 512, 64), (2, 3, 1, 8, 257, 128), (1, 3, 3, 21, 1153, 64), (1, 2, 2, 64, 385, 128), (1, 1, 3, 64, 700, 128),
    (1, 1, 1, 1, 130, 64), (1, 8, 1, 40, 3000, 64),
]


@pytest.mark.parametrize("z,group,window,n,d,one", [
    (2, 1, 32, 512, 64, True), (1, 6, 32, 2000, 128, True), (1, 7, 28, 2000, 128, False),  # 192, 196 rows
    (128, 1, 32, 512, 128, True), (129, 1, 32, 512, 128, False),   # two workgroups per CU
    (128, 3, 32, 256, 128, True), (128, 3, 32, 257, 128, False),   # one
    (8, 1, 16, 306, 128, False), (8, 1, 16, 306, 64, True),        # two launches 19.2 us, one 20.5
    # few problems and rows, short prompts, d = 128 with a prior (score stage in two launches, one)
    (4, 1, 32, 700, 128, False), (8, 1, 32, 700, 128, True),       # 13.3, 13.9
    (2, 1, 64, 900, 128, False), (2, 1, 64, 1400, 128, True), (1, 1, 8, 1500, 128, False), (4, 1, 32, 1100, 128, True),
])
def test_route(z, group, window, n, d, one):
    p = _params(z, group, window, n, d, dtype=B.AHA_F32)
    assert _one_launch("aha_prefill_scores", p) == one
    assert not _one_launch("aha_prefill_scores_rows", p)
    assert not _one_launch("aha_prefill_scores_lse", p)


@pytest.mark.parametrize("z,window,n,pool,one", [
    # each range squares the rows of its pools' halo (step in two launches, one)
    (2, 32, 512, 17, True), (2, 32, 512, 63, False),    # 18.5, 19.1
    (4, 8, 1300, 63, False), (2, 32, 1400, 255, True), (8, 128, 315, 255, True),
])
def test_route_of_wide_pools(z, window, n, pool, one):
    assert _one_launch("aha_prefill_scores", _params(z, 1, window, n, 64, dtype=B.AHA_F32, pool_kernel=pool)) == one


def test_workspace_of_two_launches_is_served():
    p = _params(2, 6, 32, 512, 64, dtype=B.AHA_F32)   # (1536 bytes of normalisers, 4096 of the prior, 256 of its maxima)
    assert B.workspace_bytes(p) > 5888
    assert _one_launch("aha_prefill_scores", p) and not _one_launch("aha_prefill_scores", p, 5888)
    assert _call("aha_prefill_scores", p, 5887) == B.AHA_ERR_WORKSPACE


def _inputs(shape, opts):
    batch, hkv, group, window, n, d = shape
    w = synth.scaled(synth.C1, name="hold_f32", batch=batch, n_q_heads=hkv * group, n_kv_heads=hkv, head_dim=d, seq_len=n,
                     window=window, budget=n // 4, recent=min(20, n // 8))
    return w, synth.make_prefill(w)


@pytest.mark.gpu
@pytest.mark.parametrize("prior", [True, False])
@pytest.mark.parametrize("shape", SHAPES)
def test_scores_and_missing_parts(shape, prior):
    opts = Opts(value_prior=prior, pool=255 if shape[4] % 2 else 7)
    w, inputs = _inputs(shape, opts)
    got, ref = H.run_prefill_gpu(w, opts, inputs).scores, H.run_prefill_oracle(w, opts, inputs).scores
    H.assert_scores_close(got, ref, w, opts)
    # a workgroup that looks once and does whatever is not there yet
    assert B.load().aha_exchange_looks(0) == B.AHA_OK
    try:
        alone = H.run_prefill_gpu(w, opts, inputs).scores
    finally:
        B.load().aha_exchange_looks(4000)
    assert np.array_equal(alone, got)


def _random(shape):
    import torch
    batch, hkv, group, window, n, d = shape
    gen = torch.Generator(device="cuda").manual_seed(n)
    q, k, v = (torch.randn((batch, h, n, d), generator=gen, device="cuda") for h in (hkv * group, hkv, hkv))
    p = B.Params(batch=batch, n_q_heads=hkv * group, n_kv_heads=hkv, head_dim=d, seq_len=n, window=window, budget=n // 4,
                 recent=0, dtype=B.AHA_F32, scale_mode=B.AHA_SCALE_FIXED, fixed_scale=d ** -0.5).with_strides(q, k, v)
    ws = B.alloc_workspace(p)
    ws.fill_(0xA5)
    return p, q, k, v, ws, torch.empty((batch, hkv, n), device="cuda")


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [SHAPES[0], SHAPES[3]])
def test_graph_replays(shape):
    import torch
    p, q, k, v, ws, scores = _random(shape)
    sets = [(q.clone(), k.clone(), v.clone()), (q.flip(2), k.roll(5, 2), 2 * v.flip(2))]
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


@pytest.mark.gpu
@pytest.mark.parametrize("bad", [float("nan"), float("inf"), float("-inf")])
@pytest.mark.parametrize("shape", [SHAPES[0], SHAPES[3]])
def test_a_row_that_is_not_finite(shape, bad):
    import torch
    p, q, k, v, ws, scores = _random(shape)
    v.fill_(1.0)
    k[..., 0] = k[..., 0].abs() + 0.5
    B.aha_prefill_scores(p, q, k, v, scores, ws)
    want = scores.clone()
    at = p.seq_len - shape[3] // 2
    if bad < 0:  # (every product -inf)
        q[:, :, at, 0] = bad
    else:
        q[:, :, at] = bad
    B.aha_prefill_scores(p, q, k, v, scores, ws)
    assert not torch.isfinite(scores[..., :at + 1]).any()
    assert scores[..., at + 1:].equal(want[..., at + 1:])


@pytest.mark.gpu
def test_captured_where_two_launches_are_shorter():
    """Few rows of a short prompt: one launch, two in a graph (those of chosen rows)."""
    import torch
    p, q, k, v, ws, scores = _random((1, 4, 1, 16, 500, 128))
    p.value_prior = 0
    rows = torch.arange(p.seq_len - p.window, p.seq_len, dtype=torch.int32, device="cuda").expand(1, 4, p.window).contiguous()
    chosen, eager = torch.empty_like(scores), torch.empty_like(scores)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        B.aha_prefill_scores(p, q, k, v, scores, ws)
    for s in ((q.clone(), k.clone()), (q.flip(2), k.roll(5, 2)), (q.clone(), k.clone())):
        q.copy_(s[0]), k.copy_(s[1])
        B.aha_prefill_scores_rows(p, q, k, v, rows, chosen, ws)
        B.aha_prefill_scores(p, q, k, v, eager, ws)
        scores.fill_(-1.0)
        graph.replay()
        torch.cuda.synchronize()
        assert scores.equal(chosen) and not eager.equal(chosen)
        # (what fp32 scores are held to)
        assert ((eager - scores).abs() <= 1e-5 * scores).all()
