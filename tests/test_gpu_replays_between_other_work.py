"""Graphs whose workspace other work overwrites between replays, in part and with the same bytes each time: a replay takes
nothing that an earlier one left there."""
import pytest

from paper_2506_03762_amd import binding as B
from tests.test_score_routes import _one_launch, _params

SHAPES = {
    # batch, KV heads, group, window, n, d: kernels whose workgroups exchange parts of a result
    "held": (1, 4, 2, 32, 3000, 128), "held_two_tiles": (1, 3, 8, 32, 900, 128), "held_in_rounds": (1, 64, 2, 32, 8300, 128),
    "stream": (2, 16, 3, 43, 2100, 128), "stream_two_tiles": (1, 3, 5, 77, 640, 128), "stream_workspace": (1, 64, 5, 32, 8300, 64),
    "share": (1, 8, 4, 64, 6000, 128), "share_two_tiles": (1, 2, 8, 64, 2100, 64), "share_workspace": (2, 64, 8, 64, 1300, 128),
    "given": (1, 4, 2, 32, 3000, 128), "given_large_tile": (1, 32, 8, 32, 2300, 128),
    "fp32": (1, 2, 2, 32, 512, 64), "fp32_short_ranges": (2, 3, 3, 21, 700, 128),
    # more words to a problem than its last workgroup takes away
    "held_many_words": (1, 1, 1, 64, 100000, 128), "stream_many_words": (2, 1, 3, 128, 17000, 64), "share_many_words": (1, 1, 7, 64, 20000, 64),
    "fp32_many_words": (1, 2, 2, 64, 6000, 64),
}


def _case(name):
    import torch
    batch, hkv, group, window, n, d = SHAPES[name]
    dtype = torch.float32 if name.startswith("fp32") else torch.bfloat16
    gen = torch.Generator(device="cuda").manual_seed(n)
    q, k, v = (torch.randn((batch, h, n, d), generator=gen, device="cuda", dtype=dtype) for h in (hkv * group, hkv, hkv))
    p = B.Params(batch=batch, n_q_heads=hkv * group, n_kv_heads=hkv, head_dim=d, seq_len=n, window=window, budget=n // 12,
                 recent=8, dtype=B.AHA_F32 if name.startswith("fp32") else B.AHA_BF16).with_strides(q, k, v)
    return p, q, k, v


def _score_call(name, p, q, k, v, scores, ws):
    import torch
    if not name.startswith("given"):
        return lambda q, k, v: B.aha_prefill_scores(p, q, k, v, scores, ws)
    lse = torch.full((p.batch, p.n_q_heads, p.window), 12.0, device="cuda")
    return lambda q, k, v: B.aha_prefill_scores_lse(p, q, k, v, lse, scores, ws)


@pytest.mark.parametrize("name", SHAPES)
def test_route(name):
    batch, hkv, group, window, n, d = SHAPES[name]
    p = _params(batch * hkv, group, window, n, d, dtype=B.AHA_F32 if name.startswith("fp32") else B.AHA_BF16)
    assert _one_launch("aha_prefill_scores_lse" if name.startswith("given") else "aha_prefill_scores", p)


@pytest.mark.gpu
@pytest.mark.parametrize("looks", [4000, 0])  # (0: a workgroup does at once what is not there yet)
@pytest.mark.parametrize("name", SHAPES)
def test_workspace_overwritten_in_part(name, looks):
    import torch
    p, q, k, v = _case(name)
    sets = [(q.clone(), k.clone(), v.clone()), (q.flip(2), k.roll(5, 2), 2 * v.flip(2))]
    ws = B.alloc_workspace(p)
    lines = ws.view(-1, 128) if ws.numel() % 128 == 0 else ws[:ws.numel() // 128 * 128].view(-1, 128)
    scores = torch.empty((p.batch, p.n_kv_heads, p.seq_len), device="cuda")
    call = _score_call(name, p, q, k, v, scores, ws)
    want = []
    for s in sets:
        call(*s)
        want.append(scores.clone())
    ws.fill_(0xA5)
    graph = torch.cuda.CUDAGraph()
    assert B.load().aha_exchange_looks(looks) == B.AHA_OK
    try:
        with torch.cuda.graph(graph):
            call(q, k, v)
    finally:
        B.load().aha_exchange_looks(4000)
    gen = torch.Generator(device="cuda").manual_seed(1)
    drawn = torch.rand((6, lines.shape[0], 1), generator=gen, device="cuda") < 0.5
    former = None
    for how in ("same bytes", "bytes of before"):
        for at, i in enumerate((1, 0, 1, 1, 0, 0)):
            for dst, src in zip((q, k, v), sets[i]):
                dst.copy_(src)
            # half of the workspace's lines (the same ones in three replays) hold what they held before the last replay,
            # the others what it left
            if how == "same bytes":
                lines.masked_fill_(drawn[at // 3], 0xA5)
            elif former is not None:
                lines.copy_(torch.where(drawn[at], former, lines))
            former = lines.clone()
            scores.fill_(-1.0)
            graph.replay()
            torch.cuda.synchronize()
            assert scores.equal(want[i]), (how, at)


@pytest.mark.gpu
def test_two_calls_in_a_graph():
    """Chosen rows behind windowed scores in one workspace: its value prior, the same for prompts with the same values,
    covers what lies behind the statistics of the first call and not these."""
    import torch
    hkv, window, n, d = 32, 64, 4096, 128
    gen = torch.Generator(device="cuda").manual_seed(3)
    q, k, v = (torch.randn((1, hkv, n, d), generator=gen, device="cuda", dtype=torch.bfloat16) for _ in range(3))
    p = B.Params(batch=1, n_q_heads=hkv, n_kv_heads=hkv, head_dim=d, seq_len=n, window=window, budget=n // 8,
                 recent=8).with_strides(q, k, v)
    rows = torch.arange(n - window, n, dtype=torch.int32, device="cuda").expand(1, hkv, window).contiguous()
    scores, chosen = (torch.empty((1, hkv, n), device="cuda") for _ in range(2))
    ws = B.alloc_workspace(p)
    sets, want = [q.clone(), q.flip(2), q.roll(1, 1)], []
    for s in sets:
        B.aha_prefill_scores(p, s, k, v, scores, ws)
        want.append(scores.clone())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        B.aha_prefill_scores(p, q, k, v, scores, ws)
        B.aha_prefill_scores_rows(p, q, k, v, rows, chosen, ws)
    for i in (1, 0, 2, 2, 0, 1):
        q.copy_(sets[i])
        graph.replay()
        torch.cuda.synchronize()
        assert scores.equal(want[i])
