"""Windowed bf16 scores in one launch whose workgroups exchange their ranges' statistics: every tile
height and number of tiles at the edges of their row counts, one and several ranges, ranges of one and
several steps, ragged ends; the workgroups that do missing parts themselves; replays of a graph."""
import numpy as np
import pytest

from paper_2506_03762_amd import binding as B
from paper_2506_03762_amd import synth
from tests import harness as H
from tests.harness import Opts

pytestmark = pytest.mark.gpu

SHAPES = [
    # batch, KV heads, group, window, n, d: rows = group * window
    (1, 2, 1, 1, 37, 128), (2, 3, 1, 32, 513, 64), (1, 3, 3, 11, 1030, 128), (2, 2, 4, 16, 770, 64),
    (1, 2, 5, 13, 3000, 128), (1, 4, 3, 32, 1025, 128), (2, 2, 1, 97, 700, 64), (1, 3, 4, 32, 511, 128),
    (1, 64, 1, 20, 7000, 64),      # ranges of four steps
    (1, 64, 2, 32, 8300, 128),     # ranges of two steps, more workgroups than fit at once
    (1, 3, 3, 43, 1100, 128), (2, 2, 4, 48, 400, 64), (1, 2, 1, 193, 1300, 128), (1, 3, 8, 32, 257, 64),  # two tiles, held
    (2, 16, 3, 43, 2100, 128), (1, 32, 7, 32, 2305, 128), (1, 32, 8, 32, 2048, 64),  # one tile, two sweeps
    (1, 32, 4, 32, 6500, 64),
    (1, 2, 1, 257, 900, 128), (2, 2, 3, 128, 1537, 64), (1, 3, 5, 77, 640, 128), (1, 2, 8, 64, 2100, 128),  # two tiles
    (2, 64, 8, 64, 1300, 128),     # two tiles, ranges longer than the LDS keeps
    (1, 2, 1, 513, 1200, 128),     # more rows than two tiles: two launches
]


def _workload(batch, hkv, group, window, n, d):
    return synth.scaled(synth.C2, name="window", batch=batch, n_q_heads=hkv * group, n_kv_heads=hkv,
                        head_dim=d, seq_len=n, window=window, budget=max(24, n // 12), recent=min(20, n // 3))


def _on_gpu(w, opts, inputs):
    p = H.gpu_params(w, opts)
    q, k, v = (H.to_device(a, w.dtype) for a in inputs)
    return p.with_strides(q, k, v), q, k, v


@pytest.mark.parametrize("prior", [True, False])
@pytest.mark.parametrize("shape", SHAPES)
def test_scores_and_missing_parts(shape, prior):
    w, opts = _workload(*shape), Opts(value_prior=prior, pool=7 if shape[0] == 1 else 17)
    inputs = synth.make_prefill(w)
    gpu, ref = H.run_prefill_gpu(w, opts, inputs), H.run_prefill_oracle(w, opts, inputs)
    # fp32 arithmetic on exact products: logits of a few tens carry 1e-5 absolute, which is the
    # relative error of their exponentials
    np.testing.assert_allclose(gpu.scores, ref.scores, rtol=2e-4, atol=2e-4 * 1e-3 * ref.scores.mean())
    H.assert_sets_match(gpu.idx, ref.idx, ref.extra["rank_scores"], w)
    # a workgroup that looks once and does whatever is not there yet
    assert B.load().aha_exchange_looks(0) == B.AHA_OK
    try:
        alone = H.run_prefill_gpu(w, opts, inputs)
    finally:
        B.load().aha_exchange_looks(4000)
    if w.group * w.window <= 512:  # (more rows: sums by atomics)
        assert np.array_equal(alone.scores, gpu.scores)


@pytest.mark.parametrize("shape", [(1, 4, 2, 32, 3000, 128), (1, 3, 8, 32, 900, 128), (1, 2, 8, 64, 2100, 64),
                                   (2, 16, 3, 43, 2100, 128)])
def test_graph_replays(shape):
    """A replay reuses the call's tag: the words of the one before must be gone."""
    import torch
    w, opts = _workload(*shape), Opts()
    sets = [_on_gpu(w, opts, synth.make_prefill(w, layer=i)) for i in range(3)]
    p = sets[0][0]
    q, k, v = (t.clone() for t in sets[0][1:])
    scores = torch.empty((w.batch, w.n_kv_heads, w.seq_len), dtype=torch.float32, device="cuda")
    ws = B.alloc_workspace(p)
    ws.fill_(0xA5)
    want = []
    for s in sets:
        B.aha_prefill_scores(p, *s[1:], scores, ws)
        want.append(scores.clone())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        B.aha_prefill_scores(p, q, k, v, scores, ws)
    for i in (1, 2, 0, 0, 2, 1):
        for dst, src in zip((q, k, v), sets[i][1:]):
            dst.copy_(src)
        scores.fill_(-1.0)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(scores, want[i])
        if i == 2:  # other work of the same workspace in between
            B.aha_prefill_scores(p, *sets[1][1:], scores, ws)


def test_two_streams_at_once():
    """Launches side by side, each more than the chip holds: neither waits for the other's end."""
    import torch
    w, opts = _workload(1, 32, 2, 32, 9000, 128), Opts()
    p, q, k, v = _on_gpu(w, opts, synth.make_prefill(w))
    outs = [torch.empty((1, 32, 9000), dtype=torch.float32, device="cuda") for _ in range(3)]
    spaces = [B.alloc_workspace(p) for _ in range(3)]
    B.aha_prefill_scores(p, q, k, v, outs[2], spaces[2])
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(2)]
    for _ in range(20):
        for s, o, ws in zip(streams, outs, spaces):
            with torch.cuda.stream(s):
                B.aha_prefill_scores(p, q, k, v, o, ws)
    torch.cuda.synchronize()
    assert torch.equal(outs[0], outs[2]) and torch.equal(outs[1], outs[2])


def test_beside_other_work():
    """A problem with as many ranges as the chip holds workgroups, beside launches that fill the chip for
    milliseconds: the ones of its workgroups that run must not keep the chip while they wait for the others."""
    import torch
    def problem(hkv, group, n, window):
        q, k, v = (torch.randn((1, h, n, 128), device="cuda", dtype=torch.bfloat16) for h in (hkv * group, hkv, hkv))
        p = B.Params(batch=1, n_q_heads=hkv * group, n_kv_heads=hkv, head_dim=128, seq_len=n, window=window, budget=512,
                     recent=16).with_strides(q, k, v)
        return p, q, k, v, torch.empty((1, hkv, n), dtype=torch.float32, device="cuda"), B.alloc_workspace(p)
    other, one = problem(8, 4, 32768, 32768), problem(1, 1, 131072, 64)
    jobs = [lambda: [B.aha_prefill_scores(*other) for _ in range(2)], lambda: [B.aha_prefill_scores(*one) for _ in range(40)]]
    streams = [torch.cuda.Stream() for _ in range(2)]

    def span(which):
        """ms until the given jobs, a stream each, are done"""
        torch.cuda.synchronize()
        begin, ends = torch.cuda.Event(enable_timing=True), []
        begin.record(streams[which[0]])
        for i in which:
            with torch.cuda.stream(streams[i]):
                jobs[i]()
                ends.append(torch.cuda.Event(enable_timing=True))
                ends[-1].record()
        torch.cuda.synchronize()
        return max(begin.elapsed_time(e) for e in ends)

    span((0,)), span((1,))
    want = one[4].clone()
    alone = span((0,)) + span((1,))
    together = min(span((0, 1)) for _ in range(3))
    # one after the other they take 18 ms, together 19.5; 48 while a workgroup waited up to 5 ms at a time and all of
    # them then formed the same parts
    assert together < 1.8 * alone, (together, alone)
    assert torch.equal(one[4], want)
