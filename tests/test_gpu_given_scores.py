"""bf16 scores from given row normalisers in one launch: every tile height at the edges of its row counts,
one and several ranges of one and several steps, as many keys as a workgroup keeps, ragged ends; the
workgroups that form missing ranges' priors themselves; replays of a graph."""
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
    (1, 3, 3, 43, 1100, 128), (2, 2, 1, 161, 400, 64), (1, 2, 6, 32, 1537, 128), (1, 2, 1, 193, 1300, 128),
    (1, 3, 8, 32, 257, 64), (1, 9, 8, 32, 6001, 128),
    (2, 100, 2, 32, 1300, 128),    # several steps, more workgroups than fit at once
    (4, 128, 1, 8, 2305, 64), (4, 64, 3, 32, 2600, 128),   # many steps
    (4, 128, 3, 32, 4700, 64),     # more keys than a workgroup keeps: two ranges
    (1, 3, 1, 32, 6500, 64),       # few heads and many ranges: two launches
    (1, 2, 1, 257, 900, 128),      # more rows than a tile: two launches
]


def _case(shape, prior=True):
    batch, hkv, group, window, n, d = shape
    w = synth.scaled(synth.C2, name="given", batch=batch, n_q_heads=hkv * group, n_kv_heads=hkv, head_dim=d,
                     seq_len=n, window=window, budget=max(24, n // 12), recent=min(20, n // 3))
    opts = Opts(value_prior=prior, pool=7 if batch == 1 else 17)
    return w, opts


def _normalisers(w, opts, q, k, v):
    """The rows' log-sum-exp as the library gives it, [b, Hq, window]."""
    import torch
    p = H.gpu_params(w, opts).with_strides(q, k, v)
    lse = torch.empty((w.batch, w.n_q_heads, w.window), dtype=torch.float32, device="cuda")
    B.aha_prefill_row_stats(p, q, k, lse, None, B.alloc_workspace(p))
    return p, lse


@pytest.mark.parametrize("prior", [True, False])
@pytest.mark.parametrize("shape", SHAPES)
def test_scores_and_missing_parts(shape, prior):
    w, opts = _case(shape, prior)
    inputs = synth.make_prefill(w)
    _, lse = _normalisers(w, opts, *(H.to_device(a, w.dtype) for a in inputs))
    lse = lse.cpu().numpy()
    got = H.run_scores_from_lse_gpu(w, opts, inputs, lse)
    ref = H.run_prefill_oracle(w, opts, inputs).scores
    # fp32 arithmetic on exact products: logits of a few tens carry 1e-5 absolute, which is the
    # relative error of their exponentials
    np.testing.assert_allclose(got, ref, rtol=2e-4, atol=2e-4 * 1e-3 * ref.mean())
    # a workgroup that looks once and does whatever is not there yet
    assert B.load().aha_exchange_looks(0) == B.AHA_OK
    try:
        alone = H.run_scores_from_lse_gpu(w, opts, inputs, lse)
    finally:
        B.load().aha_exchange_looks(4000)
    if w.group * w.window <= 256:  # (more rows: sums by atomics)
        assert np.array_equal(alone, got)


@pytest.mark.parametrize("shape", [(1, 4, 2, 32, 3000, 128), (1, 3, 8, 32, 900, 128), (4, 128, 1, 8, 2305, 64)])
def test_graph_replays(shape):
    """A replay reuses the call's tag: the words of the one before must be gone."""
    import torch
    w, opts = _case(shape)
    sets = [tuple(H.to_device(a, w.dtype) for a in synth.make_prefill(w, layer=i)) for i in range(2)]
    p, lse = _normalisers(w, opts, *sets[0])
    q, k, v = (t.clone() for t in sets[0])
    scores = torch.empty((w.batch, w.n_kv_heads, w.seq_len), dtype=torch.float32, device="cuda")
    ws = B.alloc_workspace(p)
    ws.fill_(0xA5)
    want = []
    for s in sets:
        B.aha_prefill_scores_lse(p, *s, lse, scores, ws)
        want.append(scores.clone())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        B.aha_prefill_scores_lse(p, q, k, v, lse, scores, ws)
    for i in (1, 0, 0, 1):
        for dst, src in zip((q, k, v), sets[i]):
            dst.copy_(src)
        scores.fill_(-1.0)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(scores, want[i])
        B.aha_prefill_scores_lse(p, *sets[1], lse, scores, ws)  # other work of the same workspace in between


def test_time_per_key():
    """Ranges that leave a round of the chip with parts of problems make a longer prompt slower per key."""
    import torch
    hkv, group, window, longest, d = 8, 4, 64, 1 << 20, 128
    q = torch.randn((1, hkv * group, window, d), device="cuda", dtype=torch.bfloat16)
    k, v = (torch.randn((1, hkv, longest, d), device="cuda", dtype=torch.bfloat16) for _ in range(2))
    lse = torch.full((1, hkv * group, window), 10.0, device="cuda")
    scores = torch.empty((1, hkv, longest), dtype=torch.float32, device="cuda")

    class LastRows:  # (only the last rows are read)
        def __init__(self, n):
            self.n = n

        def data_ptr(self):
            return q.data_ptr() - (self.n - window) * d * 2

    calls, times = [], ([], [])
    for n in (longest, 700000):
        p = B.Params(batch=1, n_q_heads=hkv * group, n_kv_heads=hkv, head_dim=d, seq_len=n, window=window, budget=64, recent=8,
                     q_stride=(0, window * d, d), k_stride=(0, longest * d, d), v_stride=(0, longest * d, d))
        calls.append((p, LastRows(n), k, v, lse, scores, B.alloc_workspace(p)))
    for i in range(24):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        B.aha_prefill_scores_lse(*calls[i % 2])
        b.record()
        torch.cuda.synchronize()
        times[i % 2].append(a.elapsed_time(b) / calls[i % 2][0].seq_len)
    # 0.87 ns per key either way; 1.24 for the longer one in 158 ranges to a problem
    assert sorted(times[0])[6] < 1.12 * sorted(times[1])[6]
