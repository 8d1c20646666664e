"""Selection at the edges of its launch variants: rows that just fill or just exceed the keys a
workgroup holds in registers, odd rows (no alignment), crowded threshold bins, infinities."""
import numpy as np
import pytest

from tests.test_gpu_parity import topk_both

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_cand", [1, 63, 512, 513, 1025, 2048, 2049, 4096, 4097, 6145, 8193, 12289,
                                    16385, 24577, 32768, 32769, 41023, 70001])
@pytest.mark.parametrize("kind", ["random", "few_values", "narrow"])
def test_topk_at_variant_edges(n_cand, kind):
    """Indices equal to the oracle's, bit for bit: scores are fp32 on both sides and ties go to
    the lower position."""
    rng = np.random.default_rng(n_cand)
    recent, sink = 5, min(3, n_cand - 1)
    n = n_cand + recent
    s = {"random": lambda: np.exp(rng.standard_normal((3, n))),
         "few_values": lambda: rng.integers(0, 3, (3, n)) * 0.25,  # crowded bin, many ties
         "narrow": lambda: 1.0 + rng.integers(0, 4 * n, (3, n)) * 2.0 ** -23}[kind]().astype(np.float32)
    s[0, rng.integers(0, n)] = np.inf       # one key far above the others: all share one bin
    s[1, rng.integers(0, n)] = -1.0
    for k in sorted({0, 1, (n_cand - sink) // 5, n_cand - sink}):
        got, want = topk_both(s[None], k + recent + sink, recent, sink=sink)
        assert np.array_equal(got, want), (n_cand, kind, k)


@pytest.mark.parametrize("n_cand", [300, 2049, 20000, 40000])
@pytest.mark.parametrize("sink", [0, 7])
def test_topk_survives_scores_of_all_ones(n_cand, sink):
    """A fill of 0xff bytes reads as NaN in every score: such scores rank below all others, ties to the
    lower position, and the list stays ascending and inside the sequence, also when they have to be
    selected."""
    import torch
    from paper_2506_03762_amd import binding as B
    rng = np.random.default_rng(n_cand)
    recent, n = 5, n_cand + 5
    bits = np.exp(rng.standard_normal((3, n))).astype(np.float32).view(np.uint32)
    bits[0, rng.random(n) < 0.5] = 0xffffffff
    bits[1] = 0xffffffff
    bits[2, rng.random(n) < 0.99] = 0xffffffff
    rank = np.where(bits == 0xffffffff, np.float32(-1), bits.view(np.float32))
    for k in (1, (n_cand - sink) // 2 + 9, n_cand - sink):
        p = B.Params(batch=1, n_q_heads=3, n_kv_heads=3, head_dim=64, seq_len=n, window=1,
                     budget=k + recent + sink, recent=recent, sink=sink)
        idx = torch.full((1, 3, p.budget), -7, dtype=torch.int32, device="cuda")
        B.aha_select_topk(p, torch.from_numpy(bits.view(np.float32)[None]).cuda(), idx)
        for got, s in zip(idx[0].cpu().numpy(), rank):
            best = sink + np.lexsort((np.arange(n_cand - sink), -s[sink:n_cand]))[:k]
            want = np.concatenate([np.arange(sink), np.sort(best), np.arange(n_cand, n)])
            assert np.array_equal(got, want), (n_cand, sink, k)
