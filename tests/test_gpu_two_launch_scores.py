"""Windowed bf16 scores on the paths that larger problems take: two launches, the first of which forms the value prior
beside the row statistics, in ranges of one key step and of several; and the two-sweep kernel on ranges whose
norms and prior do not fit the LDS."""
import numpy as np
import pytest

from paper_2506_03762_amd import binding as B
from paper_2506_03762_amd import synth
from tests import harness as H
from tests.harness import Opts
from tests.test_score_routes import _one_launch, _params

TWO = [
    # batch, KV heads, group, window, n, d
    (11, 50, 1, 20, 250, 64),   # ranges of one step
    (1, 64, 1, 20, 8500, 64), (2, 16, 1, 32, 17000, 64),     # up to 32 rows
    (1, 1, 1, 64, 262500, 128), (1, 1, 2, 32, 262700, 64), (4, 2, 1, 33, 88600, 64),   # up to 64
    (1, 2, 4, 32, 66000, 128), (1, 3, 1, 65, 66001, 128), (1, 2, 3, 40, 65900, 128), (1, 1, 1, 100, 131500, 128),   # up to 128
    (1, 1, 1, 100, 131501, 64),
]
# (two sweeps by four workgroups per problem, 2560 keys each, where the LDS keeps 2048)
LONG_RANGES = [(1, 64, 5, 32, 8300, 64), (1, 56, 2, 100, 9100, 64)]


@pytest.mark.parametrize("shape", TWO)
def test_takes_two_launches(shape):
    batch, hkv, group, window, n, d = shape
    p = _params(batch * hkv, group, window, n, d)
    assert not _one_launch("aha_prefill_scores", p)


def _case(shape):
    batch, hkv, group, window, n, d = shape
    w = synth.scaled(synth.C2, name="two", batch=batch, n_q_heads=hkv * group, n_kv_heads=hkv, head_dim=d, seq_len=n,
                     window=window, budget=n // 12, recent=20)
    return w, Opts(pool=17 if n % 2 else 7), synth.make_prefill(w)


def _check(w, opts, inputs):
    gpu, ref = H.run_prefill_gpu(w, opts, inputs), H.run_prefill_oracle(w, opts, inputs)
    # fp32 arithmetic on exact products: logits of a few tens carry 1e-5 absolute, which is the
    # relative error of their exponentials; a wrong neighbour in a pool of 17 would be 1e-2
    np.testing.assert_allclose(gpu.scores, ref.scores, rtol=2e-4, atol=2e-4 * 1e-3 * ref.scores.mean())
    return gpu


@pytest.mark.gpu
@pytest.mark.parametrize("shape", TWO)
def test_scores(shape):
    _check(*_case(shape))


@pytest.mark.gpu
@pytest.mark.parametrize("shape", LONG_RANGES)
def test_ranges_longer_than_the_lds_keeps(shape):
    case = _case(shape)
    gpu = _check(*case)
    # a workgroup that looks once and does whatever is not there yet
    assert B.load().aha_exchange_looks(0) == B.AHA_OK
    try:
        alone = H.run_prefill_gpu(*case)
    finally:
        B.load().aha_exchange_looks(4000)
    assert np.array_equal(alone.scores, gpu.scores)


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [(1, 12, 8, 32, 6001, 128), (2, 9, 4, 57, 4100, 64), (1, 33, 8, 32, 1800, 128)])
def test_given_normalisers_of_a_full_tile(shape):
    """225 to 256 rows in one launch, several steps and ranges."""
    import torch
    w, opts, inputs = _case(shape)
    p = H.gpu_params(w, opts)
    q, k, v = (H.to_device(a, w.dtype) for a in inputs)
    lse = torch.empty((w.batch, w.n_q_heads, w.window), dtype=torch.float32, device="cuda")
    B.aha_prefill_row_stats(p.with_strides(q, k, v), q, k, lse, None, B.alloc_workspace(p))
    got = H.run_scores_from_lse_gpu(w, opts, inputs, lse.cpu().numpy())
    ref = H.run_prefill_oracle(w, opts, inputs).scores
    np.testing.assert_allclose(got, ref, rtol=2e-4, atol=2e-4 * 1e-3 * ref.mean())
    assert B.load().aha_exchange_looks(0) == B.AHA_OK
    try:
        alone = H.run_scores_from_lse_gpu(w, opts, inputs, lse.cpu().numpy())
    finally:
        B.load().aha_exchange_looks(4000)
    assert np.array_equal(alone, got)
