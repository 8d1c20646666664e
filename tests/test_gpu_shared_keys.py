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
