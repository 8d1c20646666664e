"""Windowed bf16 scores of problems whose workgroups get one key step each (the value rows are
then requested together with the keys): ranges of 256 keys, a last one of a few keys, pooling
halos that reach into the neighbouring ranges, every tile height."""
import numpy as np
import pytest

from paper_2506_03762_amd import synth
from tests import harness as H
from tests.harness import Opts

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("n", [250, 256, 257, 519, 2050])
@pytest.mark.parametrize("group,window,pool", [(1, 9, 1), (2, 31, 7), (1, 100, 17), (7, 33, 3)])
def test_one_step_ranges(head_dim, n, group, window, pool):
    w = synth.scaled(synth.C2, name="one_step", batch=2, n_q_heads=3 * group, n_kv_heads=3,
                     head_dim=head_dim, seq_len=n, window=window, budget=120, recent=20)
    opts = Opts(pool=pool)
    inputs = synth.make_prefill(w)
    gpu, ref = H.run_prefill_gpu(w, opts, inputs), H.run_prefill_oracle(w, opts, inputs)
    # fp32 arithmetic on exact products: logits of a few tens carry 1e-5 absolute, which is the
    # relative error of their exponentials; a wrong neighbour in a pool of 17 would be 1e-2
    np.testing.assert_allclose(gpu.scores, ref.scores, rtol=2e-4,
                               atol=2e-4 * 1e-3 * ref.scores.mean())
    H.assert_sets_match(gpu.idx, ref.idx, ref.extra["rank_scores"], w)
