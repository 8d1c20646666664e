"""fp32 scores where a workgroup takes four rows (row statistics) and 64 keys (column sums), the
variants for problems with many workgroups; the small variants are covered by the tiny workload."""
import pytest

import oracle
from paper_2506_03762_amd import synth
from tests import harness as H
from tests.harness import Opts

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("n,group,window", [(1025, 2, 33),   # one key, one row past the last block
                                            (1153, 3, 22)])
def test_many_workgroups(head_dim, n, group, window):
    hkv, batch = 8, 4
    assert group * window * hkv * batch >= 2048 and (n + 15) // 16 * hkv * batch >= 2048
    w = synth.scaled(synth.C1, name="f32_many", batch=batch, n_q_heads=hkv * group, n_kv_heads=hkv,
                     head_dim=head_dim, seq_len=n, window=window, budget=200, recent=20)
    inputs = synth.make_prefill(w)
    gpu = H.run_prefill_gpu(w, Opts(), inputs)
    ref = H.run_prefill_oracle(w, Opts(), inputs)
    H.assert_scores_close(gpu.scores, ref.scores, w, Opts())
    H.assert_sets_match(gpu.idx, ref.idx, ref.extra["rank_scores"], w)
