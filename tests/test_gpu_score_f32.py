"""fp32 scores of problems large enough for the matrix core: ragged key and row blocks, one to many
row blocks, given row normalisers; the vector ALU's variants are covered by the tiny workload."""
import pytest

import oracle
from paper_2506_03762_amd import synth
from tests import harness as H
from tests.harness import Opts

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("n,group,window", [(1601, 1, 32), (1633, 1, 33), (999, 3, 40), (600, 4, 90)])
def test_matrix_core(head_dim, n, group, window):
    """Also with the rows' normalisers given."""
    import torch
    from paper_2506_03762_amd import binding as B
    from paper_2506_03762_amd import workload
    hkv, batch = 4, 2
    w = synth.scaled(synth.C1, name="f32_mfma", batch=batch, n_q_heads=hkv * group, n_kv_heads=hkv,
                     head_dim=head_dim, seq_len=n, window=window, budget=150, recent=20)
    assert batch * hkv * group * window * n >= 4e5
    inputs = synth.make_prefill(w)
    gpu, ref = H.run_prefill_gpu(w, Opts(), inputs), H.run_prefill_oracle(w, Opts(), inputs)
    H.assert_scores_close(gpu.scores, ref.scores, w, Opts())
    H.assert_sets_match(gpu.idx, ref.idx, ref.extra["rank_scores"], w)
    p = H.gpu_params(w)
    q, k, v = (workload.to_device(x, w.dtype) for x in inputs)
    p = p.with_strides(q, k, v)
    lse = torch.empty((batch, hkv * group, window), device="cuda")
    got = torch.empty((batch, hkv, n), device="cuda")
    B.aha_prefill_row_stats(p, q, k, lse, None, B.alloc_workspace(p))
    B.aha_prefill_scores_lse(p, q, k, v, lse, got, B.alloc_workspace(p))
    H.assert_scores_close(got.double().cpu().numpy(), ref.scores, w, Opts())


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
