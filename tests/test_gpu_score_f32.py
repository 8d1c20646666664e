"""fp32 scores on the matrix core: ragged key and row blocks, one to many row blocks, given row
normalisers, chosen rows; and on the vector ALU with four rows or keys per group of four lanes (the
variants with one of each are the tiny workload's)."""
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
    """More workgroups than the chip holds at a time."""
    hkv, batch = 8, 4
    assert group * window * hkv * batch >= 2048 and (n + 15) // 16 * hkv * batch >= 2048
    w = synth.scaled(synth.C1, name="f32_many", batch=batch, n_q_heads=hkv * group, n_kv_heads=hkv,
                     head_dim=head_dim, seq_len=n, window=window, budget=200, recent=20)
    inputs = synth.make_prefill(w)
    gpu = H.run_prefill_gpu(w, Opts(), inputs)
    ref = H.run_prefill_oracle(w, Opts(), inputs)
    H.assert_scores_close(gpu.scores, ref.scores, w, Opts())
    H.assert_sets_match(gpu.idx, ref.idx, ref.extra["rank_scores"], w)


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("batch,hkv,n,group,window", [
    (4, 8, 1025, 1, 8),      # four keys per quad, one key past the last 64; one row
    (16, 8, 150, 2, 9),      # four rows, a last group of two; one key
    (16, 8, 257, 3, 7),      # four of both, a last group of one row
    (8, 8, 90, 4, 8),        # 32 rows and few pairs: four rows, one key
])
def test_vector_variants(head_dim, batch, hkv, n, group, window):
    """Four from 2048 workgroups of one row, or of 16 keys, on; the value prior's tiles follow the rows'
    workgroups in the same launch."""
    z, rows = batch * hkv, group * window
    assert rows < 24 or z * rows * n < 2e5          # not on the matrix core
    assert z * rows >= 2048 or z * ((n + 15) // 16) >= 2048
    w = synth.scaled(synth.C1, name="f32_vector", batch=batch, n_q_heads=hkv * group, n_kv_heads=hkv,
                     head_dim=head_dim, seq_len=n, window=window, budget=n // 4, recent=8)
    inputs = synth.make_prefill(w)
    gpu, ref = H.run_prefill_gpu(w, Opts(), inputs), H.run_prefill_oracle(w, Opts(), inputs)
    H.assert_scores_close(gpu.scores, ref.scores, w, Opts())
    H.assert_sets_match(gpu.idx, ref.idx, ref.extra["rank_scores"], w)


@pytest.mark.parametrize("head_dim", [64, 128])
def test_chosen_rows_on_the_matrix_core(head_dim):
    """Rows anywhere in the sequence, in any order and repeated: a block of 32 of them spans most of it."""
    import numpy as np
    from tests.test_gpu_row_stats import run_scores_rows
    w = synth.scaled(synth.C1, name="f32_rows", batch=2, n_q_heads=12, n_kv_heads=4, head_dim=head_dim,
                     seq_len=1300, window=35, budget=150, recent=20)
    assert 2 * 4 * 3 * 35 * 1300 >= 2e5
    inputs, opts = synth.make_prefill(w), Opts()
    rows = np.random.default_rng(head_dim).integers(0, w.seq_len, (2, 12, 35))
    rows[:, :, :3] = (0, w.seq_len - 1, w.seq_len - 1)
    want = oracle.prefill_scores_rows(*inputs, rows, H.oracle_cfg(w, opts))
    H.assert_scores_close(run_scores_rows(w, opts, inputs, rows), want, w, opts)
