"""Which kernels a score call takes: one launch whose workgroups exchange their parts, or two launches.  Without a
GPU a call that is accepted fails at its first launch, and the reason names it."""
import ctypes

import pytest

from paper_2506_03762_amd import binding as B

PTR = ctypes.c_void_p(4096)


def _params(z, group, window, n, d=128, **more):
    heads = z * group
    return B.Params(batch=1, n_q_heads=heads, n_kv_heads=z, head_dim=d, seq_len=n, window=window, budget=max(1, n // 10),
                    recent=0, q_stride=(heads * n * d, n * d, d), k_stride=(z * n * d, n * d, d),
                    v_stride=(z * n * d, n * d, d), **more)


def _call(name, p, size):
    import torch
    if torch.cuda.is_available():
        pytest.skip("would launch with the dummy pointers")
    lib = B.load()
    tensors = {"aha_prefill_scores": 4, "aha_prefill_scores_lse": 5, "aha_prefill_scores_rows": 5,
               "aha_prefill_row_stats": 4}[name]
    return getattr(lib, name)(ctypes.byref(p.c()), *([PTR] * tensors), PTR if size else None, size, None)


def _one_launch(name, p, size=None):
    rc = _call(name, p, B.workspace_bytes(p) if size is None else size)
    assert rc == B.AHA_ERR_HIP, B.load().aha_last_error()
    return b"windowed score kernel" in B.load().aha_last_error()


@pytest.mark.parametrize("z,n,one", [
    # 33 to 64 rows, d = 128, ranges of 512 keys (us: two launches, one).  No more ranges than the chip
    # holds workgroups, whatever the length:
    (1, 262144, True), (1, 524288, False), (1, 1 << 20, False), (1, 1 << 30, False), (2, 262145, False),
    (8, 262145, False), (8, 300000, False), (8, 1 << 20, False), (24, 262145, False), (256, 1 << 20, False),
    # where a round of the chip holds enough problems whole
    (16, 32768, True),     # 71.7, 66.5
    (16, 49152, False),    # 101, 105
    (64, 65536, True),     # 565, 562
    (64, 98304, False),    # 867, 1003
    (24, 131072, True),    # 559, 471
    (24, 163840, False),   # 713, 793
    (128, 16384, True), (8, 65536, False),
])
def test_ranges_of_a_problem_fit_the_chip(z, n, one):
    for group, window in ((1, 64), (2, 17), (3, 20)):
        assert _one_launch("aha_prefill_scores", _params(z, group, window, n)) == one
