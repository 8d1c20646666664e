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
    # in several rounds of the chip, up to 256 ranges; more where two launches would leave their last round nearly empty
    (16, 32768, True), (16, 49152, True),     # (x 101 ranges) 72.2, 58.3
    (8, 65536, True),      # 71.1, 54.9
    (64, 65536, True), (64, 98304, True),     # 871, 727
    (16, 131072, True),    # 276, 237
    (16, 163840, False),   # 349, 371
    (24, 131072, True), (24, 163840, True),   # 717, 553
    (2, 163840, True),     # 62.9, 51.5
    (128, 16384, True),
])
def test_ranges_of_a_problem_fit_the_chip(z, n, one):
    for group, window in ((1, 64), (2, 17), (3, 20)):
        assert _one_launch("aha_prefill_scores", _params(z, group, window, n)) == one


@pytest.mark.parametrize("z,n,d,prior,one", [
    # 225 to 256 rows from given normalisers (us: two launches, one)
    (8, 3600, 128, 1, False),     # 18.5, 19.9
    (4, 12000, 64, 1, False),     # 13.7, 15.4
    (16, 3600, 128, 1, False),    # 19.2, 20.3
    (8, 12000, 128, 1, True),     # 23.9, 22.3
    (32, 2300, 128, 1, True),     # 25.7, 19.6
    (8, 3600, 128, 0, True),
])
def test_few_steps_of_large_tiles(z, n, d, prior, one):
    for window in (58, 64):
        assert _one_launch("aha_prefill_scores_lse", _params(z, 4, window, n, d, value_prior=prior)) == one
    assert _one_launch("aha_prefill_scores_lse", _params(z, 4, 56, n, d, value_prior=prior))


# KV heads, group, window, keys, d, and a workspace that holds two launches; one launch, swept twice by more ranges than the
# chip holds at once, needs up to a sixth more
SMALLER = [(183, 4, 29, 13938, 64, 10805248), (89, 4, 100, 14177, 128, 7254272), (141, 2, 173, 22503, 64, 15051520),
           (43, 4, 114, 25641, 128, 6541312), (94, 4, 103, 36264, 64, 15998976)]


@pytest.mark.parametrize("z,group,window,n,d,size", SMALLER)
def test_workspace_of_two_launches_is_served(z, group, window, n, d, size):
    p = _params(z, group, window, n, d)
    assert B.workspace_bytes(p) > size
    assert _one_launch("aha_prefill_scores", p)
    for name in ("aha_prefill_scores", "aha_prefill_scores_lse"):
        _one_launch(name, p, size)
    assert not _one_launch("aha_prefill_scores", p, size)
    assert _call("aha_prefill_row_stats", p, size) == B.AHA_ERR_HIP
    assert _call("aha_prefill_scores_rows", p, size) != B.AHA_ERR_WORKSPACE
    for name in ("aha_prefill_scores", "aha_prefill_scores_lse", "aha_prefill_row_stats"):
        assert _call(name, p, size // 4) == B.AHA_ERR_WORKSPACE


@pytest.mark.parametrize("z,group,window,n,d,prior,size", [
    # sizes that were asked for when statistics took four bytes a value and norms and prior always lay in the workspace
    (64, 7, 32, 6233, 128, 1, 3726336), (8, 8, 64, 131072, 128, 1, 8923392), (22, 3, 57, 196890, 128, 1, 34848768),
    (42, 1, 398, 14322, 64, 1, 5339136), (11, 1, 73, 111119, 64, 1, 9912832), (256, 3, 41, 9749, 64, 1, 20109312),
    (171, 1, 271, 45870, 64, 1, 65446912), (89, 4, 100, 14177, 128, 1, 11581696),
    # held: short prompts, with a prior and without
    (61, 3, 1, 50, 64, 0, 28416), (212, 7, 2, 41, 128, 0, 91136), (253, 8, 1, 46, 64, 1, 112640), (44, 5, 49, 50, 128, 1, 99328),
    (50, 8, 31, 46, 128, 1, 111872),
    # two launches' sizes, which hold one launch as well
    (64, 7, 32, 3170, 64, 1, 1863424), (64, 5, 77, 7257, 64, 1, 3962368), (64, 7, 64, 6233, 128, 1, 3699200),
    (128, 3, 128, 77252, 64, 1, 41804800),
])
def test_one_launch_at_former_sizes(z, group, window, n, d, prior, size):
    p = _params(z, group, window, n, d, value_prior=prior)
    assert B.workspace_bytes(p) <= size
    assert _one_launch("aha_prefill_scores", p, size)


@pytest.mark.gpu
@pytest.mark.parametrize("z,group,window,n,d,size", SMALLER[:3])
def test_results_in_it(z, group, window, n, d, size):
    import torch
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n)
    q, k, v = (torch.randn((1, h, n, d), generator=gen, device="cuda").to(torch.bfloat16) for h in (z * group, z, z))
    p = _params(z, group, window, n, d).with_strides(q, k, v)
    got = []
    for have in (B.workspace_bytes(p), size):
        scores = torch.empty((1, z, n), dtype=torch.float32, device="cuda")
        B.aha_prefill_scores(p, q, k, v, scores, torch.full((have,), 0xA5, dtype=torch.uint8, device="cuda"))
        got.append(scores.double())
    # fp32 arithmetic on exact products: logits of a few tens carry 1e-5 absolute, which is the relative error of their
    # exponentials, on either side
    assert ((got[0] - got[1]).abs() <= 4e-4 * got[0] + 2e-7 * got[0].mean()).all()


@pytest.mark.parametrize("z,window,n,d,prior,one", [
    # several rounds of the chip (us: two launches, one)
    (80, 128, 2304, 128, 1, True),    # 55.6, 32.3
    (128, 32, 16384, 64, 1, True),    # 142, 110
    (173, 32, 2481, 64, 1, False),    # hardly more than one round
    (173, 32, 2481, 128, 1, True),    # (shorter ranges) 79.3, 50.0
    (64, 128, 16384, 128, 1, False),  # 151, 156
    (32, 96, 32768, 128, 1, False),   # 147, 162
    (64, 64, 16384, 64, 0, True),     # 54.4, 51.1
    (128, 64, 16384, 64, 0, False),   # 93.5, 99.1
    (8, 64, 88500, 64, 1, False),     # 60.4, 68.8
    (6, 96, 19416, 128, 1, True),     # one round, many ranges: 32.6, 22.4
    (1, 128, 12800, 128, 1, True),    # and few workgroups: 20.5, 13.4
    (2, 70, 12544, 64, 0, True),      # 15.4, 9.1
    (1, 128, 25600, 128, 0, True), (1, 128, 32768, 128, 0, True),   # 20.1, 12.6; 20.7, 12.7
    (11, 128, 26368, 128, 1, True),   # several rounds: 69.3, 50.9
    (37, 96, 37120, 128, 1, True),    # 261, 214
    (6, 128, 46080, 128, 1, True),    # few heads in many ranges: 70.9, 56.2
    (16, 128, 25600, 128, 0, True),   # 55.3, 52.2
    (16, 70, 38400, 128, 0, False),   # 65.5, 71.0
    (17, 70, 44544, 128, 0, False),   # 84.5, 93.6
    (8, 64, 71680, 64, 1, True),      # 51.9, 49.2
    (27, 64, 66560, 64, 1, True),     # 139, 131
    (27, 40, 66560, 64, 0, False),    # 86.2, 97.0
    (4, 128, 48640, 64, 1, True),     # 36.6, 33.4
])
def test_held_in_rounds(z, window, n, d, prior, one):
    assert _one_launch("aha_prefill_scores", _params(z, 1, window, n, d, value_prior=prior)) == one


@pytest.mark.parametrize("z,group,window,n,one", [
    # up to 32 rows with a prior, d = 128, in ranges of two steps (us: two launches, one): hardly more than one round
    (33, 8, 1, 8848, True),    # 62.5, 38.0
    (53, 4, 4, 4736, True),    # 52.4, 36.4
    (257, 1, 15, 537, True),   # 44.2, 32.9
    # many ranges to a problem
    (5, 1, 5, 103215, True),   # 85.3, 68.7
    (8, 1, 32, 131072, True),  # 139, 109
    (64, 1, 8, 131073, False), (8, 1, 32, 204550, False),
    # more of them than that: of four steps, in one round
    (2, 5, 1, 199437, True), (3, 1, 32, 168740, True), (1, 1, 32, 500000, True),
    (2, 1, 32, 270000, False),
])
def test_ranges_beside_value_rows(z, group, window, n, one):
    assert _one_launch("aha_prefill_scores", _params(z, group, window, n)) == one
