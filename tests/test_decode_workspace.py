"""The generation step's split follows the workspace: the workspace_bytes() of the plan, the smaller size of
the former count of splits, none where a head may keep one workgroup."""
import ctypes

import numpy as np
import pytest

from paper_2506_03762_amd import binding as B


def _params(z, group, d, live, dtype=B.AHA_BF16):
    return B.Params(batch=1, n_q_heads=z * group, n_kv_heads=z, head_dim=d, seq_len=0, window=0, budget=live - 1,
                    recent=16, dtype=dtype)


def _up(x):
    return (x + 255) // 256 * 256


@pytest.mark.parametrize("z,group,d,live,former", [
    (96, 8, 128, 1537, 3), (48, 5, 128, 3073, 6), (64, 4, 64, 1537, 4), (128, 8, 128, 1537, 1), (128, 4, 128, 801, 1),
])
def test_smaller_workspaces_are_served(z, group, d, live, former):
    import torch
    if torch.cuda.is_available():
        pytest.skip("would launch with the dummy pointers")
    p = _params(z, group, d, live)
    sps = -(-live // former)
    need = 0 if former == 1 else _up(4 * z * group * live) + _up(4 * z * -(-live // sps) * group * (d + 4))
    assert B.workspace_bytes(p) > need
    ptr = ctypes.c_void_p(4096)
    def call(bytes_):
        return B.load().aha_decode_step(ctypes.byref(p.c()), *([ptr] * 8), live, live, ptr, ptr if bytes_ else None,
                                        bytes_, None)
    for have in (need, B.workspace_bytes(p) - 1, B.workspace_bytes(p)):
        assert call(have) == B.AHA_ERR_HIP  # (accepted: it is the launch that finds no GPU)
    if need:
        assert call(need - 1) == B.AHA_ERR_WORKSPACE


@pytest.mark.gpu
@pytest.mark.parametrize("z,group,d,live", [(96, 8, 128, 1537), (128, 8, 128, 1537), (128, 4, 128, 801), (128, 5, 64, 97),
                                            (40, 4, 128, 2081)])
def test_results_do_not_depend_on_it(z, group, d, live):
    import torch
    p = _params(z, group, d, live)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(live)
    def rand(*shape):
        return torch.randn(shape, generator=gen, device="cuda").to(torch.bfloat16)
    first = B.CompactCache.empty(p)
    first.k.copy_(rand(*first.k.shape))
    first.v.copy_(rand(*first.v.shape))
    first.scores.copy_(torch.rand(first.scores.shape, generator=gen, device="cuda"))
    first.pos.copy_(torch.arange(live, device="cuda", dtype=torch.int32).expand_as(first.pos))
    first.free_slot.fill_(live // 2)
    q, k, v = rand(1, z * group, d), rand(1, z, d), rand(1, z, d)
    got = []
    sps = -(-live // -(-256 // z))
    former = _up(4 * z * group * live) + _up(4 * z * -(-live // sps) * group * (d + 4)) if z < 128 else 0
    for size in (B.workspace_bytes(p), former):
        c = B.CompactCache(*(getattr(first, n).clone() for n in ("k", "v", "scores", "pos", "free_slot")))
        ws = torch.full((size,), 0xA5, dtype=torch.uint8, device="cuda") if size else None
        out = torch.empty_like(q)
        B.aha_decode_step(p, q, k, v, c.k, c.v, c.scores, c.pos, c.free_slot, 6 * live, out, ws)
        got.append([t.double().cpu().numpy() for t in (out, c.scores, c.pos, c.free_slot, c.k, c.v)])
    a, b = got
    # one unit of the rounded output (2^-7 of the value at most) and the weights' 2^-17 of its size;
    # running scores: sums of some ten fp32 terms of at most 1
    rms = np.sqrt((b[0] ** 2).mean(-1, keepdims=True))
    assert (np.abs(a[0] - b[0]) <= 2.0 ** -7 * np.abs(b[0]) + 2.0 ** -15 * 3 * rms).all()
    np.testing.assert_allclose(a[1], b[1], rtol=1e-5, atol=1e-7)
    for x, y in zip(a[2:], b[2:]):
        assert np.array_equal(x, y)


NO_ROOM = [
    # heads, group, d, live slots: a head may keep one workgroup, whatever is passed as workspace
    (96, 4, 128, 801), (87, 4, 128, 899), (114, 4, 64, 1053), (127, 4, 128, 600), (128, 4, 128, 801), (128, 8, 64, 1111),
    (129, 8, 128, 801), (144, 6, 128, 97), (137, 7, 128, 1537),
]


@pytest.mark.parametrize("z,group,d,live", NO_ROOM)
def test_steps_that_need_no_workspace(z, group, d, live):
    import torch
    if torch.cuda.is_available():
        pytest.skip("would launch with the dummy pointers")
    p, ptr = _params(z, group, d, live), ctypes.c_void_p(4096)
    assert B.workspace_bytes(p) > 0
    for workspace, size in ((None, 0), (None, 1 << 30), (ptr, 0), (ptr, 4096), (ctypes.c_void_p(4096 + 16), 1 << 30)):
        rc = B.load().aha_decode_step(ctypes.byref(p.c()), *([ptr] * 8), live, live, ptr, workspace, size, None)
        assert rc == B.AHA_ERR_HIP, (workspace, size)  # (accepted: it is the launch that finds no GPU)


@pytest.mark.gpu
@pytest.mark.parametrize("z,group,d,live", NO_ROOM)
def test_results_without_one(z, group, d, live):
    import torch
    p = _params(z, group, d, live)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(live)
    def rand(*shape):
        return torch.randn(shape, generator=gen, device="cuda").to(torch.bfloat16)
    first = B.CompactCache.empty(p)
    first.k.copy_(rand(*first.k.shape))
    first.v.copy_(rand(*first.v.shape))
    first.scores.copy_(torch.rand(first.scores.shape, generator=gen, device="cuda"))
    first.pos.copy_(torch.arange(live, device="cuda", dtype=torch.int32).expand_as(first.pos))
    first.free_slot.fill_(live - 1)
    q, k, v = rand(1, z * group, d), rand(1, z, d), rand(1, z, d)
    size, got = B.workspace_bytes(p), []
    space = torch.full((size + 512,), 0xA5, dtype=torch.uint8, device="cuda")
    for ws in (space[:size], None, space[16:16 + size]):
        c = B.CompactCache(*(getattr(first, n).clone() for n in ("k", "v", "scores", "pos", "free_slot")))
        out = torch.empty_like(q)
        B.aha_decode_step(p, q, k, v, c.k, c.v, c.scores, c.pos, c.free_slot, 6 * live, out, ws)
        got.append([t.double().cpu().numpy() for t in (out, c.scores, c.pos, c.free_slot, c.k, c.v)])
    a, b, c = got
    assert all(np.array_equal(x, y) for x, y in zip(b, c))
    # as above: one unit of the rounded output, the weights' 2^-17 (without a split at 128 heads) of its size
    rms = np.sqrt((b[0] ** 2).mean(-1, keepdims=True))
    assert (np.abs(a[0] - b[0]) <= 2.0 ** -7 * np.abs(b[0]) + 2.0 ** -15 * 3 * rms).all()
    np.testing.assert_allclose(a[1], b[1], rtol=1e-5, atol=1e-7)
    for x, y in zip(a[2:], b[2:]):
        assert np.array_equal(x, y)


@pytest.mark.parametrize("z,group,d,live,split", [
    # us in one launch, split
    (129, 4, 128, 801, False),    # 22.4, 23.9
    (129, 5, 64, 801, False),     # 15.1, 16.5
    (129, 8, 128, 801, True), (144, 8, 128, 300, True), (136, 6, 128, 2500, True),
    (145, 8, 128, 300, False), (192, 8, 128, 1537, False),   # 41.1, 43.6
])
def test_most_heads_that_are_split(z, group, d, live, split):
    assert (B.workspace_bytes(_params(z, group, d, live)) > 0) == split
