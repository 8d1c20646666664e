"""Keys and values whose tokens lie 512 MB apart: the rows of one load of the kernels whose waves share the keys are further
apart than a 32-bit lane offset reaches.  Against the same rows lying together."""
import pytest

from paper_2506_03762_amd import binding as B

pytestmark = pytest.mark.gpu

STRIDE, N, HEADS = 1 << 28, 70, 257


@pytest.fixture(scope="module")
def buffer():
    import torch
    if torch.cuda.mem_get_info()[0] < 60 << 30:
        pytest.skip("37 GB of device memory")
    t = [torch.empty((N - 1) * STRIDE + 2 * HEADS * 128, dtype=torch.bfloat16, device="cuda")]
    yield t[0]
    t.clear()
    torch.cuda.empty_cache()


def _inputs(buffer, hkv, group, window, d):
    import torch
    gen = torch.Generator(device="cuda").manual_seed(hkv + d)
    q, k, v = (torch.randn((1, h, N, d), generator=gen, device="cuda", dtype=torch.bfloat16) for h in (hkv * group, hkv, hkv))
    far = [buffer.as_strided((1, hkv, N, d), (0, d, STRIDE, 1), at) for at in (0, hkv * d)]
    for dst, src in zip(far, (k, v)):
        dst.copy_(src)
    p = B.Params(batch=1, n_q_heads=hkv * group, n_kv_heads=hkv, head_dim=d, seq_len=N, window=window, budget=20, recent=4)
    return p, q, (k, v), far


@pytest.mark.parametrize("hkv,group,window,d", [
    (257, 4, 64, 128), (3, 8, 64, 128), (3, 8, 60, 64),      # keys shared in one launch: 256 rows, 512, 480 with d = 64
    (2, 8, 70, 128), (3, 8, 70, 64), (2, 5, 32, 128),        # several tiles (the last one with a pool that is too wide otherwise)
])
def test_scores(buffer, hkv, group, window, d):
    import torch
    p, q, near, far = _inputs(buffer, hkv, group, window, d)
    if group * window <= 160:
        p.pool_kernel = 19
    got = []
    for k, v in (near, far):
        p = p.with_strides(q, k, v)
        scores = torch.full((1, hkv, N), float("nan"), device="cuda")
        B.aha_prefill_scores(p, q, k, v, scores, B.alloc_workspace(p))
        got.append(scores)
    if group * window > 512 or group * window <= 160:  # (sums by atomics)
        torch.testing.assert_close(got[1], got[0], rtol=1e-5, atol=0)
    else:
        assert got[1].equal(got[0])


def test_attention(buffer):
    import torch
    p, q, near, far = _inputs(buffer, 128, 4, 64, 128)
    got = []
    for k, v in (near, far):
        p = p.with_strides(q, k, v)
        size = B.window_attention_workspace_bytes(p)
        assert size == 128 * 2 * 8 * 32 * 130 * 4  # (two ranges of a step of 64 keys: waves share the keys)
        out = torch.full((1, 512, 64, 128), float("nan"), dtype=torch.bfloat16, device="cuda")
        B.aha_prefill_window_attention(p, q, k, v, out, None, torch.empty(size, dtype=torch.uint8, device="cuda"))
        got.append(out)
    assert got[1].equal(got[0])
