"""One generation step over the ways a head's slots are divided (one workgroup per head; split on
the vector ALU; split on the matrix core) at the edges of their tiles: one slot, a last block of
a few slots, the new token in the first, the last and a middle slot."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _step(dtype, z, group, d, budget, seed, stale=None, masked=0):
    import torch
    from paper_2506_03762_amd import binding as B
    rng = np.random.default_rng(seed)
    live, n = budget + 1, 5 * budget + 7
    recent, sink = min(5, budget // 2), 1 if budget > 12 else 0
    p = B.Params(batch=1, n_q_heads=z * group, n_kv_heads=z, head_dim=d, seq_len=0, window=0,
                 budget=budget, recent=recent, sink=sink, dtype=dtype)
    tdt = torch.float32 if dtype == B.AHA_F32 else torch.bfloat16
    def dev(*shape):
        return torch.from_numpy(rng.standard_normal(shape).astype(np.float32)).to(tdt).cuda()
    c = B.CompactCache.empty(p)
    c.k.copy_(dev(*c.k.shape))
    c.v.copy_(dev(*c.v.shape))
    q, k, v = dev(1, z * group, d), dev(1, z, d), dev(1, z, d)
    if masked:  # dots of -inf in the first slots
        q[..., 0] = q[..., 0].abs() + 0.5
        k[..., 0] = 0
        c.k[0, :, :masked, 0] = float("-inf")
    fs = rng.integers(0, live, z)
    fs[:3] = [0, live - 1, live // 2][:z]
    pos = np.stack([np.insert(rng.permutation(n - recent)[:budget - recent].tolist() +
                              list(range(n - recent, n)), f, -1) for f in fs]).astype(np.int32)
    score = np.exp(rng.standard_normal((z, live))).astype(np.float32)
    c.pos[0, :, :live] = torch.from_numpy(pos).cuda()
    c.scores[0, :, :live] = torch.from_numpy(score).cuda()
    c.free_slot[0] = torch.from_numpy(fs.astype(np.int32)).cuda()
    # the step in float64
    K, V, Q = (t.double().cpu().numpy() for t in (c.k[0, :, :live], c.v[0, :, :live],
                                                  q.reshape(z, group, d)))
    rows = np.arange(z)
    if stale is not None:  # what the free slot held before the step
        for t in (c.k, c.v, c.scores):
            t[0, rows, fs] = stale
    K[rows, fs], V[rows, fs] = k[0].double().cpu().numpy(), v[0].double().cpu().numpy()
    dots = np.einsum("zgd,zsd->zgs", Q, K)
    def softmax(x):
        e = np.exp(x - x.max(-1, keepdims=True))
        return e / e.sum(-1, keepdims=True)
    lam = max(np.sqrt(2 * max(np.log((n + 1) / budget), 0) / d), d ** -0.5)
    out = np.einsum("zgs,zsd->zgd", softmax(dots * d ** -0.5), V)
    f = score.astype(np.float64)
    f[rows, fs] = 0
    f += softmax(dots * lam).sum(1)
    where = pos.copy()
    where[rows, fs] = n
    got = torch.full((1, z * group, d), float("nan"), dtype=tdt, device="cuda")
    ws = torch.full((max(256, B.workspace_bytes(p)),), 0xA5, dtype=torch.uint8, device="cuda")
    B.aha_decode_step(p, q, k, v, c.k, c.v, c.scores, c.pos, c.free_slot, n + 1, got, ws)
    got = got.double().cpu().numpy().reshape(z, group, d)
    assert np.array_equal(c.k[0, :, :live].double().cpu().numpy(), K)
    assert np.array_equal(c.v[0, :, :live].double().cpu().numpy(), V)
    gf = c.scores[0, :, :live].double().cpu().numpy()
    # fp32 sums of products of up to d terms: an absolute 1e-5 on logits of some tens
    np.testing.assert_allclose(gf, f, rtol=1e-4, atol=1e-6)
    for i in range(z):
        free = (where[i] < n + 1 - recent) & (where[i] >= sink)
        if not free.any():
            continue
        order = np.lexsort((-where[i], np.where(free, f[i], np.inf)))
        victim = int(c.free_slot[0, i])
        assert f[i, victim] <= f[i, order[0]] * (1 + 1e-4) and free[victim]
        assert int(c.pos[0, i, victim]) == -1
    return got, out


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("z,group", [(3, 1), (5, 3), (2, 4), (7, 5), (4, 8), (100, 2), (97, 8),
                                     (130, 4), (128, 8)])
@pytest.mark.parametrize("budget", [1, 30, 31, 127, 128, 330, 1030])
def test_step_against_float64(dtype, d, z, group, budget):
    from paper_2506_03762_amd import binding as B
    got, out = _step(B.AHA_F32 if dtype == "f32" else B.AHA_BF16, z, group, d, budget,
                     z * 1000 + budget + d)
    rms = np.sqrt((out ** 2).mean(-1, keepdims=True))
    if dtype == "f32":
        assert (np.abs(got - out) <= 2e-5 * rms + 1e-5 * np.abs(out)).all()
        return
    # half a unit of the rounded output (bf16 has 8 significant bits: half a unit is at most 2^-8
    # of the value), and the weights: fp32, or the sum of two bf16 numbers, 2^-17 each
    assert (np.abs(got - out) <= 2.0 ** -8 * np.abs(out) * 1.01 + 2.0 ** -15 * 3 * rms + 1e-6).all()


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("z,group", [(3, 1), (3, 4), (4, 8), (100, 4), (128, 4), (128, 8)])
@pytest.mark.parametrize("budget", [30, 100, 330])
def test_the_free_slots_old_contents_are_not_used(d, z, group, budget):
    """The slot is overwritten by the step, whatever it held; in the second head it is the last slot,
    as after a compaction, and the last block of slots is ragged."""
    from paper_2506_03762_amd import binding as B
    got, out = _step(B.AHA_BF16, z, group, d, budget, budget + d, stale=float("nan"))
    rms = np.sqrt((out ** 2).mean(-1, keepdims=True))
    assert (np.abs(got - out) <= 2.0 ** -8 * np.abs(out) * 1.01 + 2.0 ** -15 * 3 * rms + 1e-6).all()


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("z,group,budget", [(3, 4, 30), (3, 4, 1030), (5, 5, 330), (4, 8, 100)])
def test_output_weights_keep_fp32(d, z, group, budget):
    """Two slots weigh a third or so each, a few 1e-5 apart, and their value rows of 256 cancel: what is
    left is the error of the weights.  (A third slot, with values of 0, holds the largest dot.)"""
    import torch
    from paper_2506_03762_amd import binding as B
    rng = np.random.default_rng(d + budget)
    n, recent, live = 5 * budget, 5, budget + 1
    p = B.Params(batch=1, n_q_heads=z * group, n_kv_heads=z, head_dim=d, seq_len=0, window=0,
                 budget=budget, recent=recent, dtype=B.AHA_BF16)
    c = B.CompactCache.empty(p)
    c.k.zero_()
    c.scores.zero_()
    c.v.copy_(torch.from_numpy(rng.standard_normal(tuple(c.v.shape))))
    c.pos.copy_(torch.arange(live, device="cuda", dtype=torch.int32).expand_as(c.pos))
    c.free_slot.fill_(budget)
    c.k[0, :, :, 0] = -128                                # logits of -11 or -16
    c.k[0, :, 7:9, 0] = 0                                 # and of 0 and a few 1e-5
    c.k[0, :, 8, 1:9] = 2.0 ** -13
    c.k[0, :, 9, 0] = 8
    c.v[0, :, 9] = 0
    c.v[0, :, 7] = 256
    c.v[0, :, 8] = -256
    q = torch.from_numpy(rng.standard_normal((1, z * group, d))).to(torch.bfloat16).cuda()
    q[..., 0] = 1
    new = torch.zeros((1, z, d), dtype=torch.bfloat16, device="cuda")
    knew = c.k[0, :, 0].clone()
    K, V, Q = (t.double().cpu().numpy() for t in (c.k[0, :, :live], c.v[0, :, :live], q.reshape(z, group, d)))
    V[:, budget] = 0
    s = np.einsum("zgd,zsd->zgs", Q, K) * d ** -0.5
    w = np.exp(s - s.max(-1, keepdims=True))
    ref = np.einsum("zgs,zsd->zgd", w / w.sum(-1, keepdims=True), V)
    out = torch.empty_like(q)
    ws = torch.empty((max(256, B.workspace_bytes(p)),), dtype=torch.uint8, device="cuda")
    B.aha_decode_step(p, q, knew, new, c.k, c.v, c.scores, c.pos, c.free_slot, n, out, ws)
    err = np.abs(out.double().cpu().numpy().reshape(ref.shape) - ref)
    # half a unit of the output; of 256 times the weights' sum of 1: an exponential's last bit (2^-23),
    # the normalisation's and the products' roundings (2^-24 each, at most four of them).  (The two
    # dots are of 1e-4: an error of theirs would show in the weights' difference.)
    assert (err <= 2.0 ** -8 * 1.01 * np.abs(ref) + 2.0 ** -21 * 256).all(), err.max()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("z,group,budget,masked", [
    (3, 1, 1030, 130), (3, 4, 1030, 40), (3, 4, 1030, 130), (4, 8, 330, 130), (100, 2, 330, 130), (128, 8, 330, 130)])
def test_slots_with_dots_of_minus_infinity(dtype, z, group, budget, masked):
    """They weigh nothing, also where a block or a whole range of slots has no others (ranges of 61
    slots in the cases of 3 heads)."""
    from paper_2506_03762_amd import binding as B
    got, out = _step(B.AHA_F32 if dtype == "f32" else B.AHA_BF16, z, group, 128, budget, budget, masked=masked)
    rms = np.sqrt((out ** 2).mean(-1, keepdims=True))
    if dtype == "f32":
        assert (np.abs(got - out) <= 2e-5 * rms + 1e-5 * np.abs(out)).all()
    else:
        assert (np.abs(got - out) <= 2.0 ** -8 * np.abs(out) * 1.01 + 2.0 ** -15 * 3 * rms + 1e-6).all()


@pytest.mark.parametrize("d,live", [(64, 64), (128, 32)])
@pytest.mark.parametrize("group", [1, 4])
def test_the_waves_small_parts_add_up(d, live, group):
    """Slots of equal weight, one per group of lanes: the first wave's part of the output is 1, each of
    the other fifteen's 0.9 of half a unit of that.  Added to it one by one, all of those would be lost."""
    import torch
    from paper_2506_03762_amd import binding as B
    z, budget, n = 3, live - 1, 5 * live
    rows = live // 16
    p = B.Params(batch=1, n_q_heads=z * group, n_kv_heads=z, head_dim=d, seq_len=0, window=0,
                 budget=budget, recent=5, dtype=B.AHA_F32)
    c = B.CompactCache.empty(p)
    c.k.zero_()
    c.scores.zero_()
    c.v.fill_(0.9 * 2.0 ** -24 * live / rows)
    new = c.v[0, :, 0].clone().unsqueeze(0)
    c.v[0, :, 0] = live
    c.pos.copy_(torch.arange(live, device="cuda", dtype=torch.int32).expand_as(c.pos))
    c.free_slot.fill_(budget)
    ref = (c.v[0, :, :budget].double().sum(1) + new[0].double()) / live
    ref = ref.cpu().numpy()[:, None]
    q = torch.randn((1, z * group, d), device="cuda")
    out = torch.empty_like(q)
    ws = torch.empty((max(256, B.workspace_bytes(p)),), dtype=torch.uint8, device="cuda")
    B.aha_decode_step(p, q, torch.zeros_like(new), new, c.k, c.v, c.scores, c.pos, c.free_slot, n, out, ws)
    err = np.abs(out.double().cpu().numpy().reshape(z, group, d) - ref)
    # half a unit of 1 (2^-24) for each sum that the first row goes through: of the rows of its wave
    # in pairs, then of sixteen waves in pairs (weights of 1 / live and their products are exact but
    # for the small parts' last bits); in one chain 13.5 of them are lost
    assert err.max() <= (np.log2(rows) + 4.1) * 2.0 ** -24, err.max() * 2.0 ** 24
