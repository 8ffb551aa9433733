"""The reductions behind the calibration kernels against the sums they stand for, bit for bit: the partial sums that a call
leaves in its workspace added in tile order, divided by the number of query rows, and the batch rows added in order."""
import numpy as np
import pytest
import torch

import paper_2605_14877_amd as hk

pytestmark = pytest.mark.gpu


# Query tiles (of 16 rows, bf16: 128): one, one group of sixteen less one, whole, one over, two over; batch rows: one turn of
# eight less seven, whole, one over, two turns and one; 5 * 7 entries of beta are a block of 32 and three.
@pytest.mark.parametrize("with_mass", [True, False])
@pytest.mark.parametrize("dtype,t,batch", [
    ("f32", 16, 8), ("f32", 239, 1), ("f32", 256, 9), ("f32", 257, 2), ("f32", 520, 17), ("bf16", 128, 9), ("bf16", 2100, 3),
])
def test_partial_sums_in_order(dtype, t, batch, with_mass):
    H, K, d, k1, L = 5, 7, 64, 4, 2
    tokens = [1, 2, 5, 9, t, 11, 13]
    tile = 16 if dtype == "f32" else 128
    tiles = -(-t // tile)
    torch.manual_seed(91)
    kind = torch.float32 if dtype == "f32" else torch.bfloat16
    q = torch.randn(batch, H, t, d).to("cuda", kind)
    k = torch.randn(batch, H, sum(tokens[:k1 + 1]), d).to("cuda", kind)
    shape = hk.Shape(L, H, d, tokens, batch, dtype)
    ws = torch.empty(hk.binding.calibrate_workspace_bytes(shape, k1), dtype=torch.uint8, device="cuda")
    mass = torch.full((batch, H, K), -1.0, device="cuda")
    beta = torch.rand(L, H, K, K).cuda()
    before = beta.cpu().numpy()
    hk.heatkv_calibrate_accumulate(shape, 1, k1, q, k, d ** -0.5, 0.25, beta, mass if with_mass else None, ws)
    parts = ws.cpu().numpy().view(np.float32)[:batch * H * tiles * K].reshape(batch, H, tiles, K)
    want = np.zeros((batch, H, K), np.float32)
    for i in range(tiles):
        want[..., :k1 + 1] += parts[:, :, i, :k1 + 1]
    want /= np.float32(t)
    if with_mass:
        assert np.array_equal(mass.cpu().numpy(), want)
    total = np.zeros((H, K), np.float32)
    for b in range(batch):
        total += want[b]
    after = before.copy()
    after[1, :, k1] += np.float32(0.25) * total  # a power of two: one rounding, with or without a fused multiply-add
    assert np.array_equal(beta.cpu().numpy(), after)
    hk.heatkv_calibrate(shape, 1, k1, q, k, d ** -0.5, mass, ws)
    assert np.array_equal(mass.cpu().numpy(), want)


# A call for one scale of at most 16 rows with one or two batch rows reduces in its own launch; a call for several scales has
# the second launch: same bits, in all of mass and beta, with a weight that rounds.
@pytest.mark.parametrize("with_mass", [True, False])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("H,batch,tokens", [
    (5, 1, (1, 15, 16, 17)), (5, 2, (1, 15, 16, 17)), (5, 3, (2, 16)), (9, 2, (3, 16) + (1, 4) * 14 + (16,)),
])
def test_scales_of_one_query_tile_have_the_bits_of_a_call_for_all_scales(H, batch, tokens, d, with_mass):
    K, L = len(tokens), 2
    torch.manual_seed(92)
    q = [torch.randn(batch, H, t, d).cuda() for t in tokens]
    k = torch.randn(batch, H, sum(tokens), d)
    k_all = [k[:, :, :sum(tokens[:i + 1])].contiguous().cuda() for i in range(K)]
    shape = hk.Shape(L, H, d, tokens, batch, "f32")
    start = torch.rand(L, H, K, K).cuda()
    one, each = start.clone(), start.clone()
    masses = [[torch.full((batch, H, K), -1.0, device="cuda") if with_mass else None for _ in tokens] for _ in range(2)]
    scales = list(range(K))
    ws = torch.empty(hk.binding.calibrate_scales_workspace_bytes(shape, scales), dtype=torch.uint8, device="cuda")
    hk.heatkv_calibrate_scales_accumulate(shape, 1, scales, q, k_all, d ** -0.5, 0.3, one, masses[0] if with_mass else None, ws)
    for i in scales:
        hk.heatkv_calibrate_accumulate(shape, 1, i, q[i], k_all[i], d ** -0.5, 0.3, each, masses[1][i], ws)
    assert torch.equal(one, each) and not torch.equal(one[1], start[1]) and torch.equal(one[0], start[0])
    for a, b in zip(*masses):
        assert a is b is None or torch.equal(a, b)


# Two batch rows of one query tile share a workgroup while the walk over the keys is short, or where there are units for half of
# the workgroups only; one row has its own at any length.  The form with a second launch leaves its partial sums in the workspace.
@pytest.mark.parametrize("d,H,batch,tokens,one_launch", [
    (64, 3, 2, (304, 16), True), (64, 3, 2, (305, 16), False),   # 20 and 21 key tiles
    (128, 3, 2, (112, 16), True), (128, 3, 2, (113, 16), False),  # 8 and 9
    (128, 3, 2, (1,) * 7 + (16,), True), (128, 3, 2, (1,) * 8 + (16,), False),
    (128, 128, 2, (500, 16), False), (128, 129, 2, (500, 16), True), (128, 256, 2, (500, 16), True), (64, 257, 2, (500, 16), False),
    (128, 3, 1, (900, 16), True), (64, 3, 1, (900, 16), True), (64, 3, 3, (1, 16), False),
    (64, 129, 2, (1,) * 30 + (16,), True), (128, 129, 2, (1,) * 30 + (16,), True),  # 31 scales: the most LDS, 64 and 98 KB
])
def test_two_batch_rows_share_a_workgroup_for_short_walks(d, H, batch, tokens, one_launch):
    K = len(tokens)
    torch.manual_seed(93)
    q = torch.randn(batch, H, tokens[-1], d, device="cuda")
    k = torch.randn(batch, H, sum(tokens), d, device="cuda")
    shape = hk.Shape(1, H, d, tokens, batch, "f32")
    ws = torch.full((hk.binding.calibrate_scales_workspace_bytes(shape, [K - 1]),), 255, dtype=torch.uint8, device="cuda")
    one, each = torch.zeros(1, H, K, K, device="cuda"), torch.zeros(1, H, K, K, device="cuda")
    hk.heatkv_calibrate_accumulate(shape, 0, K - 1, q, k, d ** -0.5, 0.5, one, None, ws)
    assert bool((ws == 255).all()) == one_launch
    mass = torch.empty(batch, H, K, device="cuda")
    hk.heatkv_calibrate(shape, 0, K - 1, q, k, d ** -0.5, mass, ws)
    each[0, :, K - 1] = 0.5 * sum(mass[b] for b in range(batch))
    assert torch.equal(one, each)
    assert torch.allclose(mass.sum(-1), torch.ones(batch, H, device="cuda"), atol=1e-5)
