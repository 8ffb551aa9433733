"""bf16 attention of few workgroups or short walks (csrc/attend_short.hip): every row against the oracle, and the bits of the
kernels that take the same heads in a launch of many workgroups."""
import numpy as np
import pytest
import torch

import heatkv_inputs as hi
import paper_2605_14877_amd as hk
from tests.gpu_driver import device_generation
from tests.test_gpu_parity import _bf16_case, _dev

pytestmark = pytest.mark.gpu


def _outputs(d, H, tokens, qkv, batch, fused):
    shape = hk.Shape(1, H, d, tokens, batch, "bf16")
    w = hi.head_weights(61, 1, H, len(tokens))
    beta = hi.expected_beta_from_weights(w, tokens).astype(np.float32)
    c = hi.cumulative_tokens(tokens)
    plan = hk.heatkv_build_schedule(shape, beta, (H * c[-2] // 2 + H * c[0]) * 2 * d * 2, 1)
    rep = lambda x: x.repeat(batch, 1, 1, 1).contiguous()
    return device_generation(plan, 0, *(rep(x) for x in qkv), tokens, 1.0 / np.sqrt(d), fused=fused)


# Chunks of 16, blocks of 32 and tiles of 64 keys, query sets of 32: sizes at and next to their ends, as scale and in runs.
EDGES = [
    (128, 3, (1, 15, 16, 17, 31)),             # one round throughout, up to 32 + 49 keys
    (128, 5, (1, 2, 29, 33, 63)),              # one round of two query tiles, then two rounds
    (128, 3, (1, 16, 32, 48, 64, 65, 128)),    # whole chunks, blocks and tiles; three and more rounds
    (128, 4, (1, 49, 79, 129, 191, 257)),      # ragged ends of 1, 15, 49, 63 keys in the middle of a round
    (64, 3, (1, 15, 16, 17, 31)),
    (64, 5, (1, 2, 29, 33, 63)),               # the second query set is ragged
]


@pytest.mark.parametrize("d,H,tokens", EDGES)
def test_short_walks_against_the_oracle(d, H, tokens):
    _bf16_case(1, H, tuple((1, n) for n in tokens), 1, 2, 3, seed=62, fused=True, d=d)


def _rising(q, k):
    """Scores that raise the reference from tile to tile: logits climb by far more than 8 in the exponent of 2 along the walk."""
    n = k.shape[2]
    q[..., 0], k[..., 0] = 8.0, -torch.arange(n, device=k.device).to(k.dtype) * (400.0 / n)
    k[:, :, :n // 2, 0] += 300.0  # the run's scores lie above the current scale's


@pytest.mark.parametrize("rising", [False, True])
@pytest.mark.parametrize("d,H,tokens", EDGES)
def test_short_walks_have_the_bits_of_the_long_ones(d, H, tokens, rising):
    # 512 / H + 1 batch rows: more workgroups than the compute units take at once, so that all scales beyond a workgroup's
    # queries go to the other kernels (at d = 128 those of up to 32 queries and two tiles do not; next test).
    cfg = dict(L=1, H=H, d=d, dtype="bf16", batch=1, sides=[(1, n) for n in tokens])
    q, k, v = _dev(*hi.make_qkv(63, 0, cfg))
    if rising:
        _rising(q, k)
    few = _outputs(d, H, tokens, (q, k, v), 1, False)
    fused = _outputs(d, H, tokens, (q, k, v), 1, True)
    many = _outputs(d, H, tokens, (q, k, v), 512 // H + 1, False)
    for a, b, m in zip(few, fused, many):
        assert torch.isfinite(a).all() and torch.equal(a, b)
        assert torch.equal(m, a.expand_as(m))


# At most 256 workgroups of 128 queries that the short-walk kernel does not take: wavefronts of their own copy the tiles.  Query
# tiles of one row and of 127, idle wavefronts, walks of two tiles and more, and the cache update by workgroups of 512 lanes.
@pytest.mark.parametrize("rising", [False, True])
@pytest.mark.parametrize("d,H,few,tokens", [
    (128, 4, 16, (1, 63, 129, 200, 255)),   # 64, 128, 128, 128 workgroups
    (128, 4, 16, (2, 64, 65, 257, 383)),    # 192 workgroups
    (128, 4, 64, (1, 64, 66, 97, 128)),     # 256 workgroups: with the cache update by the other form, at four tiles by either
    (64, 3, 5, (1, 65, 130, 256, 300)),
    (64, 4, 64, (3, 64, 100, 33, 128)),     # 256 workgroups, likewise
])
def test_copying_wavefronts_change_no_bits(d, H, few, tokens, rising):
    cfg = dict(L=1, H=H, d=d, dtype="bf16", batch=1, sides=[(1, n) for n in tokens])
    q, k, v = _dev(*hi.make_qkv(65, 0, cfg))
    if rising:
        _rising(q, k)
    alone = _outputs(d, H, tokens, (q, k, v), few, False)
    fused = _outputs(d, H, tokens, (q, k, v), few, True)
    many = _outputs(d, H, tokens, (q, k, v), 256 // H + 1, False)
    for a, b, m in zip(alone, fused, many):
        assert torch.isfinite(a).all() and torch.equal(a, b)
        assert torch.equal(m, a[:1].expand_as(m)) and torch.equal(a, a[:1].expand_as(a))


@pytest.mark.parametrize("d,batch,tokens", [(128, 16, (1, 64, 130, 200)), (64, 4, (2, 65, 130, 300))])
def test_copying_wavefronts_against_the_oracle(d, batch, tokens):
    _bf16_case(1, 4, tuple((1, n) for n in tokens), 1, 2, batch, seed=66, fused=True, d=d)


# 256 workgroups of 400 queries.  The first two have walks of 8 and 14 tiles and updates of 256 and 512 workgroups behind them,
# which would wait for units: one stream, the bits of a launch of more workgroups, with the update in the launch or not.  The last
# scale, without an update and of 21 tiles, has two streams, whose last bits are others.
def test_updates_of_many_workgroups_keep_one_stream_at_head_dimension_64():
    d, H, tokens = 64, 4, [1, 400, 400, 401]
    K = len(tokens)
    cfg = dict(L=1, H=H, d=d, dtype="bf16", batch=1, sides=[(1, n) for n in tokens])
    q, k, v = _dev(*hi.make_qkv(67, 0, cfg))
    present = np.zeros((K, 1, H, K), np.uint8)
    for kk in range(1, K):
        present[kk, 0, :, :kk] = 1
    outs = []
    for rows, fused in ((16, False), (16, True), (17, False)):
        plan = hk.heatkv_load_schedule(hk.Shape(1, H, d, tokens, rows, "bf16"), present)
        qkv = (x.repeat(rows, 1, 1, 1).contiguous() for x in (q, k, v))
        outs.append(device_generation(plan, 0, *qkv, tokens, 1.0 / np.sqrt(d), fused=fused))
    for kk, (a, b, m) in enumerate(zip(*outs)):
        assert torch.equal(a, b) and torch.equal(a, a[:1].expand_as(a)) and torch.equal(m, m[:1].expand_as(m))
        assert torch.equal(m[0], a[0]) == (kk < 3), kk


# One round of up to 32 queries, d = 128, goes to the short-walk kernel whatever the number of workgroups, but not in a launch
# with a longer walk: the same heads next to one that keeps the 100 rows of the first scale, in more workgroups than there
# are compute units.
@pytest.mark.parametrize("rising", [False, True])
@pytest.mark.parametrize("tokens", [(100, 1, 15, 16, 17, 31), (100, 30, 32, 2, 1), (100, 31, 33, 32)])
def test_one_round_walks_have_the_bits_of_the_long_ones(tokens, rising):
    H, K, d, batch, tokens = 5, len(tokens), 128, 47, list(tokens)
    cfg = dict(L=1, H=H + 1, d=d, dtype="bf16", batch=1, sides=[(1, n) for n in tokens])
    q, k, v = _dev(*hi.make_qkv(64, 0, cfg))
    if rising:
        _rising(q, k)
    outs = []
    for heads, rows in ((H, 1), (H + 1, batch)):
        present = np.zeros((K, 1, heads, K), np.uint8)
        for kk in range(1, K):
            present[kk, 0, :, 1:kk] = 1
            present[kk, 0, H:, 0] = 1
        plan = hk.heatkv_load_schedule(hk.Shape(1, heads, d, tokens, rows, "bf16"), present)
        qkv = (x[:, :heads].repeat(rows, 1, 1, 1).contiguous() for x in (q, k, v))
        outs.append(device_generation(plan, 0, *qkv, tokens, 1.0 / np.sqrt(d)))
    tiles = lambda *rows: sum(-(-n // 64) for n in rows)
    for kk in range(1, K):
        run = sum(tokens[1:kk])
        assert tiles(tokens[kk], run) <= 2 < tiles(tokens[kk], 100 + run) and (H + 1) * batch > 256
        assert torch.isfinite(outs[0][kk]).all()
        assert torch.equal(outs[1][kk][:, :H], outs[0][kk].expand(batch, -1, -1, -1)), kk


# The same in both kernels where operands are not finite, masked to the lowest value or scaled to one-hot rows.
@pytest.mark.parametrize("kind", ["keys of -inf", "keys of the lowest value", "all keys of -inf", "an infinite key", "large keys",
                                  "an infinite value", "a NaN value", "a NaN query", "large scale"])
@pytest.mark.parametrize("d", [64, 128])
def test_special_operands_as_in_the_long_walks(d, kind):
    H, batch, tokens = 5, 47, [100, 31, 33, 32, 70]
    K, n = len(tokens), sum(tokens)
    sm = 1e30 if kind == "large scale" else 1.0 / np.sqrt(d)
    g = torch.Generator(device="cuda").manual_seed(66)
    q, k, v = (torch.randn(1, H + 1, n, d, generator=g, device="cuda").to(torch.bfloat16) for _ in range(3))
    if "keys of" in kind:
        q[..., 0] = 1.0
        k[:, :, ::1 if kind.startswith("all") else 3, 0] = -float("inf") if "inf" in kind else torch.finfo(k.dtype).min
    elif kind == "an infinite key":
        k[:, :, 120::40, 5] = float("inf")
    elif kind == "large keys":
        k[:, :, 2::7] *= 2.0 ** 100
    elif "value" in kind:
        v[:, :, 110::31, 3] = float("inf") if "inf" in kind else float("nan")
    elif kind == "a NaN query":
        q[:, :, 3::17, 7] = float("nan")
    outs = []
    for heads, rows in ((H, 1), (H + 1, batch)):
        present = np.zeros((K, 1, heads, K), np.uint8)
        for kk in range(1, K):
            present[kk, 0, :, 1:kk] = 1
            present[kk, 0, H:, 0] = 1
        plan = hk.heatkv_load_schedule(hk.Shape(1, heads, d, tokens, rows, "bf16"), present)
        qkv = (x[:, :heads].repeat(rows, 1, 1, 1).contiguous() for x in (q, k, v))
        outs.append(device_generation(plan, 0, *qkv, tokens, sm))
    for a, m in zip(*outs):
        torch.testing.assert_close(m[:, :H], a.expand(batch, -1, -1, -1), rtol=0, atol=0, equal_nan=True)


# Two key streams at d = 64 (385 and more tokens, 12 tiles and more), whose merge brings two references together: operands that
# raise them far apart, tiles of one stream masked throughout, and the special ones above, against 64 bits.  Probabilities and
# outputs are rounded to bf16, 2^-9 each, the row sum is taken over the rounded ones, and scores of up to 750 in fp32 move
# a probability by 1e-4.
@pytest.mark.parametrize("kind", ["ordinary", "rising", "falling", "one stream of -inf", "one stream of the lowest value",
                                  "other stream of -inf", "keys of -inf", "all keys of -inf", "an infinite key", "large keys",
                                  "an infinite value", "a NaN value", "a NaN query"])
def test_two_key_streams_of_head_dimension_64_on_special_operands(kind):
    d, H, tokens = 64, 3, [100, 300, 385, 450]
    K, n, sm = len(tokens), sum(tokens), 1.0 / np.sqrt(64)
    g = torch.Generator(device="cuda").manual_seed(68)
    q, k, v = (torch.randn(1, H, n, d, generator=g, device="cuda").to(torch.bfloat16) for _ in range(3))
    if kind in ("rising", "falling"):
        _rising(q, k)
        if kind == "falling":
            k[..., 0] = k[..., 0].flip(2)
    elif "stream" in kind:  # of the last scale: current tiles 0..7, then those of the run
        q[..., 0] = 1.0
        first = 1 if kind.startswith("one") else 0
        for tile in range(first, 8 + 13, 2):
            lo, end = (785 + 64 * tile, n) if tile < 8 else (64 * (tile - 8), 785)
            k[:, :, lo:min(lo + 64, end), 0] = -float("inf") if "inf" in kind else torch.finfo(k.dtype).min
    elif "keys of" in kind:
        q[..., 0] = 1.0
        k[:, :, ::1 if kind.startswith("all") else 3, 0] = -float("inf")
    elif kind == "an infinite key":
        k[:, :, 120::40, 5] = float("inf")
    elif kind == "large keys":
        k[:, :, 2::7] *= 2.0 ** 7
    elif "value" in kind:
        v[:, :, 110::31, 3] = float("inf") if "inf" in kind else float("nan")
    elif kind == "a NaN query":
        q[:, :, 3::17, 7] = float("nan")
    plan = hk.heatkv_load_schedule(hk.Shape(1, H, d, tokens, 1, "bf16"),
                                   np.tril(np.ones((K, K), np.uint8), -1)[:, None, None].repeat(H, 2))
    outs = device_generation(plan, 0, q, k, v, tokens, sm)
    for kk in (2, 3):
        end = sum(tokens[:kk + 1])
        qs = q[0, :, end - tokens[kk]:end].double().cpu()
        ks, vs = k[0, :, :end].double().cpu(), v[0, :, :end].double().cpu()
        p = torch.softmax(torch.matmul(qs, ks.transpose(1, 2)) * sm, -1)
        want, got = torch.matmul(p, vs), outs[kk][0].double().cpu()
        finite = torch.isfinite(want)
        assert torch.equal(torch.isfinite(got), finite) and torch.equal(torch.isnan(got), torch.isnan(want)), kind
        size = torch.matmul(p, vs.abs())
        bound = (2.0 ** -8 + 2e-4) * size + 2.0 ** -9 * want.abs() + 1e-30
        assert ((got - want).abs() <= bound)[finite].all(), (kind, kk, ((got - want).abs() / bound)[finite].max())


# Tensors need not start on a 16-byte boundary: views of a longer one at 4, 8 and 12 bytes, and queries at 2 (another kernel).
@pytest.mark.parametrize("d,dtype,tokens,batch", [(128, "bf16", [1, 17, 31, 70, 129], 2), (64, "bf16", [1, 17, 31], 2),
                                                  (128, "f32", [1, 33, 147], 32), (64, "f32", [1, 33, 147], 32)])
def test_operands_off_the_16_byte_grid(d, dtype, tokens, batch):
    kind = torch.bfloat16 if dtype == "bf16" else torch.float32
    K, c, sm = len(tokens), hi.cumulative_tokens(tokens), 1.0 / np.sqrt(d)
    plan = hk.heatkv_load_schedule(hk.Shape(1, 2, d, tokens, batch, dtype),
                                   np.tril(np.ones((K, K), np.uint8), -1)[:, None, None].repeat(2, 2))
    g = torch.Generator(device="cuda").manual_seed(65)
    q, k, v = (torch.randn(batch, 2, c[-1], d, generator=g, device="cuda").to(kind) for _ in range(3))

    def moved(x, n_bytes):
        skip = n_bytes // x.element_size()
        y = torch.empty(x.numel() + skip, dtype=x.dtype, device="cuda")[skip:].view(x.shape)
        return y.copy_(x)

    def outputs(q_at, at):
        ka, va = (moved(torch.zeros(plan.arena_bytes, dtype=torch.uint8, device="cuda"), at) for _ in range(2))
        outs = []
        for i in range(K):
            cut = slice(c[i] - tokens[i], c[i])
            out = moved(torch.zeros(batch, 2, tokens[i], d, dtype=kind, device="cuda"), at)
            hk.heatkv_attend_append_scale(plan, 0, i, moved(q[:, :, cut], q_at), moved(k[:, :, cut], at),
                                          moved(v[:, :, cut], at), ka, va, sm, out)
            outs.append(out)
        return outs

    want = outputs(0, 0)
    for q_at, at in [(4, 4), (8, 8), (12, 12)] + ([(2, 0)] if dtype == "bf16" else []):
        for a, b in zip(outputs(q_at, at), want):
            assert torch.equal(a, b), (q_at, at)
