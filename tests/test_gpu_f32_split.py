"""fp32 attention and calibration on three bf16 parts (csrc/f32_split.h): every row against the oracle at the edges of its
tiles, and operands outside the range of the parts against the kernels on the fp32 instructions, which the same heads take
in a launch of few workgroups."""
import numpy as np
import pytest
import torch

import heatkv_inputs as hi
import paper_2605_14877_amd as hk
from oracle import heatkv_oracle as orc
from tests import harness
from tests.gpu_driver import device_generation
from tests.test_gpu_parity import TOL, _check_all, _dev

pytestmark = pytest.mark.gpu


# From the third scale on more than 256 workgroups of 16 queries, at most 256 of 32; the last one takes more than one turn of
# either.  Blocks of 32 keys and queries: one row over, whole, one short; runs that end next to and at a block's end.
@pytest.mark.parametrize("d,H,batch,tokens", [
    (128, 6, 5, (1, 31, 129, 160, 191)),
    (64, 5, 6, (2, 30, 143, 224)),
    (128, 5, 13, (1, 64, 257)),
])
def test_attention_at_the_edges(d, H, batch, tokens):
    t0, K, sm = list(tokens), len(tokens), 1.0 / np.sqrt(d)
    cfg = dict(L=1, H=H, d=d, dtype="f32", batch=batch, sides=[(1, n) for n in t0])
    c = hi.cumulative_tokens(t0)
    B = H * c[-2] * 2 // 3 + H * c[0]
    w = hi.head_weights(71, 1, H, K)
    beta = hi.expected_beta_from_weights(w, t0).astype(np.float32)
    plan = hk.heatkv_build_schedule(hk.Shape(1, H, d, t0, batch, "f32"), beta, B * 2 * d * 4, 1)
    q, k, v = hi.make_qkv(71, 0, cfg, w=w)
    outs = device_generation(plan, 0, *_dev(q, k, v), t0, sm, fused=True)
    for a, b in zip(outs, device_generation(plan, 0, *_dev(q, k, v), t0, sm)):
        assert torch.equal(a, b)
    _check_all(outs, q, k, v, t0, harness.oracle_schedule(beta, 1, H, t0, 1, B)["present"], 0, sm, TOL["f32"])


# Calibration takes it from 1920 workgroups of 16 queries on (d = 64: 8192).
@pytest.mark.parametrize("d,H,batch,tokens", [(128, 6, 5, (1, 31, 129, 961)), (128, 6, 23, (2, 30, 143, 224)),
                                              (64, 8, 31, (2, 30, 143, 544))])
def test_calibration_at_the_edges(d, H, batch, tokens):
    t0, c, K, sm = list(tokens), hi.cumulative_tokens(tokens), len(tokens), 1.0 / np.sqrt(d)
    cfg = dict(L=1, H=H, d=d, dtype="f32", batch=batch, sides=[(1, n) for n in t0])
    q, k, _ = hi.make_qkv(72, 0, cfg, w=hi.head_weights(72, 1, H, K))
    shape = hk.Shape(1, H, d, t0, batch, "f32")
    mass = torch.empty(batch, H, K, device="cuda")
    ws = torch.empty(hk.binding.calibrate_workspace_bytes(shape, K - 1), dtype=torch.uint8, device="cuda")
    hk.heatkv_calibrate(shape, 0, K - 1, *_dev(q[:, :, c[-1] - t0[-1]:].contiguous(), k), sm, mass, ws)
    got = mass.cpu().double().numpy()
    for b in range(batch):
        for h in range(H):
            want = orc.beta_row(q[b, h].double().numpy(), k[b, h].double().numpy(), orc.one_based(t0), K, sm)
            assert np.abs(got[b, h] - want[1:]).max() <= 1e-5, (b, h)  # as the kernel on the fp32 instructions


KINDS = ["plain", "keys of -inf", "keys of the lowest value", "an infinite key", "large keys", "large queries, small keys",
         "large values", "tiny values", "an infinite value", "a NaN value", "a NaN query"]


def _operands(kind, d, n):
    g = torch.Generator().manual_seed(73)
    q, k, v = (torch.randn(1, 1, n, d, generator=g) for _ in range(3))
    if kind.startswith("keys of"):
        q[..., 0], k[:, :, 3::5, 0] = 1.0, -float("inf") if "inf" in kind else torch.finfo(torch.float32).min
    elif kind == "an infinite key":
        k[:, :, n - 7, 5] = float("inf")
    elif kind == "large keys":
        k[:, :, 2::7] *= 2.0 ** 70
    elif kind == "large queries, small keys":
        q, k = q * 2.0 ** 65, k * 2.0 ** -65
    elif kind == "large values":
        v = v * 2.0 ** 110
    elif kind == "tiny values":
        v = v * 2.0 ** -112
    elif kind == "an infinite value":
        v[:, :, n - 9, 3] = float("inf")
    elif kind == "a NaN value":
        v[:, :, n - 9, 3] = float("nan")
    elif kind == "a NaN query":
        q[:, :, n - 3, 7] = float("nan")
    return q, k, v


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("d", [64, 128])
def test_attention_beyond_the_range_of_the_parts(d, kind):
    tokens, many = [1, 33, 147], 32
    q, k, v = _dev(*_operands(kind, d, sum(tokens)))
    outs = []
    for batch in (1, many):
        plan = hk.heatkv_build_schedule(hk.Shape(1, 1, d, tokens, batch, "f32"), harness.random_beta(5, 1, 1, 3),
                                        34 * 2 * d * 4, 1)
        rep = lambda x: x.repeat(batch, 1, 1, 1).contiguous()
        outs.append(device_generation(plan, 0, rep(q), rep(k), rep(v), tokens, 1.0 / np.sqrt(d))[-1])
    a, b = outs[0].double(), outs[1].double()
    assert torch.equal(b, b[:1].expand_as(b)) or torch.isnan(b).any()
    # Two fp32 evaluations: scores of up to 2^3 in the exponent with errors of 1e-6, and sums of 181 products.  One-hot
    # softmax rows (large keys) are decided by scores far apart.
    scale = v[torch.isfinite(v)].abs().max().item()
    torch.testing.assert_close(b[:1], a, rtol=1e-5, atol=1e-5 * scale, equal_nan=True)


def _exact(q, k, v, idx, rows, sm):
    """Attention of the last `rows` queries over the keys idx, in 64 bits."""
    q, k, v = (x[0, 0].double().cpu() for x in (q, k, v))
    return torch.softmax(q[-rows:] @ k[idx].T * sm, -1) @ v[idx]


# Errors against 64 bits.  The fp32 instructions have up to 3.3e-7 (norm) here, the parts 1.9e-7, and without one of the
# six products, in the scores or in P V, 1.7e-6 or more.  Bound: twice that of the fp32 instructions.  Keys of 2^-117 whose
# softmax scale makes ordinary scores of them have an inexact third part (4e-6): such a scale takes the fp32 instructions.
SCALED = [("plain", 0), ("tiny keys, large softmax scale", 117)]


@pytest.mark.parametrize("kind,up", SCALED)
@pytest.mark.parametrize("d", [64, 128])
def test_attention_error_against_64_bits(d, kind, up):
    tokens, many = [1, 33, 147], 32
    g = torch.Generator().manual_seed(75)
    q, k, v = (torch.randn(many, 1, sum(tokens), d, generator=g) for _ in range(3))
    sm = 2.0 ** up / np.sqrt(d)
    k *= 2.0 ** -up
    plan = hk.heatkv_build_schedule(hk.Shape(1, 1, d, tokens, many, "f32"), harness.random_beta(5, 1, 1, 3), 34 * 2 * d * 4, 1)
    idx = list(plan.retained(2, 0, 0)) + list(range(34, 181))
    out = device_generation(plan, 0, *_dev(q, k, v), tokens, sm)[-1]
    for b in (0, 9, many - 1):
        want = _exact(q[b:], k[b:], v[b:], idx, tokens[-1], sm)
        assert (out[b, 0].double().cpu() - want).norm() <= 6.6e-7 * want.norm()


# Masses of blocks of one key, the query rows of a head all the same, so that no error averages out: rms of the relative error.
# The fp32 instructions have 2.4e-7, the parts 2.2e-7, and without one of the products 2e-6.  Bound: twice the former.
@pytest.mark.parametrize("kind,up", SCALED)
@pytest.mark.parametrize("d,rows,many", [(128, 197, 152), (64, 513, 256)])
def test_calibration_error_against_64_bits(d, rows, many, kind, up):
    ones = 12  # with more scales the block sums do not fit next to the stages of the parts (d = 128)
    tokens = [1] * ones + [rows]
    g = torch.Generator().manual_seed(76)
    q = torch.randn(many, 1, 1, d, generator=g).expand(many, 1, rows, d).contiguous()
    k = torch.randn(many, 1, sum(tokens), d, generator=g) * 2.0 ** -up
    sm = 2.0 ** up / np.sqrt(d)
    shape = hk.Shape(1, 1, d, tokens, many, "f32")
    mass = torch.empty(many, 1, ones + 1, device="cuda")
    ws = torch.empty(hk.binding.calibrate_workspace_bytes(shape, ones), dtype=torch.uint8, device="cuda")
    hk.heatkv_calibrate(shape, 0, ones, *_dev(q, k), sm, mass, ws)
    want = torch.softmax((q[:, 0, :1].double() @ k[:, 0].double().transpose(1, 2)) * sm, -1)[:, 0, :ones]
    error = mass[:, 0, :ones].double().cpu() / want - 1
    assert error.square().mean().sqrt() <= 5e-7


# What decides an output need not be large: a column of tiny values next to ordinary ones, values that are zero but where the
# probabilities are tiny.  The third bf16 part of a number below 2^-110 is inexact, in the worst column by 4e-6 (values of
# 2^-117) and 2e-4 (probabilities of 2^-117, taken 2^-8 times).  Bounds: sums of fp32 products that are subnormal, each off
# by 2^-150 where the result is about 2^-125: 6e-7, three times that; scores of 113 in the exponent of 2, off by 2^-24 of that
# and as much again in the sum of the products: 1e-5, twice that.
@pytest.mark.parametrize("kind,bound", [("a column of tiny values", 2e-6), ("values under tiny probabilities", 2e-5)])
@pytest.mark.parametrize("d", [64, 128])
def test_attention_decided_by_tiny_numbers(d, kind, bound):
    tokens, many, column, sm = [1, 33, 147], 32, 3, 1.0 / np.sqrt(d)
    q, k, v = _operands("plain", d, sum(tokens))
    if kind == "a column of tiny values":
        v[..., column] *= 2.0 ** -117
    else:
        q[..., 0], k[..., 0] = 8.0, 0.0
        weak = torch.arange(sum(tokens)) % 5 == 3
        k[:, :, weak, 0] = -78.0 * np.sqrt(d) / 8.0
        v[:, :, :, column] = torch.where(weak, v[..., column] * 2.0 ** 40, 0.0)
    plan = hk.heatkv_build_schedule(hk.Shape(1, 1, d, tokens, many, "f32"), harness.random_beta(5, 1, 1, 3), 34 * 2 * d * 4, 1)
    idx = list(plan.retained(2, 0, 0)) + list(range(34, 181))
    out = device_generation(plan, 0, *_dev(*(x.repeat(many, 1, 1, 1).contiguous() for x in (q, k, v))), tokens, sm)[-1]
    want, got = _exact(q, k, v, idx, tokens[-1], sm), out[many - 1, 0].double().cpu()
    error = (got - want).norm(dim=0) / want.norm(dim=0)
    assert error[column] <= bound
    assert error.max() <= (bound if kind == "a column of tiny values" else 2e-5)


@pytest.mark.parametrize("kind", [x for x in KINDS if "value" not in x or "lowest" in x])
@pytest.mark.parametrize("d", [64, 128])
def test_calibration_beyond_the_range_of_the_parts(d, kind):
    tokens, many = ([1, 33, 197], 152) if d == 128 else ([1, 33, 513], 256)
    q, k, _ = _dev(*_operands(kind, d, sum(tokens)))
    got = []
    for batch in (1, many):
        shape = hk.Shape(1, 1, d, tokens, batch, "f32")
        mass = torch.empty(batch, 1, 3, device="cuda")
        ws = torch.empty(hk.binding.calibrate_workspace_bytes(shape, 2), dtype=torch.uint8, device="cuda")
        hk.heatkv_calibrate(shape, 0, 2, q[:, :, 34:].repeat(batch, 1, 1, 1).contiguous(), k.repeat(batch, 1, 1, 1).contiguous(),
                            1.0 / np.sqrt(d), mass, ws)
        got.append(mass.double())
    torch.testing.assert_close(got[1], got[0].expand_as(got[1]), rtol=0, atol=1e-6, equal_nan=True)


# Scales of enough 16-query workgroups among shorter ones: a launch over all of them has the bits of one each.
@pytest.mark.parametrize("d,tokens", [(128, (1, 250, 40, 190, 230)), (64, (1030, 9, 150, 260))])
def test_calibration_of_several_scales_has_the_bits_of_one_each(d, tokens):
    t0, c, K, H, batch, sm = list(tokens), hi.cumulative_tokens(tokens), len(tokens), 8, 16, 1.0 / np.sqrt(d)
    g = torch.Generator().manual_seed(74)
    q, k = _dev(*(torch.randn(batch, H, c[-1], d, generator=g) for _ in range(2)))
    shape = hk.Shape(1, H, d, t0, batch, "f32")
    qs = [q[:, :, c[i] - t0[i]:c[i]].contiguous() for i in range(K)]
    ks = [k[:, :, :c[i]].contiguous() for i in range(K)]
    one, several = (torch.zeros(1, H, K, K, device="cuda") for _ in range(2))
    for i in range(K):
        ws = torch.empty(hk.binding.calibrate_workspace_bytes(shape, i), dtype=torch.uint8, device="cuda")
        hk.heatkv_calibrate_accumulate(shape, 0, i, qs[i], ks[i], sm, 0.25, one, None, ws)
    for scales in (list(range(K)), [K - 1, 1]):
        several.zero_()
        ws = torch.empty(hk.binding.calibrate_scales_workspace_bytes(shape, scales), dtype=torch.uint8, device="cuda")
        hk.heatkv_calibrate_scales_accumulate(shape, 0, scales, [qs[i] for i in scales], [ks[i] for i in scales], sm, 0.25,
                                              several, None, ws)
        assert torch.equal(several[:, :, scales], one[:, :, scales])
