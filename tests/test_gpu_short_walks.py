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


@pytest.mark.parametrize("rising", [False, True])
@pytest.mark.parametrize("d,H,tokens", EDGES)
def test_short_walks_have_the_bits_of_the_long_ones(d, H, tokens, rising):
    # 512 / H + 1 batch rows: more workgroups than the compute units take at once, so that all scales beyond a workgroup's
    # queries go to the other kernels.  Rising scores: the reference is raised from tile to tile (logits climb by far more
    # than 8 in the exponent of 2 along the walk).
    cfg = dict(L=1, H=H, d=d, dtype="bf16", batch=1, sides=[(1, n) for n in tokens])
    q, k, v = _dev(*hi.make_qkv(63, 0, cfg))
    if rising:
        n = k.shape[2]
        q[..., 0], k[..., 0] = 8.0, -torch.arange(n, device="cuda").to(k.dtype) * (400.0 / n)
        k[:, :, :n // 2, 0] += 300.0  # the run's scores lie above the current scale's
    few = _outputs(d, H, tokens, (q, k, v), 1, False)
    fused = _outputs(d, H, tokens, (q, k, v), 1, True)
    many = _outputs(d, H, tokens, (q, k, v), 512 // H + 1, False)
    for a, b, m in zip(few, fused, many):
        assert torch.isfinite(a).all() and torch.equal(a, b)
        assert torch.equal(m, a.expand_as(m))
