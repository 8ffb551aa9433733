"""The native call path (csrc/call_path.cpp): that it makes the calls it is there for, declines the others, and takes the
stream that the caller means."""
import threading

import numpy as np
import pytest
import torch

import heatkv_inputs as hi
import paper_2605_14877_amd as hk
from paper_2605_14877_amd import binding
from tests.gpu_driver import device_generation

pytestmark = pytest.mark.gpu

T0, H, D, NB = [1, 4, 9, 30], 3, 64, 2
K, SM = len(T0), 0.125
C = hi.cumulative_tokens(T0)


def _problem(dtype, seed=5):
    cfg = dict(L=1, H=H, d=D, dtype=dtype, batch=NB, sides=[(1, n) for n in T0])
    w = hi.head_weights(seed, 1, H, K)
    q, k, v = (x.cuda() for x in hi.make_qkv(seed, 0, cfg, w=w))
    plan = hk.heatkv_build_schedule(hk.Shape(1, H, D, T0, NB, dtype), hi.expected_beta_from_weights(w, T0).astype(np.float32),
                                    H * C[-2] * 2 * D * hi.elem_bytes(dtype), 1)
    plan.upload()
    return plan, q, k, v


def _scale(x, kk):
    return x[:, :, C[kk] - T0[kk]:C[kk]].contiguous()


def _arenas(plan):
    return [torch.zeros(plan.arena_bytes, dtype=torch.uint8, device="cuda") for _ in range(2)]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_native_path_makes_plain_calls_and_declines_malformed_ones(dtype):
    plan, q, k, v = _problem(dtype)
    call, shape, kk = binding._call, plan.shape, 2
    (ka, va), other = _arenas(plan), torch.float32 if dtype == "bf16" else torch.bfloat16
    qk, kc, vc = (_scale(x, kk) for x in (q, k, v))
    out, ws = torch.zeros_like(qk), torch.empty(1 << 20, dtype=torch.uint8, device="cuda")
    args = [plan.call_info, 0, 0, kk, qk, kc, vc, ka, va, SM, out, ws, None]
    for which in (0, 1, 2):
        good = args[:1] + [which] + args[2:]
        assert call.scale_call(*good) == 0
        bad = {2: [1, -1, "0"], 3: [K, -1], 5: [kc[:, :, 1:].contiguous(), kc.to(other), kc.transpose(0, 1), kc.cpu(), kc.tolist()],
               7: [ka[:-1]], 8: [va[:-1], va[::2]], 12: ["stream", 1.5]}
        if which:
            bad.update({4: [qk[:1], qk.to(other)], 9: ["0.1"], 10: [out[..., :-1].contiguous()], 11: [ws[::2]]})
        for i, values in bad.items():
            for x in values:
                assert call.scale_call(*good[:i], x, *good[i + 1:]) is None, (which, i, x)
        assert call.scale_call(*good[:-1]) is None

    k_all = k[:, :, :C[kk]].contiguous()
    beta, mass = torch.zeros(1, H, K, K, device="cuda"), torch.zeros(NB, H, K, device="cuda")
    for which in (0, 1, 2):
        good = [shape.address, which, 0, kk, qk, k_all, SM, 0.5, beta if which == 2 else None, mass, ws, None]
        assert call.calibrate_call(*good) == 0
        for i, x in ((0, 0), (3, K), (4, qk[:1]), (5, kc), (5, k_all.to(other)), (6, "0.1"), (9, mass.double()),
                     (10, ws.cpu()), (11, "stream")):
            assert call.calibrate_call(*good[:i], x, *good[i + 1:]) is None, (which, i)
    assert call.calibrate_call(shape.address, 2, 0, kk, qk, k_all, SM, 0.5, beta[..., 1:], mass, ws, None) is None

    good = [shape.address, 0, [kk, 0], [qk, _scale(q, 0)], [k_all, k[:, :, :1].contiguous()], SM, 0.5, beta, [mass, None], ws,
            None]
    assert call.calibrate_scales_call(*good) == 0
    for i, x in ((2, [kk]), (2, [kk, K]), (2, (kk, 0)), (3, [qk, qk]), (4, [k_all, k_all]), (7, beta[0]), (8, [mass]),
                 (8, [mass, mass.cpu()])):
        assert call.calibrate_scales_call(*good[:i], x, *good[i + 1:]) is None, i
    torch.cuda.synchronize()


def test_declined_calls_that_are_in_order_give_the_same_result():
    # Tuples for lists: the ctypes path takes them.
    plan, q, k, _ = _problem("bf16")
    scales = list(range(K))
    lists = scales, [_scale(q, i) for i in scales], [k[:, :, :C[i]].contiguous() for i in scales]
    ws = torch.empty(binding.calibrate_scales_workspace_bytes(plan.shape, scales), dtype=torch.uint8, device="cuda")
    got = []
    for kind in (list, tuple):
        beta = torch.zeros(1, H, K, K, device="cuda")
        mass = kind(torch.zeros(NB, H, K, device="cuda") for _ in scales)
        hk.heatkv_calibrate_scales_accumulate(plan.shape, 0, *(kind(x) for x in lists), SM, 0.5, beta, mass, ws)
        got.append([beta, *mass])
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(*got)) and got[0][0].any()


@pytest.mark.parametrize("given", ["current stream", "stream as a number"])
def test_calls_go_to_the_stream_that_is_meant(given):
    # While `side` is captured, a call that reaches it does not run before the replay.
    plan, q, k, v = _problem("f32")
    want = device_generation(plan, 0, q, k, v, T0, SM, fused=True)
    ka, va = _arenas(plan)
    parts = [[_scale(x, kk) for x in (q, k, v)] for kk in range(K)]
    outs = [torch.zeros_like(p[0]) for p in parts]
    ws = torch.empty(1 << 16, dtype=torch.uint8, device="cuda")
    side, other = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        graph.capture_begin(capture_error_mode="relaxed")
        for kk, (qk, kc, vc) in enumerate(parts):
            if given == "current stream":
                hk.heatkv_attend_append_scale(plan, 0, kk, qk, kc, vc, ka, va, SM, outs[kk], ws)
            else:
                with torch.cuda.stream(other):
                    hk.heatkv_attend_append_scale(plan, 0, kk, qk, kc, vc, ka, va, SM, outs[kk], ws, stream=side.cuda_stream)
        graph.capture_end()
    torch.cuda.synchronize()
    assert not any(o.any() for o in outs)
    for _ in range(3):
        for x in (*outs, ka, va):
            x.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(outs, want))


def test_two_threads_call_at_once():
    # The interpreter's lock is released during the library call; each thread has a stream and arenas of its own.
    plan, *_ = _problem("bf16")
    inputs = [_problem("bf16", seed)[1:] for seed in (5, 6)]
    want = [device_generation(plan, 0, *x, T0, SM, fused=True) for x in inputs]
    wrong = []

    def work(i):
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(20):
                got = device_generation(plan, 0, *inputs[i], T0, SM, fused=True)
                if not all(torch.equal(a, b) for a, b in zip(got, want[i])):
                    wrong.append(i)

    threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong
