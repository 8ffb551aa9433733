"""Performance cases of the HeatKV path: what a user of this framework has it do, through its public entry points.

A case is a dict of plain values.  The fields of the problem are those of heatkv_inputs.CONFIGS (layers L, heads H,
head dimension d, dtype, batch, token maps, sinks, compression factor); `what` says which part of the path runs:

  generate        every scale of an image, every layer: attention and cache update in one call, generation order
  separate        the same with heatkv_attend_scale and heatkv_append_scale as two calls
  cache_update    the cache updates of an image alone
  calibrate       calibration masses of all scales of one layer in one call, averaged into beta
  calibrate_each  the same with one call per scale
  schedule        the pruning schedule from a beta table, and its tables on the device

Token maps are written as "1x1 2x2 4x4 ..." (height x width per scale).  Activations come from the seed; the plan is
part of what a program keeps, so it is the same for every seed (the head weights behind it are those of seed 0), except
in `schedule`, whose input is the beta table.
"""
import math

import numpy as np
import torch

import heatkv_inputs as hi
import paper_2605_14877_amd as hk


def _square(sides):
    return " ".join(f"{s}x{s}" for s in sides)


PYRAMID_1024 = _square(hi.SIDES_1024)                         # a 1024 x 1024 image: 13 scales, 10521 tokens
PYRAMID_256 = _square((1, 2, 3, 4, 5, 6, 8, 10, 13, 16))      # a 256 x 256 image: 10 scales, 680 tokens
PYRAMID_2TO1 = "1x2 2x3 3x6 5x10 7x13 9x19 12x23 17x34 24x47"  # a 2:1 image, odd token counts

_DEFAULT = dict(what="generate", L=1, H=16, d=128, dtype="bf16", batch=2, maps=PYRAMID_1024, sinks=3, factor=4,
                variant=hk.VARIANT_HEATKV, fp8=False)


def _case(name, **fields):
    case = dict(_DEFAULT, **fields)
    if name is not None:
        case["name"] = name
    return case


def listed():
    return [
        # The smallest problem: one fp32 layer of 4 heads, 85 tokens in all.  A few calls of almost no work.
        _case("tiny_f32_image", H=4, d=64, dtype="f32", batch=1, maps=_square(hi.SIDES_TINY), sinks=1, factor=2),
        # One layer of a 2B-like model generating one image with its guidance row: the default benchmark's attention.
        _case("layer2b_image"),
        # One image at a time through layers of an 8B-like model, 20x compression: interactive use.
        _case("stack8b_image", L=6, H=32, factor=20),
        # Sixteen images with their guidance rows at once, 20x compression: serving throughput on a full chip.
        _case("serving_images", L=2, batch=32, factor=20),
        # The same with the cache rows stored as 8-bit codes.
        _case("serving_images_fp8_cache", L=2, batch=32, factor=20, fp8=True),
        # 256 x 256 images, head dimension 64, eight images at once: many short launches.
        _case("small_images_d64", L=4, d=64, batch=16, maps=PYRAMID_256),
        # A 2:1 image with odd token counts, odd batch, binary schedule, attention and cache update as two calls.
        _case("wide_image_separate_calls", what="separate", L=2, batch=3, maps=PYRAMID_2TO1, sinks=2,
              variant=hk.VARIANT_BINARY),
        # The cache updates of the serving load alone: a program that runs its own attention, or updates on the side.
        _case("serving_cache_update", what="cache_update", L=2, batch=32, factor=20),
        # Offline calibration of one 2B-like layer on one image with its guidance row, all scales in one call.
        _case("layer2b_calibrate", what="calibrate"),
        # Offline calibration in fp32, scale by scale: the numerics check that goes before a deployment.
        _case("calibrate_f32_each_scale", what="calibrate_each", H=8, dtype="f32", maps=_square((1, 2, 4, 6, 8, 12, 16, 20)),
              sinks=2),
        # Generation in fp32 (reference outputs for a bf16 deployment), ragged token counts.
        _case("image_f32", L=2, H=8, dtype="f32", maps=_square((1, 2, 4, 7, 9, 13, 18, 25)), sinks=2),
        # Building a schedule for a whole 8B-like stack, as after every calibration or change of budget.
        _case("stack8b_schedule", what="schedule", L=40, H=32, factor=20),
    ]


def _log_uniform(rng, lo, hi_):
    return math.exp(rng.uniform(math.log(lo), math.log(hi_)))


def _draw_maps(rng, top, n):
    """n token maps growing from about one token to `top` x `top` tokens, of one aspect ratio, sizes off the grid."""
    aspect = rng.choice((1.0, 1.0, 1.0, 0.5, 0.75, 1.5, 2.0))
    maps, last = [], 0
    for i in range(n):
        side = top ** (i / (n - 1)) * rng.uniform(0.93, 1.0)
        h = max(1, round(side / math.sqrt(aspect)))
        w = max(1, round(side * math.sqrt(aspect)))
        while h * w <= last:
            w += 1
        last = h * w
        maps.append((h, w))
    return maps


def draw(rng):
    what = rng.choice(("generate",) * 9 + ("separate",) * 3 + ("cache_update",) * 2 + ("calibrate",) * 3 +
                      ("calibrate_each", "schedule"))
    dtype = "bf16" if what == "schedule" else rng.choice(("bf16",) * 4 + ("f32",))
    top = _log_uniform(rng, 6, 64 if dtype == "bf16" else 28)
    n = rng.randint(5, 13) if top > 12 else rng.randint(4, 8)
    case = _case(None, what=what, dtype=dtype, d=rng.choice((64, 128, 128)), H=rng.randint(3, 32),
                 batch=round(_log_uniform(rng, 1, 32)),
                 L=round(_log_uniform(rng, 1, 40 if what == "schedule" else 6)),
                 maps=" ".join(f"{h}x{w}" for h, w in _draw_maps(rng, top, n)), sinks=rng.randint(1, min(3, n - 2)),
                 factor=round(_log_uniform(rng, 1, 20)), variant=rng.choice((hk.VARIANT_HEATKV,) * 3 + (hk.VARIANT_BINARY,)))
    case["fp8"] = dtype == "bf16" and case["d"] == 128 and what in ("generate", "separate", "cache_update") and \
        rng.random() < 0.3
    if what.startswith("calibrate"):
        case["L"] = 1
    while what != "schedule" and _cost(case) > 0.8 * _COST_CAP:  # no drawn case costs more than the largest listed one
        if case["batch"] > 1:
            case["batch"] //= 2
        elif case["L"] > 1:
            case["L"] //= 2
        else:
            case["H"] = max(1, case["H"] // 2)
    return case


def _cost(case):
    """Upper bound of the time of a pass, in seconds, at modest rates; from the sizes alone."""
    t = _tokens(case)
    c = hi.cumulative_tokens(t)
    pairs = case["L"] * case["H"] * case["batch"]
    flops = 4.0 * case["d"] * pairs * sum(a * b for a, b in zip(t, c))
    return flops / (0.5e15 if case["dtype"] == "bf16" else 4e12) + pairs * c[-1] * case["d"] * 4e-12 + 5e-5


_COST_CAP = 0.03  # about the time of the largest listed case


def _tokens(case):
    return hi.tokens_per_scale([tuple(int(x) for x in m.split("x")) for m in case["maps"].split()])


def _budget_bytes(case, t, c):
    """KV bytes of a sequence at the case's compression factor, but no less than its sink scales and a little."""
    heads = case["L"] * case["H"]
    rows = max(heads * c[-2] // case["factor"], heads * c[case["sinks"] - 1] + c[-2])
    return rows * 2 * case["d"] * (1 if case["fp8"] else hi.elem_bytes(case["dtype"]))


def _shape(case, t):
    return hk.Shape(case["L"], case["H"], case["d"], t, case["batch"], case["dtype"])


def _plan(case):
    """Shape, planted head weights and schedule of a case (host only)."""
    t = _tokens(case)
    c = hi.cumulative_tokens(t)
    w = hi.head_weights(0, case["L"], case["H"], len(t))
    beta = hi.expected_beta_from_weights(w, t).astype(np.float32)
    shape = _shape(case, t)
    plan = hk.heatkv_build_schedule(shape, beta, _budget_bytes(case, t, c), case["sinks"], case["variant"],
                                    hk.KV_FP8_E4M3 if case["fp8"] else hk.KV_NATIVE)
    return t, c, w, shape, plan


def prepare(case, seed):
    dev = torch.device("cuda:0")
    t = _tokens(case)
    c = hi.cumulative_tokens(t)
    K = len(t)
    st = {"what": case["what"], "K": K, "L": case["L"], "sm": 1.0 / math.sqrt(case["d"])}
    if case["what"] == "schedule":
        w = hi.head_weights(seed, case["L"], case["H"], K)
        st.update(shape=_shape(case, t), beta=hi.expected_beta_from_weights(w, t).astype(np.float32),
                  budget=_budget_bytes(case, t, c), sinks=case["sinks"], variant=case["variant"])
        return st
    cfg = dict(case, sides=[tuple(int(x) for x in m.split("x")) for m in case["maps"].split()])
    cut = [slice(c[k] - t[k], c[k]) for k in range(K)]
    if case["what"].startswith("calibrate"):
        w = hi.head_weights(0, case["L"], case["H"], K)
        q, k, _ = hi.make_qkv_device(seed, 0, cfg, w, dev)
        shape = _shape(case, t)
        scales = list(range(K))
        st.update(shape=shape, scales=scales, weight=1.0 / case["batch"],
                  q=[q[:, :, s].contiguous() for s in cut], k_all=[k[:, :, :c[i]].contiguous() for i in scales],
                  beta=torch.zeros(case["L"], case["H"], K, K, device=dev),
                  mass=[torch.zeros(case["batch"], case["H"], K, device=dev) for _ in scales])
        if case["what"] == "calibrate":
            st["ws"] = torch.empty(hk.binding.calibrate_scales_workspace_bytes(shape, scales), dtype=torch.uint8, device=dev)
        else:
            st["ws"] = torch.empty(max(hk.binding.calibrate_workspace_bytes(shape, i) for i in scales),
                                   dtype=torch.uint8, device=dev)
        return st
    t, c, w, shape, plan = _plan(case)
    plan.upload()
    acts, outs = [], []  # acts[l][k] = (q, k, v, out); the outputs of a layer's scales lie in one buffer
    for layer in range(case["L"]):
        q, k, v = hi.make_qkv_device(seed, layer, cfg, w, dev)
        outs.append(torch.zeros(q.numel(), dtype=q.dtype, device=dev))
        parts = torch.split(outs[-1], [case["batch"] * case["H"] * n * case["d"] for n in t])
        acts.append([(q[:, :, s].contiguous(), k[:, :, s].contiguous(), v[:, :, s].contiguous(),
                      parts[i].view(case["batch"], case["H"], t[i], case["d"])) for i, s in enumerate(cut)])
        del q, k, v
    ws_bytes = max(plan.attend_workspace_bytes(layer, k) for layer in range(case["L"]) for k in range(K))
    st.update(plan=plan, acts=acts, outs=outs, ws=torch.empty(max(ws_bytes, 4), dtype=torch.uint8, device=dev),
              k_arena=torch.zeros(max(plan.arena_bytes, 16), dtype=torch.uint8, device=dev),
              v_arena=torch.zeros(max(plan.arena_bytes, 16), dtype=torch.uint8, device=dev))
    return st


def run(st):
    what, sm = st["what"], st["sm"]
    if what == "schedule":
        plan = hk.heatkv_build_schedule(st["shape"], st["beta"], st["budget"], st["sinks"], st["variant"])
        plan.upload()
        return [plan.N(), plan.sets(st["K"] - 1, hk.binding.SET_A), np.array([plan.arena_tokens])]
    if what == "calibrate":
        st["beta"].zero_()
        hk.heatkv_calibrate_scales_accumulate(st["shape"], 0, st["scales"], st["q"], st["k_all"], sm, st["weight"],
                                              st["beta"], st["mass"], st["ws"])
        return [st["beta"]] + st["mass"]
    if what == "calibrate_each":
        st["beta"].zero_()
        for k in st["scales"]:
            hk.heatkv_calibrate_accumulate(st["shape"], 0, k, st["q"][k], st["k_all"][k], sm, st["weight"], st["beta"],
                                           st["mass"][k], st["ws"])
        return [st["beta"]] + st["mass"]
    plan, ka, va, ws = st["plan"], st["k_arena"], st["v_arena"], st["ws"]
    for k in range(st["K"]):
        for layer in range(st["L"]):
            q, kc, vc, out = st["acts"][layer][k]
            if what == "generate":
                hk.heatkv_attend_append_scale(plan, layer, k, q, kc, vc, ka, va, sm, out, ws)
            elif what == "separate":
                hk.heatkv_attend_scale(plan, layer, k, q, kc, vc, ka, va, sm, out, ws)
                hk.heatkv_append_scale(plan, layer, k, kc, vc, ka, va)
            else:
                hk.heatkv_append_scale(plan, layer, k, kc, vc, ka, va)
    if what == "cache_update":
        return [ka, va]
    return st["outs"]


def work(case):
    """Algorithmic bytes and operations of one pass: every input read once, every output written once."""
    t = _tokens(case)
    c = hi.cumulative_tokens(t)
    K, rows = len(t), case["batch"] * case["H"]
    d, esz = case["d"], hi.elem_bytes(case["dtype"])
    if case["what"] == "schedule":
        table = case["L"] * case["H"] * K
        return {"bytes": table * K * 4 + table * 16, "flops": table * K / 2}
    if case["what"].startswith("calibrate"):
        return {"bytes": sum(rows * (t[k] + c[k]) * d * esz + rows * K * 4 for k in range(K)),
                "flops": sum(2.0 * d * t[k] * c[k] * rows for k in range(K))}
    plan = _plan(case)[4]
    kv = d * (1 if case["fp8"] else esz)  # bytes of a cached K or V row
    byts = flops = 0.0
    for layer in range(case["L"]):
        prior = [case["batch"] * int(plan.runs(k, layer)[1].astype(np.int64).sum()) for k in range(K)]
        for k in range(K):
            new = 0  # rows of scale k that enter the cache
            if k + 1 < K:
                for h in range(case["H"]):
                    ids = plan.retained(k + 1, layer, h)
                    new += case["batch"] * t[k] if len(ids) and ids[-1] == c[k] - 1 else 0
            if case["what"] == "cache_update":  # a layer's runs are rewritten into the region that the next scale reads
                if k + 1 < K:
                    byts += 2.0 * (kv * prior[k + 1] + kv * (prior[k + 1] - new) + d * esz * new)
            else:
                flops += 4.0 * t[k] * d * (prior[k] + rows * t[k])
                byts += 4.0 * rows * t[k] * d * esz + 2.0 * kv * (prior[k] + new)
    return {"bytes": byts, "flops": flops}


def tolerance(case):
    if case["what"] in ("cache_update", "schedule"):
        return "exact"
    # Measured against the same path in fp64 over the listed cases (norm, largest element); stated: about four times.
    if case["what"].startswith("calibrate"):  # 9.4e-8, 2.6e-7: fp32 sums of probabilities
        return {"rel": 5e-7, "max": 2e-6}
    if case["dtype"] == "f32":  # 6.9e-7, 5.4e-6: fp32 scores, probabilities and sums
        return {"rel": 3e-6, "max": 2.5e-5}
    return {"rel": 1e-2, "max": 6e-2}  # 2.4e-3, 1.5e-2: probabilities and outputs rounded to bf16
