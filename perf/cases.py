"""The calls a parameter server makes of this library, as timed cases.

Each case is one call (or one captured graph of calls) through the Python
binding over inputs that are already on the GPU.  The listed cases run from
one LayerNorm tensor to whole model shards; draw() gives other sizes, worker
counts, element types, modes and offsets of the same ranges.

A case is a dict:
  kind    "fused" (aggregate_adam), "dev" (aggregate_adam_dev), "adam"
          (adam_step), "aggregate", "quantize", "multi" (MultiTensorStep) or
          "graph" (aggregate_adam_dev over a list of tensors, captured once)
  n       elements (for multi and graph it follows from the tensor list)
  W       worker contributions
  gdtype  their type: "f32", "bf16" or "i32" (the integer format, fixed mode)
  mode    "fp32" or "fixed" (scale 2^frac_bits)
  place   "shard" (allocate_shard, one slab), "offset" (arrays of their own,
          each a sub-range from element `off` on) or "scattered" (as offset,
          and each contribution at an offset of its own)
  agg     also write the aggregate: "", "f32", "i32" or "both"
"""
import math

import torch

import paper_2409_00918_amd as dd
import synth

DEV = "cuda"
SIGMA = 1e-4             # gradient standard deviation of the shard recipes
HP = dict(lr=1e-4, beta1=0.9, beta2=0.95, eps=1e-8, weight_decay=0.1, step=5)
TORCH = {"f32": torch.float32, "bf16": torch.bfloat16, "i32": torch.int32}
BYTES = {"f32": 4, "bf16": 2, "i32": 4}
HEADLINE_BYTES = 875_000_000 * 58


def _case(kind, n, W=1, gdtype="f32", mode="fp32", frac_bits=0, place="shard", off=0, agg="",
          contiguous=False, **more):
    return dict(kind=kind, n=n, W=W, gdtype=gdtype, mode=mode, frac_bits=frac_bits, place=place,
                off=off, agg=agg, contiguous=contiguous, **more)


def listed():
    opt_layer = dict(hidden=4096, ffn=16384, vocab=50272, positions=2048)
    opt_small = dict(hidden=768, ffn=3072, vocab=50272, positions=2048)
    cases = [
        # one LayerNorm or bias tensor stepped by itself: the smallest call
        ("norm_n4096_w8_f32", _case("fused", 4096, 8, place="offset")),
        # the tiny shard: a working set that fits the last-level cache
        ("tiny_n1M_w4_f32", _case("fused", 1_048_576, 4)),
        # the ten tensors of one decoder layer of an OPT-6.7B shard of 64,
        # one call each, captured once and replayed
        ("layer_graph_w8_f32", _case("graph", 0, 8, layers=1, shards=64, embed=False, pad=0,
                                     **opt_layer)),
        # a layer of a flat shard, a sub-range at an odd element offset
        ("subrange_n2M_w8_f32", _case("fused", 2_097_155, 8, place="offset", off=37)),
        # the optimizer step alone on an aggregate that came from elsewhere:
        # the token embedding of an OPT-6.7B shard of 8
        ("adam_n25M", _case("adam", 25_739_264)),
        # the switch's job alone for many workers (run-time worker count)
        ("aggregate_n25M_w32_bf16", _case("aggregate", 25_739_267, 32, "bf16", agg="f32")),
        # every tensor of a small OPT-style model's shard of 8, each on a
        # 512-byte boundary of its bucket, as separate allocations would be
        ("multi_small_w4_bf16", _case("multi", 0, 4, "bf16", layers=12, shards=8, embed=True,
                                      pad=256, **opt_small)),
        # the 322 tensors of an OPT-6.7B shard of 64, sub-ranges of flat arrays
        ("multi_opt67b_w8_f32", _case("multi", 0, 8, layers=32, shards=64, embed=True, pad=0,
                                      **opt_layer)),
        # a worker's conversion of its 13B/16 contribution
        ("quantize_13b_bf16", _case("quantize", 812_500_000, 1, "bf16", "fixed", 24)),
        # the headline: the 7B/8 shard
        ("opt7b_shard8_w8_f32", _case("fused", 875_000_000, 8, contiguous=True)),
        # the 13B/16 shard, 16 bf16 contributions
        ("opt13b_shard16_w16_bf16", _case("fused", 812_500_000, 16, "bf16", contiguous=True)),
        # integer aggregation of float contributions, with the int32
        # aggregate: an eighth of the 175B/64 shard
        ("c175b_slice_w8_fixed24", _case("fused", 341_796_875, 8, "f32", "fixed", 24, agg="i32",
                                         contiguous=True)),
    ]
    return [dict(c, name=name) for name, c in cases]


def draw(rng):
    """Sizes log-uniform from a bias tensor to a shard, at most the
    headline's bytes; worker counts log-uniform over 1-64."""
    kind = rng.choice(["fused", "fused", "fused", "dev", "adam", "aggregate", "quantize", "multi",
                       "graph"])
    W = min(64, int(math.exp(rng.uniform(0, math.log(65)))))
    gdtype = rng.choice(["f32", "bf16"])
    mode = rng.choice(["fp32", "fp32", "fixed"])
    if mode == "fixed" and rng.random() < 0.3:
        gdtype = "i32"
    frac_bits = rng.choice([16, 20, 24]) if mode == "fixed" else 0
    if kind in ("multi", "graph"):
        hidden = 64 * rng.randint(8, 64)
        case = _case(kind, 0, min(W, 16), gdtype, mode, frac_bits, shards=rng.choice([7, 8, 16, 64]),
                     layers=rng.randint(1, 4) if kind == "graph" else rng.randint(2, 32),
                     embed=kind == "multi", pad=rng.choice([0, 64, 256]), hidden=hidden,
                     ffn=4 * hidden, vocab=50272, positions=2048)
        while work(case)["bytes"] > HEADLINE_BYTES / 2:
            case["shards"] *= 2
        return case
    if kind == "adam":
        W, gdtype, mode, frac_bits = 1, "f32", "fp32", 0
    if kind == "quantize":
        W, mode, frac_bits = 1, "fixed", rng.choice([16, 20, 24])
        gdtype = "f32" if gdtype == "i32" else gdtype
    agg = ""
    if kind == "aggregate":
        agg = "f32" if mode == "fp32" else rng.choice(["f32", "i32", "both"])
    elif kind in ("fused", "dev") and rng.random() < 0.2:
        agg = "f32" if mode == "fp32" else rng.choice(["f32", "i32"])
    place = rng.choice(["shard", "shard", "offset", "scattered"])
    case = _case(kind, 1, W, gdtype, mode, frac_bits, place, 0, agg)
    most = HEADLINE_BYTES // max(per_element(case), 58)
    case["n"] = int(math.exp(rng.uniform(math.log(1000), math.log(most))))
    if place != "shard":
        case["off"] = rng.randint(1, 1000)
    elif case["n"] < 1 << 20:            # a slab's gaps are for shards: plain arrays
        case["place"] = "offset"
    return case


def per_element(case):
    """Bytes one element cannot do without."""
    kind = case["kind"]
    if kind == "quantize":
        return BYTES[case["gdtype"]] + 4
    b = case["W"] * BYTES[case["gdtype"]]
    b += {"": 0, "f32": 4, "i32": 4, "both": 8}[case["agg"]]
    return b if kind == "aggregate" else b + 26   # p, m, v in and out, the bf16 copy out


def tensor_sizes(case):
    sizes = synth.opt_tensor_shards(case["hidden"], case["ffn"], case["layers"], case["vocab"],
                                    case["positions"], case["shards"])
    return sizes if case["embed"] else sizes[2:]


def tensor_starts(case):
    """(starts, sizes, length of the flat arrays) of a tensor list, each
    tensor on a boundary of `pad` elements with at least one element between
    it and the one before (pad 0: back to back)."""
    sizes, starts, at, pad = tensor_sizes(case), [], 0, case["pad"]
    for s in sizes:
        starts.append(at)
        at += s
        if pad:
            at = (at // pad + 1) * pad
    return starts, sizes, at


def work(case):
    n = sum(tensor_sizes(case)) if case["kind"] in ("multi", "graph") else case["n"]
    flops = {"quantize": 2, "aggregate": case["W"]}.get(case["kind"], case["W"] + 17)
    return {"bytes": n * per_element(case), "flops": n * flops}


def tolerance(case):
    # The C ABI states the results bit for bit: the order of the sums, one
    # rounding per operation, correctly rounded divisions and square roots.
    return "exact"


# ------------------------------------------------------------------ inputs --
def _gen(seed, k):
    return torch.Generator(device=DEV).manual_seed((seed * 1_000_003 + k) & ((1 << 62) - 1))


def _fill_grad(t, seed, k, frac_bits):
    """Gradients N(0, SIGMA) with a 1% x100 outlier tail; in the integer
    format, such values at scale 2^frac_bits."""
    gen, n = _gen(seed, k), t.numel()
    x = t if t.dtype != torch.int32 else torch.empty(n, dtype=torch.float32, device=DEV)
    x.normal_(0.0, SIGMA, generator=gen)
    if n >= 100:
        i = torch.randint(n, (n // 100,), generator=gen, device=DEV)
        x[i] = x[i] * 100
    if x is not t:
        t.copy_(x.mul_(2.0 ** frac_bits).round_())


def _fill_state(p, m, v, seed):
    """A state after some steps: weights N(0, 0.02), moments of the
    gradients' size."""
    p.normal_(0.0, 0.02, generator=_gen(seed, 1000))
    m.normal_(0.0, SIGMA, generator=_gen(seed, 1001))
    v.normal_(0.0, SIGMA, generator=_gen(seed, 1002))
    v.mul_(v)


def _length(case):
    return tensor_starts(case)[2] if case["kind"] in ("multi", "graph") else case["n"]


def _place(case):
    """(grads, p, m, v, p16, agg_f32, agg_i32) of a case, uninitialised
    (outputs zeroed), None where it has none."""
    n, W, kind, off = _length(case), case["W"], case["kind"], case["off"]
    state = kind not in ("aggregate", "quantize")
    af = case["agg"] in ("f32", "both")
    ai = case["agg"] in ("i32", "both") or kind == "quantize"
    if case["place"] == "shard" and state:
        sh = dd.allocate_shard(n, W, case["gdtype"], agg_f32=af, agg_i32=ai, device=DEV,
                               contiguous=case["contiguous"])
        p16 = sh.param_bf16.view(torch.bfloat16)
        grads = [g.view(torch.bfloat16) if case["gdtype"] == "bf16" else g for g in sh.grads]
        got = [grads, sh.param, sh.m, sh.v, p16, sh.agg_f32, sh.agg_i32]
    else:
        def array(dtype, o):
            return torch.empty(o + n, dtype=dtype, device=DEV)[o:]
        at = [off + 2 * (w * w % 23) if case["place"] == "scattered" else off for w in range(W)]
        got = [[array(TORCH[case["gdtype"]], o) for o in at]]
        got += [array(torch.float32, off) if state else None for _ in range(3)]
        got += [array(torch.bfloat16, off) if state else None,
                array(torch.float32, off) if af else None,
                array(torch.int32, off) if ai else None]
    for t in got[4:]:
        if t is not None:
            t.zero_()
    return got


def prepare(case, seed):
    arrays = _place(case)
    grads, p, m, v, p16, agg_f32, agg_i32 = arrays
    for w, g in enumerate(grads):
        _fill_grad(g, seed, w, case["frac_bits"])
    if p is not None:
        _fill_state(p, m, v, seed)
    s = dict(kind=case["kind"], grads=grads, p=p, m=m, v=v, p16=p16, agg_f32=agg_f32,
             agg_i32=agg_i32, agg=dict(mode=case["mode"], frac_bits=case["frac_bits"]))
    if case["kind"] in ("dev", "graph"):
        sc = dd.step_scalars(**HP)
        s["scalars"] = torch.frombuffer(bytearray(sc), dtype=torch.float32).to(DEV)
    if case["kind"] in ("multi", "graph"):
        starts, sizes, _ = tensor_starts(case)
        tensors = [([g[a:a + k] for g in grads], p[a:a + k], m[a:a + k], v[a:a + k], p16[a:a + k])
                   for a, k in zip(starts, sizes)]
        if case["kind"] == "multi":
            s["step"] = dd.MultiTensorStep(tensors, **s["agg"])
        else:
            s["graph"] = torch.cuda.CUDAGraph()
            with torch.cuda.graph(s["graph"]):
                for t in tensors:
                    dd.aggregate_adam_dev(*t, scalars=s["scalars"], **s["agg"])
    return s


def run(s):
    kind, out = s["kind"], dict(agg_out_f32=s["agg_f32"], agg_out_i32=s["agg_i32"])
    if kind == "fused":
        dd.aggregate_adam(s["grads"], s["p"], s["m"], s["v"], s["p16"], **HP, **s["agg"], **out)
    elif kind == "dev":
        dd.aggregate_adam_dev(s["grads"], s["p"], s["m"], s["v"], s["p16"], scalars=s["scalars"],
                              **s["agg"], **out)
    elif kind == "adam":
        dd.adam_step(s["grads"][0], s["p"], s["m"], s["v"], s["p16"], **HP)
    elif kind == "aggregate":
        dd.aggregate(s["grads"], **s["agg"], **out)
    elif kind == "quantize":
        dd.quantize(s["grads"][0], s["agg_i32"], frac_bits=s["agg"]["frac_bits"])
    elif kind == "multi":
        s["step"](**HP)
    else:
        s["graph"].replay()
    return [s[k] for k in ("p", "m", "v", "p16", "agg_f32", "agg_i32") if s[k] is not None]


def exact(case, seed):
    """The same outputs in 64-bit torch (no value in the place of integers).
    Fixed mode's conversion to the integer format is part of the result."""
    kind, n, frac = case["kind"], _length(case), case["frac_bits"]
    if kind == "quantize":               # whole numbers only
        return None
    grads = [torch.empty(n, dtype=TORCH[case["gdtype"]], device=DEV) for _ in range(case["W"])]
    for w, g in enumerate(grads):
        _fill_grad(g, seed, w, frac)
    state = kind != "aggregate"
    p = m = v = None
    if state:
        p, m, v = (torch.empty(n, dtype=torch.float32, device=DEV) for _ in range(3))
        _fill_state(p, m, v, seed)
    af = case["agg"] in ("f32", "both")
    outs = [torch.empty(n, dtype=torch.float64, device=DEV) for _ in range(3 * state + af)]
    f32 = torch.tensor([HP[k] for k in ("lr", "beta1", "beta2", "eps", "weight_decay")])
    lr, b1, b2, eps, wd = f32.double().tolist()      # as the call's fp32 arguments hold them
    t = HP["step"]
    for a in range(0, n, 1 << 25):
        cut = slice(a, min(n, a + (1 << 25)))
        g = torch.zeros(cut.stop - a, dtype=torch.float64, device=DEV)
        for x in grads:
            x = x[cut].double()
            if case["mode"] == "fixed" and case["gdtype"] != "i32":
                x = (x * 2.0 ** frac).round_().clamp_(-2.0 ** 31, 2.0 ** 31 - 1)
            g += x
        if case["mode"] == "fixed":
            g = g.clamp_(-2.0 ** 31, 2.0 ** 31 - 1) * 2.0 ** -frac
        if state:
            mm = b1 * m[cut].double() + (1 - b1) * g
            vv = b2 * v[cut].double() + (1 - b2) * g * g
            d = (vv / (1 - b2 ** t)).sqrt_() + eps
            outs[0][cut] = p[cut].double() * (1 - lr * wd) - lr * (mm / (1 - b1 ** t)) / d
            outs[1][cut], outs[2][cut] = mm, vv
        if af:
            outs[-1][cut] = g
    if kind in ("multi", "graph") and case["pad"]:   # what lies between the tensors stays
        starts, sizes, _ = tensor_starts(case)
        gap = torch.ones(n, dtype=torch.bool, device=DEV)
        for a, k in zip(starts, sizes):
            gap[a:a + k] = False
        for out, x in zip(outs, (p, m, v)):
            out[gap] = x[gap].double()
    if state:
        p16 = outs[0] if not (kind in ("multi", "graph") and case["pad"]) else None
        outs = outs[:3] + [p16] + outs[3:]
    return outs + ([None] if case["agg"] in ("i32", "both") else [])
