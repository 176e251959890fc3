"""The native half of the binding: it takes calls in the ordinary form and
leaves every other to the Python code, without having done anything.  On the
GPU, both ways must give the same bits and the same errors."""
import os
import subprocess
import sys

import numpy as np
import pytest
import torch

import paper_2409_00918_amd as dd

KW = dict(lr=1e-4, beta1=0.9, beta2=0.95, eps=1e-8, weight_decay=0.1, step=3)


class Sub(torch.Tensor):
    pass


def _native(op, grads, p=None, m=None, v=None, c=None, af=None, ai=None, sc=None, mode="fp32",
            frac=0, step=1):
    dd.lib()
    return dd._call(op, grads, p, m, v, c, af, ai, sc, mode, frac, 1e-4, 0.9, 0.95, 1e-8, 0.1,
                    step, 1.0)


@pytest.mark.parametrize("grads", [
    lambda: [torch.zeros(8)] * 2,                                   # host tensors
    lambda: (torch.zeros(8) for _ in range(2)),                     # an iterator (not consumed)
    lambda: [], lambda: None, lambda: [1, 2], lambda: [torch.zeros(8)] * 65,
    lambda: [torch.zeros(8).as_subclass(Sub)], lambda: [torch.zeros(8, dtype=torch.float64)]])
def test_other_forms_are_left_to_python(grads):
    out = torch.zeros(8)
    g = grads()
    assert _native(dd._AGGREGATE, g, af=out) == -1
    if hasattr(g, "__next__"):
        assert len(list(g)) == 2
    assert _native(dd._FUSED, g, p=out, m=out, v=out) == -1


def test_odd_arguments_are_left_to_python():
    g = [torch.zeros(8)]
    assert _native(dd._AGGREGATE, g, mode="float") == -1
    assert _native(dd._AGGREGATE, g, frac=2.0) == -1
    assert _native(dd._AGGREGATE, g, frac=1 << 40) == -1
    assert _native(dd._FUSED, g, step=1 << 70) == -1
    assert _native(dd._FUSED, g, step="x") == -1
    assert _native(9, g) == -1
    with pytest.raises(TypeError):
        dd._call(0)
    with pytest.raises(ValueError):
        dd.aggregate([torch.zeros(8)], mode="float", agg_out_f32=torch.zeros(8))


def test_without_the_native_half_python_takes_every_call():
    code = """
import sys, warnings
sys.modules["paper_2409_00918_amd._binding"] = None      # an import of it fails
import torch
import paper_2409_00918_amd as dd
with warnings.catch_warnings(record=True) as seen:
    warnings.simplefilter("always")
    assert dd.status_string(0) == "ok"
assert any("_binding" in str(w.message) for w in seen), seen
assert dd.raw_aggregate([0], 1, dd.DT_F32, 0, dd.AGG_FP32, 0, 0, 0, 0) == dd.OK
assert dd._call(dd._AGGREGATE, [torch.zeros(8)]) == -1
try:
    dd.aggregate([torch.zeros(8)], agg_out_f32=torch.zeros(8))
except ValueError as e:
    assert "device tensor" in str(e)
else:
    raise AssertionError("a host tensor was taken")
"""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", code], cwd=root, capture_output=True, text=True,
                       timeout=120)
    assert r.returncode == 0, r.stderr


def _tensors(n, W, gdtype):
    gen = torch.Generator(device="cuda").manual_seed(n + W)
    def r(scale):
        return torch.randn(n, generator=gen, device="cuda") * scale
    g = [r(1e-4) for _ in range(W)]
    if gdtype == "bf16":
        g = [x.bfloat16() for x in g]
    elif gdtype == "i32":
        g = [(x * 2.0**24).round().int() for x in g]
    return g, r(0.02), r(1e-4), r(1e-4) ** 2


@pytest.mark.gpu
@pytest.mark.parametrize("n", [1, 4099])
@pytest.mark.parametrize("gdtype,mode", [("f32", "fp32"), ("bf16", "fp32"), ("f32", "fixed"),
                                         ("i32", "fixed")])
def test_both_ways_give_the_same_bits(n, gdtype, mode, monkeypatch):
    dd.lib()
    native, taken = dd._call, []
    def call(op, *args):
        st = native(op, *args)
        taken.append((op, st))
        return st
    monkeypatch.setattr(dd, "_call", call)
    g, p, m, v = _tensors(n, 3, gdtype)
    sc = torch.frombuffer(bytearray(dd.step_scalars(**KW)), dtype=torch.float32).cuda()
    here = torch.cuda.current_stream()               # an explicit stream: the Python way
    got = []
    for stream in (None, here):
        out = []
        for op in ("fused", "dev", "adam", "aggregate", "quantize"):
            P, M, V = torch.nn.Parameter(p.clone()), m.clone(), v.clone()
            c = torch.zeros(n, dtype=torch.int16, device="cuda")
            af = torch.zeros(n, device="cuda")
            ai = torch.zeros(n, dtype=torch.int32, device="cuda") if mode == "fixed" else None
            agg = dict(mode=mode, frac_bits=24, agg_out_f32=af, agg_out_i32=ai, stream=stream)
            if op == "fused":
                dd.aggregate_adam(tuple(g), P, M, V, c, **KW, **agg)
            elif op == "dev":
                dd.aggregate_adam_dev(g, P, M, V, c, scalars=sc, **agg)
            elif op == "adam":
                dd.adam_step(m, P, M.add_(1e-6), V, None, **KW, stream=stream)
            elif op == "aggregate":
                dd.aggregate(g, **agg)
            elif gdtype != "i32":
                ai = torch.zeros(n, dtype=torch.int32, device="cuda")
                dd.quantize(g[0], ai, frac_bits=20, stream=stream)
            torch.cuda.synchronize()
            out += [x.detach().cpu().numpy().tobytes() for x in (P, M, V, c, af, ai)
                    if x is not None]
        got.append(out)
    assert got[0] == got[1]
    # the native half took every call without a stream, none of the others saw it
    ops = [dd._FUSED, dd._FUSED_DEV, dd._ADAM_STEP, dd._AGGREGATE]
    ops += [dd._QUANTIZE] if gdtype != "i32" else []
    assert taken == [(op, dd.OK) for op in ops]


@pytest.mark.gpu
def test_pinned_memory_is_left_to_python(monkeypatch):
    dd.lib()
    native, taken = dd._call, []
    monkeypatch.setattr(dd, "_call", lambda *a: taken.append(native(*a)) or taken[-1])
    g, p, m, v = _tensors(4096, 2, "f32")
    want = [p.clone(), m.clone(), v.clone()]
    dd.aggregate_adam(g, *want, None, **KW)
    host = torch.empty(4096, pin_memory=True)
    host.copy_(m)
    torch.cuda.synchronize()
    dd.aggregate_adam(g, p, host, v, None, **KW)
    torch.cuda.synchronize()
    assert taken == [dd.OK, -1]
    assert torch.equal(p, want[0]) and torch.equal(host, want[1].cpu()) and torch.equal(v, want[2])


@pytest.mark.gpu
def test_both_ways_raise_the_same_errors():
    g, p, m, v = _tensors(64, 2, "f32")
    here = torch.cuda.current_stream()
    wide = torch.zeros(128, device="cuda")
    def fused(stream, grads=g, P=p, M=m, V=v, c=None, **kw):
        dd.aggregate_adam(grads, P, M, V, c, stream=stream, **{**KW, **kw})
    bad = [dict(P=m), dict(step=0), dict(grads=[]), dict(grads=[g[0], wide]), dict(P=wide[::2]),
           dict(M=m.double()), dict(c=torch.zeros(64, device="cuda")), dict(V=v.cpu()),
           dict(mode="mean"), dict(lr="x"), dict(beta1=1.0), dict(grads=[g[0], g[1].bfloat16()]),
           dict(grads=[x.int() for x in g]), dict(P=None)]
    for kw in bad:
        seen = []
        for stream in (None, here):
            with pytest.raises(Exception) as e:
                fused(stream, **kw)
            seen.append((type(e.value), str(e.value)))
        assert seen[0] == seen[1], kw
    ai = torch.zeros(64, dtype=torch.int32, device="cuda")
    sc = torch.zeros(10, device="cuda")
    # a caller's None is not "an argument this operation does not take"
    nones = [lambda s: fused(s, mode=None), lambda s: fused(s, mode="fixed", frac_bits=None),
             lambda s: dd.aggregate(g, mode=None, agg_out_f32=wide[:64], stream=s),
             lambda s: dd.aggregate(g, frac_bits=None, agg_out_f32=wide[:64], stream=s),
             lambda s: dd.aggregate_adam_dev(g, p, m, v, scalars=sc, mode=None, stream=s),
             lambda s: dd.aggregate_adam_dev(g, p, m, v, scalars=sc, frac_bits=None, stream=s),
             lambda s: dd.aggregate_adam_dev(g, p, m, v, scalars=None, stream=s),
             lambda s: dd.quantize(g[0], ai, frac_bits=None, stream=s),
             lambda s: dd.quantize(g[0], None, frac_bits=20, stream=s),
             lambda s: fused(s, lr=None), lambda s: fused(s, step=None)]
    for k, call in enumerate(nones):
        seen = []
        for stream in (None, here):
            with pytest.raises(Exception) as e:
                call(stream)
            seen.append((type(e.value), str(e.value)))
        assert seen[0] == seen[1], k
    assert not wide.any() and not ai.any()
    with pytest.raises(Exception):
        torch.func.vmap(lambda x: fused(None, P=x))(torch.stack([p, p]))
    assert np.isfinite(p.cpu().numpy()).all()
