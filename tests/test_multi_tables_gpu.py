"""Lists of tensors around the sizes where a many-tensor call packs its
launches differently: tensors that follow one another (one tensor to the
kernels), slices of flat buffers (232 to a launch at W = 8, found in steps of
16), buffers of their own (36 rows of W + 4 pointers), and the smallest tensors,
which may have no whole group of four elements.  Every bit against the oracle
on the flat arrays, and nothing written between the tensors.
"""
import numpy as np
import pytest

import oracle
import synth
from gpu_common import HP, assert_parity, to_dev, to_host, torch

pytestmark = pytest.mark.gpu

KW = dict(lr=HP["lr"], beta1=HP["beta1"], beta2=HP["beta2"], eps=HP["eps"],
          weight_decay=HP["wd"])


def _sizes(T, seed):
    rng = np.random.default_rng(seed)
    n = rng.choice([1, 2, 3, 4, 5, 63, 255, 256, 257, 260, 1023, 2051], T)
    n[rng.integers(T)] = 0
    n[0] = max(n[0], 1)
    return [int(x) for x in n]


@pytest.mark.parametrize("pad", ["adjacent", "gaps", "own", "mixed"])
@pytest.mark.parametrize("T,W,gdtype,mode,off", [
    (2, 8, "f32", "fp32", 0), (15, 1, "f32", "fp32", 1), (16, 8, "f32", "fp32", 37),
    (17, 4, "bf16", "fp32", 2), (239, 2, "f32", "fixed", 0), (240, 8, "bf16", "fixed", 6),
    (241, 1, "bf16", "fp32", 0), (500, 13, "f32", "fp32", 3), (70, 64, "bf16", "fp32", 0),
    (40, 16, "f32", "fp32", 255), (36, 8, "bf16", "fp32", 4), (37, 8, "f32", "fixed", 9),
    (232, 8, "f32", "fp32", 4), (233, 8, "bf16", "fp32", 0)])
def test_packed_launches_match_oracle(pad, T, W, gdtype, mode, off):
    import paper_2409_00918_amd as dd
    sizes = _sizes(T, T)
    rng = np.random.default_rng(T + 1)
    starts, at = [], 0
    for j, s in enumerate(sizes):
        starts.append(at)
        at += s
        if pad == "gaps" or (pad == "mixed" and j % 5 == 0):
            at += 2 * int(rng.integers(1, 200))
    n = at
    gs = synth.host_grads(700 + T, 2, W, n, 1e-4, gdtype=gdtype, outlier_frac=0.01,
                          outlier_scale=100.0)
    p, m, v = synth.host_state(700 + T, n, mv_sigma=1e-4)
    if pad == "own":
        def cut(a):
            return [to_dev(a[s:s + k], off) for s, k in zip(starts, sizes)]
    else:
        def cut(a):
            flat = to_dev(a, off)
            return [flat[s:s + k] for s, k in zip(starts, sizes)]
    dg = [cut(g) for g in gs]
    dp, dm, dv, dc = cut(p), cut(m), cut(v), cut(np.full(n, 0x1234, np.uint16))
    dd.MultiTensorStep([([dg[w][j] for w in range(W)], dp[j], dm[j], dv[j], dc[j])
                        for j in range(T)], mode=mode, frac_bits=24)(step=2, **KW)
    torch().cuda.synchronize()
    want = oracle.fused(gs, p, m, v, mode=oracle.AGG_FIXED if mode == "fixed" else oracle.AGG_FP32,
                        frac_bits=24, t=2, **HP)
    inside = np.zeros(n, bool)
    for s, k in zip(starts, sizes):
        inside[s:s + k] = True
    for key, old in (("p", p), ("m", m), ("v", v), ("p16", np.full(n, 0x1234, np.uint16))):
        want[key] = np.where(inside, want[key], old)

    def whole(parts, old):
        if pad != "own":                       # the flat array the slices view
            first = parts[0]
            flat = torch().empty(0, dtype=first.dtype, device="cuda")
            flat.set_(first.untyped_storage(), first.storage_offset(), (n,))
            return to_host(flat)
        out = old.copy()
        for s, k, x in zip(starts, sizes, parts):
            out[s:s + k] = to_host(x)
        return out

    got = {"p": whole(dp, p), "m": whole(dm, m), "v": whole(dv, v),
           "p16": whole(dc, np.full(n, 0x1234, np.uint16))}
    assert_parity(got, want, f"{pad} T={T} W={W} {gdtype} {mode} off={off}")
