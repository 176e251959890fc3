"""Launches that give each XCD two neighbouring tiles (many bf16 contributions,
more than 20 rounds of resident waves): every element against the oracle, at
lengths that end inside, at and just past the last whole set of 16 blocks, with
and without a head, in every kernel that may take the order.

Whether a launch takes the order depends on the distances of the contributions
too.  They lie at a chosen spacing in one allocation, and launch_check (the
launch's host code) is asked whether these very addresses take it."""
import os
import subprocess

import numpy as np
import pytest

import oracle
import synth
from gpu_common import HP, assert_parity, to_dev, to_host, torch

pytestmark = pytest.mark.gpu

SET = 16 * 256                       # elements of 16 tiles
BASE = 2048 * SET                    # 8.4M elements
MIB = 1 << 20
CHECK = os.path.join(os.path.dirname(os.path.abspath(__file__)), "native", "launch_check")


def _contributions(gs, off, apart):
    """Device copies of `gs`, each `off` elements past a boundary, the
    boundaries `apart` bytes from each other in one allocation."""
    t = torch()
    buf = t.empty(len(gs) * apart + MIB, dtype=t.uint8, device="cuda")
    out = []
    for w, g in enumerate(gs):
        x = buf[w * apart + 2 * off:][:2 * g.size].view(t.int16)
        x.copy_(t.from_numpy(g.view(np.int16)))
        out.append(x)
    return out


def _takes_the_order(grads, mode, adam, n, head):
    ptrs = [str(g.data_ptr() + 2 * head) for g in grads]
    r = subprocess.run([CHECK, "order", "1", "1" if mode == "fixed" else "0", str(int(adam)),
                        str(n - head), *ptrs], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stderr
    return int(r.stdout)


@pytest.mark.parametrize("W,mode,n,off,apart,taken", [
    (12, "fp32", 2 * BASE, 0, 34, 1), (16, "fp32", BASE + 5, 0, 18, 1),
    (16, "fixed", 2 * BASE + SET - 1, 37, 34, 1), (20, "fp32", 2 * BASE + 256 * 15 + 3, 2, 34, 1),
    (20, "fixed", 2 * BASE + 1, 0, 34, 1), (16, "fp32", 2 * BASE + SET + 1, 0, 64, 0)])
def test_fused(W, mode, n, off, apart, taken):
    import paper_2409_00918_amd as dd
    gs = synth.host_grads(700 + W, 2, W, n, 1e-4, gdtype="bf16", outlier_frac=0.01,
                          outlier_scale=100.0)
    p, m, v = synth.host_state(700 + W, n, mv_sigma=1e-4)
    dg = _contributions(gs, off, apart * MIB)
    dp, dm, dv, d16 = (to_dev(x, off) for x in (p, m, v, np.zeros(n, np.uint16)))
    assert _takes_the_order(dg, mode, True, n, -off % 256) == taken
    dd.aggregate_adam(dg, dp, dm, dv, d16, lr=HP["lr"], beta1=HP["beta1"], beta2=HP["beta2"],
                      eps=HP["eps"], weight_decay=HP["wd"], step=2, mode=mode, frac_bits=24)
    torch().cuda.synchronize()
    want = oracle.fused(gs, p, m, v, mode=oracle.AGG_FIXED if mode == "fixed" else oracle.AGG_FP32,
                        frac_bits=24, t=2, **HP)
    assert_parity({"p": to_host(dp), "m": to_host(dm), "v": to_host(dv), "p16": to_host(d16)}, want,
                  f"W={W} {mode} n={n} off={off} apart={apart}")


@pytest.mark.parametrize("W,mode,n,apart,taken", [
    (16, "fp32", 2 * BASE + 1, 34, 1), (16, "fixed", 2 * BASE + 256, 34, 1),
    (24, "fp32", 2 * BASE + SET, 34, 1), (24, "fixed", 2 * BASE + 2051, 34, 1),
    (16, "fp32", 2 * BASE + 1, 64, 0)])
def test_aggregate(W, mode, n, apart, taken):
    import paper_2409_00918_amd as dd
    gs = synth.host_grads(900 + W, 1, W, n, 1e-4, gdtype="bf16")
    dg = _contributions(gs, 0, apart * MIB)
    out = to_dev(np.zeros(n, np.float32))
    assert _takes_the_order(dg, mode, False, n, 0) == taken
    dd.aggregate(dg, mode=mode, frac_bits=24, agg_out_f32=out)
    torch().cuda.synchronize()
    want = oracle.aggregate_f32(gs) if mode == "fp32" else oracle.aggregate_fixed(gs, 24)[1]
    assert np.array_equal(to_host(out).view(np.uint32), want.view(np.uint32))
