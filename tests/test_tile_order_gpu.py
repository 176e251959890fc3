"""Launches that give each XCD two neighbouring tiles (many bf16 contributions,
more than 16 rounds of resident waves): every element against the oracle, at
lengths that end inside, at and just past the last whole set of 16 blocks, with
and without a head, in every kernel that may take the order."""
import numpy as np
import pytest

import oracle
import synth
from gpu_common import assert_parity, run_fused_case, to_dev, to_host, torch

pytestmark = pytest.mark.gpu

SET = 16 * 256                       # elements of 16 tiles
BASE = 2048 * SET                    # 8.4M: past 16 rounds of 8 waves on 256 CUs


@pytest.mark.parametrize("W,mode,n,off", [
    (12, "fp32", BASE, 0), (16, "fp32", BASE + 5, 0), (16, "fixed", BASE + SET - 1, 37),
    (20, "fp32", BASE + 256 * 15 + 3, 2)])
def test_fused(W, mode, n, off):
    got, want = run_fused_case(W, "bf16", mode, n, offsets=(off, off), want_agg=False)
    assert_parity(got, want, f"W={W} {mode} n={n} off={off}")


@pytest.mark.parametrize("W,mode,n", [(16, "fp32", 2 * BASE + 1), (24, "fixed", BASE + 2051)])
def test_aggregate(W, mode, n):
    import paper_2409_00918_amd as dd
    gs = synth.host_grads(900 + W, 1, W, n, 1e-4, gdtype="bf16")
    out = to_dev(np.zeros(n, np.float32))
    dd.aggregate([to_dev(g) for g in gs], mode=mode, frac_bits=24, agg_out_f32=out)
    torch().cuda.synchronize()
    want = oracle.aggregate_f32(gs) if mode == "fp32" else oracle.aggregate_fixed(gs, 24)[1]
    assert np.array_equal(to_host(out).view(np.uint32), want.view(np.uint32))
