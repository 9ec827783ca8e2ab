"""Reverse passes of the wide 16-bit generators in one, two and three
dimensions (2, 3, 4, 5 and 7 streams; the first layer's derivative
pre-activations are one row per stream), and the tiles that only large launches
take: parity with the oracle, and the whole step against the same step in
chunks of one sample, whose launches take the small tiles."""
import numpy as np
import pytest

import oracle
from paper_1910_13444_amd import configs
from paper_1910_13444_amd.inputs import make_inputs
from _parity import check, run_step_gpu, run_trunk_gpu, step_errors, trunk_errors

pytestmark = pytest.mark.gpu

BASE = configs.C2.with_(n_z=6, L=3, S=6, P=50, n_sY=12, n_sU=13, L_D=2, W_D=64, B_r=6)


@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
@pytest.mark.parametrize("d,W", [(1, 128), (1, 256), (1, 512), (2, 768), (3, 128), (3, 256), (3, 512)])
def test_step_streams(d, W, dtype):
    print(f"step d={d} W={W} {dtype}", flush=True)
    wl = BASE.with_(d=d, W=W, dtype=dtype)
    inp = make_inputs(wl, f_array=True)
    real = oracle.real_snapshots(wl, inp)
    out = run_step_gpu(wl, inp, real)
    assert out["nonfinite"] == 0
    # (a stored bf16 value is off by up to 2^-9 = 2e-3, and gradients average
    # over rows; the critic's by the cancellation of its 2^-16 split products)
    check(step_errors(wl, out, oracle.train_step(wl, inp, real)), 3e-3, f"step d={d} W={W} {dtype}")


# Launches of at least two rounds of large tiles on 256 compute units (ragged):
# reverse two and three streams at 768, forward and reverse three and forward
# five at 512, the trunk's residual rows beside five streams at 512, and the
# sensor rows' split products at 256 columns (16,384 rows and more).  A row's
# cotangents are the same bits in both runs; the sums over rows are split
# differently: fp32 partial sums of at most a few dozen matrix-core
# accumulations each (2^-24 per addition, 2e-6 in all), fp64 between them, on
# terms that cancel by a small factor: 1e-5.
@pytest.mark.parametrize("kind,d,W,S,P,n_s", [("pair", 1, 768, 8, 1400, 12), ("pair", 2, 512, 8, 2100, 12),
                                             ("trunk", 2, 512, 8, 2100, 12), ("pair", 2, 256, 4, 64, 4100)])
def test_step_large_tiles(kind, d, W, S, P, n_s):
    print(f"large tiles {kind} d={d} W={W} S={S} P={P} sensors={n_s}", flush=True)
    wl = BASE.with_(d=d, W=W, S=S, P=P, n_sY=n_s, n_sU=n_s + 1, B_r=S, dtype="bf16", arch=kind)
    inp = make_inputs(wl, f_array=True)
    if kind == "trunk":
        real, run, errors, ref = oracle.real_snapshots_trunk(wl, inp), run_trunk_gpu, trunk_errors, oracle.train_step_trunk
    else:
        real, run, errors, ref = oracle.real_snapshots(wl, inp), run_step_gpu, step_errors, oracle.train_step
    out, parts = run(wl, inp, real), run(wl, inp, real, chunk_S=1)
    assert out["nonfinite"] == 0 and parts["nonfinite"] == 0
    check(errors(wl, out, parts), 1e-5, "whole against chunks")
    check(errors(wl, out, ref(wl, inp, real)), 3e-3, "whole against the oracle")


# The timing records' byte model of five streams at 256 columns: a reverse pass
# into the first layer reads its value rows and one row per further stream; the
# fused last layer has a name of its own, writes no activations, and its sums of
# 128 columns cross twice.
def test_profile_bytes_of_seeds_and_fused_output():
    from paper_1910_13444_amd import pigan
    print("profile bytes d=2 W=256", flush=True)
    wl = BASE.with_(d=2, W=256, dtype="bf16")
    inp = make_inputs(wl, f_array=True)
    real = oracle.real_snapshots(wl, inp)
    pigan.profile_enable(True)
    try:
        run_step_gpu(wl, inp, real)
        stats = {s["name"]: s for s in pigan.profile_read()}
    finally:
        pigan.profile_enable(False)
    n, W, C = wl.S * wl.P, wl.W, 5
    M, weights = C * n, W * W * 2
    bwd = [M * W * 2 + weights + M * W * 2 + rows * W * 2 for rows in (M, n + C - 1)]   # X, weights, out, saved rows
    assert stats["gemm_bwd_c5_k256_n256"]["launches"] == 2
    assert stats["gemm_bwd_c5_k256_n256"]["bytes"] == sum(bwd)
    assert stats["gemm_fwd_c5_k256_n256_w2"]["bytes"] == M * W * 2 + 2 * weights + 2 * M * W * 2
    out = stats["gemm_fwd_c5_k256_n256_w2_out"]
    assert out["launches"] == 1
    assert out["bytes"] == M * W * 2 + 2 * weights + M * W * 2 + M * 4 + 2 * M * (W // 128) * 4
