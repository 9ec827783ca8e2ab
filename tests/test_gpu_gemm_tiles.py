"""Tile dispatch of the 16-bit hidden-layer GEMMs: the tile of a launch follows
from its streams, depth and number of points, and every tile multiplies in the
same order, so a point's jets do not depend on how many points share its call.
Each case evaluates a few points alone (32-point tiles), compares them with
the oracle, and again at the front and the back of a call large enough for the
large tiles, whose last tile is ragged: bit for bit the same.  (Four streams,
five at 256 columns and seven at 128 take the 32-point tile at every size:
there the large call is that tile in more blocks.)"""
import numpy as np
import pytest

import oracle
from paper_1910_13444_amd import pigan
from paper_1910_13444_amd.inputs import glorot_mlp
from _parity import TOL, check, rel, to_dev

pytestmark = pytest.mark.gpu

# (d, order, W): streams 1 (order 0), 2, 3 (d = 1), 3, 5 (d = 2), 4, 7 (d = 3);
# 128 columns only for the seven streams that the resident kernel does not take
CASES = [(2, 0, 256), (2, 0, 512), (1, 1, 256), (1, 2, 512), (2, 1, 256), (2, 1, 512), (2, 2, 256), (2, 2, 512),
         (3, 1, 512), (3, 2, 128), (3, 2, 256)]


@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
@pytest.mark.parametrize("d,order,W", CASES)
def test_gen_forward_tiles(d, order, W, dtype):
    import torch
    print(f"gen_forward tiles d={d} order={order} W={W} {dtype}", flush=True)
    rng = np.random.default_rng(100 * d + 10 * order + W)
    n_z, L, few = 5, 3, 45
    # points of the large call: two rounds of the largest tile (256 points) on
    # 256 compute units at W = 256, less for wider layers, plus a remainder
    many = 256 * 512 * 256 // max(W, 256) + 37 if order == 0 else 128 * 512 * 256 // max(W, 256) + 37
    shape = (d + n_z, L, W)
    p = glorot_mlp(rng, *shape)[None]
    z = rng.standard_normal((1, 1, n_z)).astype(np.float32)
    x = rng.random((1, 1, many, d)).astype(np.float32)
    x[0, 0, -few:] = x[0, 0, :few]
    small = pigan.gen_forward(to_dev(p), shape, d, to_dev(z), to_dev(x[:, :, :few]), order, dtype=dtype)
    large = pigan.gen_forward(to_dev(p), shape, d, to_dev(z), to_dev(x), order, dtype=dtype)
    torch.cuda.synchronize()
    if dtype == "fp16":
        # one sample's field is nearly constant, so w_out . h cancels: stored
        # rounding of 2^-9 per value (bf16) shows as up to 0.04 of a component's
        # norm here, 2^-12 (fp16) as an eighth of that, 0.005; bf16 is covered
        # by the comparisons below and by the parity tests over many samples
        ref = oracle.gen_jets(p[0], shape, d, z[0], x[0, :, :few], order)
        got = small.cpu().numpy()[0]
        check({f"c{k}": rel(got[k], ref[k]) for k in range(ref.shape[0])}, TOL[dtype], f"d={d} order={order} W={W}")
    assert torch.equal(small[0, :, 0], large[0, :, 0, :few])
    assert torch.equal(small[0, :, 0], large[0, :, 0, -few:])


# fp32-stored products with few output tiles run as short launches (one wave per
# tile in split products; in fp64 the contraction is shared among a
# block's waves, four, eight from K = 1024), above that they are tiled: single
# and ragged rows, contractions shorter than a block's waves and longer than
# its prefetch, both sides of the dispatch (2000 x 1024 and 9000 x 128 are tiled
# both ways)
@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("G,B,n_in,L,W", [(1, 1, 3, 2, 32), (2, 33, 7, 3, 32), (1, 31, 1040, 2, 64), (1, 65, 40, 2, 1024),
                                          (3, 17, 100, 2, 256), (1, 300, 2016, 2, 1024), (1, 9000, 128, 2, 128), (1, 2000, 64, 2, 1024)])
def test_disc_forward_short(dtype, G, B, n_in, L, W):
    import torch
    print(f"disc_forward short G={G} B={B} n_in={n_in} L={L} W={W} {dtype}", flush=True)
    rng = np.random.default_rng(B + n_in)
    shape = (n_in, L, W)
    p = np.stack([glorot_mlp(rng, *shape) for _ in range(G)])
    p[:, -1] = 0.3
    snap = rng.standard_normal((G, B, n_in)).astype(np.float32)
    sc = pigan.disc_forward(to_dev(p), shape, to_dev(snap), dtype=dtype)
    torch.cuda.synchronize()
    sc = sc.cpu().numpy()
    for g in range(G):
        ref = oracle.mlp_forward(p[g], shape, snap[g])
        check({f"g{g}": rel(sc[g], ref)}, TOL[dtype], f"disc_forward short {dtype}")


# latent part of the first layer: blocks of 32 columns x 8 samples, 64 terms at
# a time
@pytest.mark.parametrize("S,n_z,W", [(1, 1, 32), (9, 63, 64), (7, 64, 128), (8, 65, 32), (17, 130, 256)])
def test_gen_forward_latent_sum(S, n_z, W):
    import torch
    print(f"gen_forward latent S={S} n_z={n_z} W={W}", flush=True)
    rng = np.random.default_rng(S + n_z)
    shape = (1 + n_z, 2, W)
    p = glorot_mlp(rng, *shape)[None]
    z = rng.standard_normal((1, S, n_z)).astype(np.float32)
    x = rng.random((1, S, 3, 1)).astype(np.float32)
    got = pigan.gen_forward(to_dev(p), shape, 1, to_dev(z), to_dev(x), 1, dtype="fp32")
    torch.cuda.synchronize()
    got = got.cpu().numpy()[0]
    ref = oracle.gen_jets(p[0], shape, 1, z[0], x[0], 1)
    check({f"c{k}": rel(got[k], ref[k]) for k in range(ref.shape[0])}, TOL["fp32"], f"latent S={S} n_z={n_z} W={W}")


# two-term weights: all high terms are added in the order of k, then all low
# ones.  Every row of the second layer holds two weights whose high terms cancel
# against two of the last slice (of 64 inputs with equal values), and a low term of
# 2^-12 that alone is left.  2^-12 h beside a sum of 32832 h is below half a
# unit of the last place of fp32 (2^-9 h): added before the cancellation it is
# lost, and the field is zero.  After it every sum is exact (32832 h takes 21
# bits), and the field is that of the 16-bit h, a few 2^-9 from the oracle's.
@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
@pytest.mark.parametrize("d,order,W", [c for c in CASES if c[0] != 3 or c[1] == 2] + [(1, 0, 1024)])
def test_two_term_sum_order(d, order, W, dtype):
    import torch
    print(f"two-term sum order d={d} order={order} W={W} {dtype}", flush=True)
    n_z, L, pts = 2, 2, 40
    shape = (d + n_z, L, W)
    W1 = np.zeros((W, d + n_z))
    W1[:, :d] = [0.5, 0.25, 0.75][:d]
    W2 = np.zeros((W, W))
    W2[:, 0], W2[:, 1], W2[:, W - 64], W2[:, W - 63] = 32768.0, 64.0 + 2.0 ** -12, -32768.0, -64.0
    p = np.concatenate([W1.ravel(), np.full(W, 0.25), W2.ravel(), np.zeros(W), np.full(W, 1.0 / W), [0.0]])[None]
    z = np.ones((1, 1, n_z))
    x = np.random.default_rng(W).random((1, 1, pts, d))
    got = pigan.gen_forward(to_dev(p), shape, d, to_dev(z), to_dev(x), order, dtype=dtype)
    torch.cuda.synchronize()
    got = got.cpu().numpy()[0]
    ref = oracle.gen_jets(p[0], shape, d, z[0], x[0], order)
    check({f"c{k}": rel(got[k], ref[k]) for k in range(ref.shape[0])}, TOL[dtype], f"d={d} order={order} W={W}")


# output layer of a 16-bit row: eight lanes sum pieces of eight columns in turn
# (fp32), then meet pairwise, whether a pass of its own reads the row or, for 128
# columns, the block that formed it.  Saturated units (+-1) make every product
# exact, so the sum follows from its order alone: the same bits.
@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
@pytest.mark.parametrize("d,order,W,pts", [(3, 2, 128, 1), (3, 2, 128, 77), (2, 0, 256, 77), (1, 1, 512, 33)])
def test_output_layer_sum_order(d, order, W, pts, dtype):
    import torch
    print(f"output layer sum order d={d} order={order} W={W} points={pts} {dtype}", flush=True)
    rng = np.random.default_rng(W + pts)
    n_z, L = 2, 2
    shape = (d + n_z, L, W)
    h = rng.choice([-1.0, 1.0], W).astype(np.float32)
    w_out, b_out = rng.standard_normal(W).astype(np.float32), np.float32(0.3)
    p = np.concatenate([np.zeros(W * (d + n_z) + W + W * W), 40.0 * h, w_out, [b_out]])[None]
    got = pigan.gen_forward(to_dev(p), shape, d, to_dev(np.ones((1, 1, n_z))), to_dev(rng.random((1, 1, pts, d))), order,
                            dtype=dtype)
    torch.cuda.synchronize()
    lane = np.zeros(8, np.float32)
    for c in range(0, W, 64):
        for e in range(8):
            for q in range(8):
                lane[e] += w_out[c + 8 * e + q] * h[c + 8 * e + q]
    for s in (1, 2, 4):
        lane = lane + lane[np.arange(8) ^ s]
    got = got.cpu().numpy()[0].reshape(-1, pts)
    assert (got[0] == lane[0] + b_out).all(), (got[0][0], lane[0] + b_out)
    assert (got[1:] == 0).all()


# Split products (16-bit modes) of the critic: every kernel that forms them adds
# in the same order, so a snapshot's score does not depend on how many share its
# call.  Forty snapshots alone (short launches) against the oracle, and again at
# the front and the ragged back of a batch that each tiled kernel takes (32,
# 64, 128 and 1024 columns; 128 above 196,608 rows; 256 columns and more from
# 16,384 rows, contractions of both sides of 512).  The bound pins the low
# pieces: two bf16 pieces carry 16 bits (2^-17 per operand, 2^-16 per product),
# and the sums of a score cancel by about a factor of six; without a low piece
# the error is 2^-9.
@pytest.mark.parametrize("n_in,L,W,B", [(40, 2, 32, 17001), (40, 2, 64, 17001), (100, 2, 128, 17001),
                                        (96, 2, 128, 196673), (100, 2, 256, 16421), (64, 2, 512, 16421),
                                        (2016, 2, 1024, 2009)])
@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
def test_disc_forward_split_tiles(dtype, n_in, L, W, B):
    import torch
    print(f"disc_forward split tiles n_in={n_in} W={W} B={B} {dtype}", flush=True)
    rng = np.random.default_rng(n_in + W)
    few, shape = 40, (n_in, L, W)
    p = glorot_mlp(rng, *shape)[None]
    snap = rng.standard_normal((1, B, n_in)).astype(np.float32)
    snap[0, -few:] = snap[0, :few]
    small = pigan.disc_forward(to_dev(p), shape, to_dev(snap[:, :few]), dtype=dtype)
    large = pigan.disc_forward(to_dev(p), shape, to_dev(snap), dtype=dtype)
    torch.cuda.synchronize()
    ref = oracle.mlp_forward(p[0], shape, snap[0, :few])
    check({"score": rel(small.cpu().numpy()[0], ref)}, 1e-4, f"split products {dtype}")
    assert torch.equal(small[0], large[0, :few])
    assert torch.equal(small[0], large[0, -few:])
