"""GPU parity of the 5x5x5 convolution (Sec. III-A: 3^3 and 5^3 filters; two halo planes) against the CPU oracle:
all three passes, unsharded and on depth shards with two halo planes, fp32 and bf16, extents that span several
8 x 32 tiles with ragged tails, channel counts on both sides of the 16-channel blocks, canaries on what must not
be written, error paths that must not launch."""
import numpy as np
import pytest

import oracle as orc
import synth
from helpers import TOL, cut, dev_like, from_dev, quantize, close, rel_l2, slab_pair, to_dev

pytestmark = pytest.mark.gpu
SEED = synth.BASE_SEED

# (N, Cin, Cout, D, H, W)
SHAPES = [
    (1, 1, 1, 1, 1, 1),          # a single voxel: only the centre tap is inside the volume
    (2, 3, 5, 4, 11, 37),        # ragged tiles in both directions
    (1, 16, 32, 6, 16, 64),      # two channel blocks, whole tiles
    (1, 17, 18, 3, 9, 33),       # one channel past a block on both sides
    (1, 4, 16, 5, 20, 70),
    (1, 33, 34, 2, 35, 136),     # two tiles in H and in W for every kernel form, one channel past a 32-block
]


def _weights(cin, cout, dtype, stream):
    b = np.sqrt(3.0 / (125 * cin))
    w = quantize(synth.flat("uniform", SEED, stream, (cout, cin, 5, 5, 5), -b, b), dtype)
    bias = synth.round_f32(synth.flat("uniform", SEED, stream + 1, (cout,), -0.1, 0.1)).astype(np.float64)
    return w, bias


def _tol_w(dtype):
    return 1e-5 if dtype == "f32" else 2e-4


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", SHAPES)
def test_k5_three_passes_unsharded(shape, dtype):
    import torch
    import paper_2007_12856_amd as h3d
    N, Ci, Co, D, H, W = shape
    alpha = 0.01
    print("k5 unsharded", shape, dtype, flush=True)
    w, bias = _weights(Ci, Co, dtype, 510)
    wd, bd = to_dev(w, dtype), to_dev(bias, "f32")
    xo, xg = slab_pair(synth.flat("uniform", SEED, 501, (N, Ci, D, H, W)), dtype)
    zo = orc.convk_fwd(xo, w, bias, orc.ACT_LEAKY, alpha)
    zg = h3d.conv3d_k5_fwd(xg, wd, bd, dev_like(zo, dtype), h3d.ACT_LEAKY, alpha)
    close(from_dev(zg.t), zo.a, TOL[dtype])
    zq_o, zq_g = slab_pair(zo.a, dtype)
    dzo, dzg = slab_pair(synth.flat("uniform", SEED, 502, zo.a.shape), dtype)
    dxo = orc.convk_bwd_data(dzo, zq_o, w, orc.ACT_LEAKY, alpha)
    dxg = h3d.conv3d_k5_bwd_data(dzg, zq_g, wd, dev_like(dxo, dtype), h3d.ACT_LEAKY, alpha)
    close(from_dev(dxg.t), dxo.a, TOL[dtype])
    dwo, dbo = orc.convk_bwd_filter(5, xo, dzo, zq_o, orc.ACT_LEAKY, alpha)
    dw = torch.full((Co, Ci, 5, 5, 5), 777.0, device="cuda")
    db = torch.full((Co,), 777.0, device="cuda")
    h3d.conv3d_k5_bwd_filter(xg, dzg, zq_g, dw, db, h3d.ACT_LEAKY, alpha)
    close(from_dev(dw), dwo, _tol_w(dtype))
    close(from_dev(db), dbo, _tol_w(dtype))
    dw2, db2 = torch.empty_like(dw), torch.empty_like(db)
    h3d.conv3d_k5_bwd_filter(xg, dzg, zq_g, dw2, db2, h3d.ACT_LEAKY, alpha)
    assert torch.equal(dw, dw2) and torch.equal(db, db2)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("act", [orc.ACT_NONE, orc.ACT_RELU])
def test_k5_no_bias_other_activations(dtype, act):
    import torch
    import paper_2007_12856_amd as h3d
    N, Ci, Co, D, H, W = 1, 8, 16, 4, 6, 20
    print("k5 act", act, dtype, flush=True)
    w, _ = _weights(Ci, Co, dtype, 520)
    wd = to_dev(w, dtype)
    xo, xg = slab_pair(synth.flat("normal", SEED, 503, (N, Ci, D, H, W)), dtype)
    zo = orc.convk_fwd(xo, w, None, act)
    zg = h3d.conv3d_k5_fwd(xg, wd, None, dev_like(zo, dtype), act, 0.0)
    close(from_dev(zg.t), zo.a, TOL[dtype])
    zq_o, zq_g = slab_pair(zo.a, dtype)
    dzo, dzg = slab_pair(synth.flat("normal", SEED, 504, zo.a.shape), dtype)
    dxo = orc.convk_bwd_data(dzo, zq_o, w, act)
    dxg = h3d.conv3d_k5_bwd_data(dzg, zq_g, wd, dev_like(dxo, dtype), act, 0.0)
    close(from_dev(dxg.t), dxo.a, TOL[dtype])
    dwo, _ = orc.convk_bwd_filter(5, xo, dzo, zq_o, act)
    dw = torch.full((Co, Ci, 5, 5, 5), 777.0, device="cuda")
    h3d.conv3d_k5_bwd_filter(xg, dzg, zq_g, dw, None, act, 0.0)
    close(from_dev(dw), dwo, _tol_w(dtype))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shard", [0, 1, 3])
def test_k5_on_depth_shards(shard, dtype):
    """4-way depth partition of a 1 x 6 x 12 x 10 x 40 sample, two halo planes per side (zeros outside the volume):
    each shard's result is the oracle's on the same shard; outputs carry halos that must stay untouched."""
    import torch
    import paper_2007_12856_amd as h3d
    N, Ci, Co, Dg, H, W = 1, 6, 20, 12, 10, 40
    d, alpha = Dg // 4, 0.01
    off = shard * d
    print("k5 shard", shard, dtype, flush=True)
    w, bias = _weights(Ci, Co, dtype, 530)
    wd, bd = to_dev(w, dtype), to_dev(bias, "f32")
    xa = cut("uniform", SEED, 505, (N, Ci, Dg, H, W), off, d, (2, 2))
    xo, xg = slab_pair(xa, dtype, (2, 2), off, Dg)
    zo = orc.convk_fwd(xo, w, bias, orc.ACT_LEAKY, alpha)
    td = torch.float32 if dtype == "f32" else torch.bfloat16
    zg = h3d.Slab(torch.full((N, Co, d + 3, H, W), 12345.0, device="cuda", dtype=td), 1, 2, off, Dg)
    h3d.conv3d_k5_fwd(xg, wd, bd, zg, h3d.ACT_LEAKY, alpha)
    got = from_dev(zg.t)
    close(got[:, :, 1:-2], zo.a, TOL[dtype])
    canary = got[0, 0, 0, 0, 0]
    assert canary == 12345.0 or dtype == "bf16"
    assert np.all(got[:, :, 0] == canary) and np.all(got[:, :, -2:] == canary)
    # backward: dz and the saved z with two halo planes, cut from seeded full tensors
    full_z = (N, Co, Dg, H, W)
    dzo, dzg = slab_pair(cut("uniform", SEED, 506, full_z, off, d, (2, 2)), dtype, (2, 2), off, Dg)
    zso, zsg = slab_pair(cut("normal", SEED, 507, full_z, off, d, (2, 2)), dtype, (2, 2), off, Dg)
    dxo = orc.convk_bwd_data(dzo, zso, w, orc.ACT_LEAKY, alpha)
    dxg = h3d.conv3d_k5_bwd_data(dzg, zsg, wd, dev_like(dxo, dtype), h3d.ACT_LEAKY, alpha)
    close(from_dev(dxg.t), dxo.a, TOL[dtype])
    dwo, dbo = orc.convk_bwd_filter(5, xo, dzo, zso, orc.ACT_LEAKY, alpha)
    dw = torch.full((Co, Ci, 5, 5, 5), 777.0, device="cuda")
    db = torch.full((Co,), 777.0, device="cuda")
    h3d.conv3d_k5_bwd_filter(xg, dzg, zsg, dw, db, h3d.ACT_LEAKY, alpha)
    close(from_dev(dw), dwo, _tol_w(dtype))
    close(from_dev(db), dbo, _tol_w(dtype))


def test_k5_larger_volume_sampled_against_the_oracle_definition():
    """1 x 16 x 32^3 -> 32 channels in bf16: too slow for the whole oracle pass in a test; sampled output voxels are
    computed one by one from the definition (fp64 sum over the padded window)."""
    import paper_2007_12856_amd as h3d
    N, Ci, Co, D = 1, 16, 32, 32
    print("k5 sampled 32^3", flush=True)
    w, bias = _weights(Ci, Co, "bf16", 540)
    x = quantize(synth.flat("uniform", SEED, 508, (N, Ci, D, D, D)), "bf16")
    _, xg = slab_pair(x, "bf16")
    zg = h3d.conv3d_k5_fwd(xg, to_dev(w, "bf16"), to_dev(bias, "f32"), dev_like(orc.Slab(np.zeros((N, Co, D, D, D))), "bf16"),
                           h3d.ACT_NONE, 0.0)
    got = from_dev(zg.t)
    xp = np.zeros((Ci, D + 4, D + 4, D + 4))
    xp[:, 2:-2, 2:-2, 2:-2] = x[0]
    rng = np.random.default_rng(SEED + 509)
    pts = [(0, 0, 0, 0), (Co - 1, D - 1, D - 1, D - 1), (5, 0, D - 1, 17), (17, 31, 0, 1)]
    pts += [tuple(int(v) for v in (rng.integers(Co), rng.integers(D), rng.integers(D), rng.integers(D))) for _ in range(200)]
    ref = np.array([bias[co] + np.sum(w[co] * xp[:, p:p + 5, h:h + 5, v:v + 5]) for co, p, h, v in pts])
    val = np.array([got[0, co, p, h, v] for co, p, h, v in pts])
    close(val, ref, TOL["bf16"])


def test_k5_backward_at_the_bench_shape_sampled_against_the_definition():
    """The launch configuration bench.py times (32 -> 32 channels, 128 x 128 planes, an interior shard with two halo
    planes per side, leaky-ReLU mask), on 8 interior planes: sampled dx voxels and dw entries are computed one by one
    from the definition in fp64 (g = dz * act'(z) taken from the unrounded product, as the oracle does)."""
    import torch
    import paper_2007_12856_amd as h3d
    N, C, d, H, W, off, Dg, alpha = 1, 32, 8, 128, 128, 32, 128, 0.01
    print("k5 sampled backward at the bench shape", flush=True)
    w, _ = _weights(C, C, "bf16", 550)
    full = (N, C, Dg, H, W)
    xa = quantize(cut("uniform", SEED, 551, full, off, d, (2, 2)), "bf16")
    dza = quantize(cut("uniform", SEED, 552, full, off, d, (2, 2)), "bf16")
    za = quantize(cut("normal", SEED, 553, full, off, d, (2, 2)), "bf16")
    _, xg = slab_pair(xa, "bf16", (2, 2), off, Dg)
    _, dzg = slab_pair(dza, "bf16", (2, 2), off, Dg)
    _, zg = slab_pair(za, "bf16", (2, 2), off, Dg)
    g = dza * np.where(za > 0, 1.0, alpha)                       # [1, C, d+4, H, W], stored planes -2 .. d+1
    gp = np.zeros((C, d + 4, H + 4, W + 4)); gp[:, :, 2:-2, 2:-2] = g[0]
    xp = np.zeros((C, d + 4, H + 4, W + 4)); xp[:, :, 2:-2, 2:-2] = xa[0]
    rng = np.random.default_rng(SEED + 554)
    # backward-data: dx[ci,q,h,v] = sum_{co,k} w[co,ci,k] g~[co,q-k+2]  (window of g reversed against the filter)
    dxg = h3d.conv3d_k5_bwd_data(dzg, zg, to_dev(w, "bf16"), h3d.Slab(torch.full((N, C, d, H, W), 7.0, device="cuda", dtype=torch.bfloat16),
                                                                   0, 0, off, Dg), h3d.ACT_LEAKY, alpha)
    got = from_dev(dxg.t)
    pts = [(0, 0, 0, 0), (C - 1, d - 1, H - 1, W - 1), (3, 0, H - 1, 17), (17, d - 1, 0, 1)]
    pts += [tuple(int(v) for v in (rng.integers(C), rng.integers(d), rng.integers(H), rng.integers(W))) for _ in range(150)]
    ref = np.array([np.sum(w[:, ci, ::-1, ::-1, ::-1] * gp[:, q:q + 5, h:h + 5, v:v + 5]) for ci, q, h, v in pts])
    val = np.array([got[0, ci, q, h, v] for ci, q, h, v in pts])
    close(val, ref, TOL["bf16"])
    # backward-filter: dw[co,ci,k] = sum over the interior of g[co,p] x~[ci,p+k-2]; db[co] = sum g
    dw = torch.full((C, C, 5, 5, 5), 777.0, device="cuda")
    db = torch.full((C,), 777.0, device="cuda")
    h3d.conv3d_k5_bwd_filter(xg, dzg, zg, dw, db, h3d.ACT_LEAKY, alpha)
    gi = g[0][:, 2:-2]                                            # interior planes
    ent = [(0, 0, 0, 0, 0), (C - 1, C - 1, 4, 4, 4), (5, 9, 2, 2, 2), (31, 0, 0, 4, 1)]
    ent += [tuple(int(v) for v in (rng.integers(C), rng.integers(C), rng.integers(5), rng.integers(5), rng.integers(5))) for _ in range(60)]
    ref = np.array([np.sum(gi[co] * xp[ci, kd:kd + d, kh:kh + H, kw:kw + W]) for co, ci, kd, kh, kw in ent])
    gw = from_dev(dw)
    val = np.array([gw[e] for e in ent])
    close(val, ref, _tol_w("bf16"))
    close(from_dev(db), gi.sum(axis=(1, 2, 3)), _tol_w("bf16"))


def test_k5_errors_do_not_launch():
    import ctypes
    import torch
    import paper_2007_12856_amd as h3d
    w = torch.zeros((3, 2, 5, 5, 5), device="cuda")
    x1 = h3d.Slab(torch.zeros((1, 2, 4 + 1 + 2, 4, 4), device="cuda"), 1, 2, 4, 16)     # one lower halo plane only
    z = h3d.Slab(torch.zeros((1, 3, 4, 4, 4), device="cuda"), 0, 0, 4, 16)
    with pytest.raises(h3d.H3DError) as e:
        h3d.conv3d_k5_fwd(x1, w, None, z)
    assert e.value.status == -4
    dx = h3d.Slab(torch.zeros((1, 2, 4, 4, 4), device="cuda"), 0, 0, 4, 16)
    with pytest.raises(h3d.H3DError) as e:                                              # dz without halo planes
        h3d.conv3d_k5_bwd_data(z, None, w, dx)
    assert e.value.status == -4
    xs = h3d.Slab(torch.zeros((1, 2, 4, 4, 4), device="cuda"))
    with pytest.raises(h3d.H3DError) as e:                                              # extents differ
        h3d.conv3d_k5_fwd(xs, w, None, h3d.Slab(torch.zeros((1, 3, 4, 4, 5), device="cuda")))
    assert e.value.status == -1
    zs = h3d.Slab(torch.zeros((1, 3, 4, 4, 4), device="cuda"))
    st = h3d.lib().h3d_conv3d_k5_fwd(h3d.handle(), ctypes.byref(xs.desc()), ctypes.c_void_p(w.data_ptr()), None,
                                     ctypes.byref(zs.desc()), 0, 0.0, None, 0, None)
    assert st == -3
    # a shard next to the boundary needs only the planes that exist: one plane below the interior here
    xb = h3d.Slab(torch.zeros((1, 2, 1 + 4 + 2, 4, 4), device="cuda"), 1, 2, 1, 16)
    h3d.conv3d_k5_fwd(xb, w, None, h3d.Slab(torch.zeros((1, 3, 4, 4, 4), device="cuda"), 0, 0, 1, 16))


def test_k5_empty_shard():
    import torch
    import paper_2007_12856_amd as h3d
    x = h3d.Slab(torch.zeros((1, 2, 0, 4, 4), device="cuda"), 0, 0, 0, 8)
    z = h3d.Slab(torch.zeros((1, 3, 0, 4, 4), device="cuda"), 0, 0, 0, 8)
    w = torch.zeros((3, 2, 5, 5, 5), device="cuda")
    h3d.conv3d_k5_fwd(x, w, None, z)
    dw = torch.full((3, 2, 5, 5, 5), 5.0, device="cuda")
    db = torch.full((3,), 5.0, device="cuda")
    h3d.conv3d_k5_bwd_filter(x, z, None, dw, db)
    torch.cuda.synchronize()
    assert float(dw.abs().max()) == 0.0 and float(db.abs().max()) == 0.0


@pytest.mark.parametrize("act", [orc.ACT_NONE, orc.ACT_LEAKY])
@pytest.mark.parametrize("shape,shift", [
    ((1, 3, 5, 64, 33, 33), 0),      # enough tiles for the 32-row form of the convolution kernel, one row and one column past a tile
    ((2, 20, 40, 6, 3, 72), 0),      # columns of three rows: a wavefront group's run spans many, the second segment is 8 wide
    ((1, 9, 33, 3, 40, 24), 1),      # whole 16-byte rows at an odd address
    ((1, 33, 9, 3, 19, 45), 3),      # ragged rows at an odd address
    ((1, 17, 33, 2, 2, 3), 0),       # a block of one channel with planes shorter than a 16-byte load
    ((1, 17, 33, 1, 2, 5), 1),       # and one that a load just fits
    ((2, 33, 17, 1, 1, 3), 1),       # a last chunk of one channel of three elements: its loads begin in the channel before
    ((1, 2, 5, 1, 1, 4), 2),         # a sample of one load
    ((1, 1, 7, 1, 1, 7), 0),         # and of less
])
def test_k5_bf16_kernel_edges(shape, shift, act):
    import torch
    import paper_2007_12856_amd as h3d
    N, Ci, Co, D, H, W = shape
    print("k5 edges", shape, shift, act, flush=True)

    def moved(s):      # the same values `shift` elements into a larger allocation
        flat = torch.empty(s.t.numel() + 16, dtype=s.t.dtype, device="cuda")[shift:shift + s.t.numel()]
        return h3d.Slab(flat.view(s.t.shape).copy_(s.t), s.halo_lo, s.halo_hi, s.d_offset, s.d_global)

    w, bias = _weights(Ci, Co, "bf16", 540)
    wd, bd = to_dev(w, "bf16"), to_dev(bias, "f32")
    xo, xg = slab_pair(synth.flat("normal", SEED, 541, (N, Ci, D, H, W)), "bf16")
    zo = orc.convk_fwd(xo, w, bias, act, 0.01)
    zg = h3d.conv3d_k5_fwd(moved(xg), wd, bd, moved(dev_like(zo, "bf16")), act, 0.01)
    assert h3d.h3d_last_kernel().startswith("k5_conv_mfma_kernel") == (Ci * D * H * W >= 8)      # (no halo here)
    close(from_dev(zg.t), zo.a, TOL["bf16"])
    so, sg = slab_pair(synth.flat("normal", SEED, 542, zo.a.shape), "bf16")
    go, gg = slab_pair(synth.flat("normal", SEED, 543, zo.a.shape), "bf16")
    dxo = orc.convk_bwd_data(go, so, w, act, 0.01)
    dxg = h3d.conv3d_k5_bwd_data(moved(gg), moved(sg), wd, moved(dev_like(dxo, "bf16")), act, 0.01)
    assert h3d.h3d_last_kernel().startswith("k5_conv_mfma_kernel") == (Co * D * H * W >= 8)
    close(from_dev(dxg.t), dxo.a, TOL["bf16"])
    dwo, dbo = orc.convk_bwd_filter(5, xo, go, so, act, 0.01)
    dw, db = torch.empty((Co, Ci, 5, 5, 5), device="cuda"), torch.empty((Co,), device="cuda")
    h3d.conv3d_k5_bwd_filter(moved(xg), moved(gg), moved(sg), dw, db, act, 0.01)
    close(from_dev(dw), dwo, 2e-4)
    close(from_dev(db), dbo, 2e-4)


@pytest.mark.parametrize("alpha", [0.01, 0.3])
@pytest.mark.parametrize("shape", [(1, 17, 18, 3, 9, 33), (2, 33, 40, 4, 16, 30), (1, 8, 16, 2, 40, 70), (1, 32, 32, 6, 30, 50)])
def test_k5_ragged_masked_gradient_is_not_rounded(shape, alpha):
    """Rows that are no multiple of 8 with a leaky activation: g = dz * slope keeps its fp32 value.  The bar is that of a sum of the
    channel's V voxels in fp32, sqrt(V) 2^-23 (a gradient rounded to bf16 is off by alpha 2^-9: 1e-5 to 5e-4); a single element eight times that."""
    import torch
    import paper_2007_12856_amd as h3d
    N, Ci, Co, D, H, W = shape
    print("k5 ragged masked", shape, alpha, flush=True)
    xo, xg = slab_pair(synth.flat("normal", SEED, 561, (N, Ci, D, H, W)), "bf16")
    so, sg = slab_pair(synth.flat("normal", SEED, 562, (N, Co, D, H, W)), "bf16")
    go, gg = slab_pair(synth.flat("normal", SEED, 563, (N, Co, D, H, W)), "bf16")
    alpha = float(np.float32(alpha))
    dwo, dbo = orc.convk_bwd_filter(5, xo, go, so, orc.ACT_LEAKY, alpha)
    dw, db = torch.empty((Co, Ci, 5, 5, 5), device="cuda"), torch.empty((Co,), device="cuda")
    h3d.conv3d_k5_bwd_filter(xg, gg, sg, dw, db, h3d.ACT_LEAKY, alpha)
    bar = float(np.sqrt(N * D * H * W)) * 2.0 ** -23
    close(from_dev(dw), dwo, bar, elem=8 * bar)
    close(from_dev(db), dbo, bar, elem=8 * bar)


@pytest.mark.parametrize("masked", [False, True])
@pytest.mark.parametrize("shape", [(128, 128, 16, 60, 62), (100, 70, 5, 24, 40), (16, 16, 8, 64, 64)])
def test_k5_filter_gradient_sums_against_float64(shape, masked):
    """Many channels (fewer chunks than XCDs), rows for two rounds of workgroups, few channels.  A chain holds about 400 matrix products
    before a rounded addition takes it up; at one unit of the 24th bit each, in random directions, 20 2^-24.  (The slope
    is a power of two, so that aligned rows, whose g is rounded to bf16, are exact as well.)"""
    import torch
    import paper_2007_12856_amd as h3d
    Ci, Co, D, H, W = shape
    print("k5 sums", shape, masked, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(9)
    x = torch.randn((1, Ci, D + 4, H, W), device="cuda", generator=gen).bfloat16()
    dz = torch.randn((1, Co, D, H, W), device="cuda", generator=gen).bfloat16()
    z = None
    alpha = 0.25
    if masked:
        z = torch.randn(dz.shape, device="cuda", generator=gen).bfloat16()
    dw, db = torch.empty((Co, Ci, 5, 5, 5), device="cuda"), torch.empty((Co,), device="cuda")
    slab = lambda t, halo: h3d.Slab(t, halo, halo, D, 3 * D)
    h3d.conv3d_k5_bwd_filter(slab(x, 2), slab(dz, 0), slab(z, 0) if masked else None, dw, db, h3d.ACT_LEAKY if masked else h3d.ACT_NONE, alpha)
    assert h3d.h3d_last_kernel() == "k5_bwf_rows_kernel"
    g = dz.double()[0]
    if masked:
        g = torch.where(z[0] > 0, g, alpha * g)
    xp = torch.nn.functional.pad(x[0].double(), (2, 2, 2, 2))
    ref = torch.empty(dw.shape, dtype=torch.float64, device="cuda")
    gt = g.reshape(Co, -1)
    for a in range(5):
        for b in range(5):
            for c in range(5):
                ref[:, :, a, b, c] = gt @ xp[:, a:a + D, b:b + H, c:c + W].reshape(Ci, -1).t()
    bar = 20 * 2.0 ** -24
    assert float((dw.double() - ref).norm() / ref.norm()) <= bar
    assert float((db.double() - gt.sum(1)).norm() / gt.sum(1).norm()) <= bar


@pytest.mark.parametrize("shape", [(1, 33, 17, 5, 9, 33), (2, 40, 16, 3, 17, 16), (1, 9, 5, 2, 3, 5), (1, 16, 48, 9, 4, 70), (1, 5, 34, 1, 1, 17), (3, 64, 3, 6, 8, 15)])
def test_k5_f32_kernel_edges(shape):
    """fp32: one block of 16 results and two, rows up to 16 columns and beyond, two-row tiles that end within a tile, channel groups split over
    workgroups; the masked passes on an interior shard whose mask stores more planes than the gradient."""
    import torch
    import paper_2007_12856_amd as h3d
    N, Ci, Co, D, H, W = shape
    print("k5 f32 edges", shape, flush=True)
    rng = np.random.default_rng(Ci + W)
    w, bias = _weights(Ci, Co, "f32", 560)
    wd, bd = to_dev(w, "f32"), to_dev(bias, "f32")
    for off, dg in ((0, D), (3, D + 5)):
        h = (2, 2) if off else (0, 0)
        full = lambda c, hh: rng.standard_normal((N, c, D + sum(hh), H, W))
        xo, xg = slab_pair(full(Ci, h), "f32", h, off, dg)
        zo = orc.convk_fwd(xo, w, bias, orc.ACT_LEAKY, 0.01)
        zg = h3d.conv3d_k5_fwd(xg, wd, bd, dev_like(zo, "f32"), orc.ACT_LEAKY, 0.01)
        assert h3d.h3d_last_kernel().startswith("k5f_conv_kernel")
        close(from_dev(zg.t), zo.a, TOL["f32"], "z")
        go, gg = slab_pair(full(Co, h), "f32", h, off, dg)
        hs = (3, 2) if off else h
        so, sg = slab_pair(full(Co, hs), "f32", hs, off, dg)
        dxo = orc.convk_bwd_data(go, so, w, orc.ACT_LEAKY, 0.01)
        dxg = h3d.conv3d_k5_bwd_data(gg, sg, wd, dev_like(dxo, "f32"), orc.ACT_LEAKY, 0.01)
        assert h3d.h3d_last_kernel().startswith("k5f_conv_kernel")
        close(from_dev(dxg.t), dxo.a, TOL["f32"], "dx")
        dwo, dbo = orc.convk_bwd_filter(5, xo, go, so, orc.ACT_LEAKY, 0.01)
        dw, db = torch.full((Co, Ci, 5, 5, 5), float("nan"), device="cuda"), torch.full((Co,), float("nan"), device="cuda")
        h3d.conv3d_k5_bwd_filter(xg, gg, sg, dw, db, orc.ACT_LEAKY, 0.01)
        assert h3d.h3d_last_kernel().startswith("k5f_bwf_kernel")
        close(from_dev(dw), dwo, _tol_w("f32"), "dw")
        close(from_dev(db), dbo, _tol_w("f32"), "db")


def test_k5_f32_eight_row_tiles_equal_two_row_tiles():
    """Many samples take the 8-row tiles, one sample the 2-row tiles; a voxel's products come in the same order (one channel group: no split)."""
    import torch
    import paper_2007_12856_amd as h3d
    gen = torch.Generator(device="cuda").manual_seed(5)
    for W, Co in ((40, 20), (13, 20), (40, 9)):
        N = 80
        x = torch.randn((N, 3, 4, 61, W), device="cuda", generator=gen)
        w = torch.randn((Co, 3, 5, 5, 5), device="cuda", generator=gen)
        z = torch.randn((N, Co, 4, 61, W), device="cuda", generator=gen)
        y, y1 = torch.empty_like(z), torch.empty_like(z[:1])
        h3d.conv3d_k5_fwd(h3d.Slab(x), w, None, h3d.Slab(y), h3d.ACT_LEAKY, 0.01)
        assert ",8," in h3d.h3d_last_kernel()
        wt = torch.randn((3, Co, 5, 5, 5), device="cuda", generator=gen)      # of a layer Co -> 3: its data gradient has Co channels
        d, d1 = torch.empty_like(z), torch.empty_like(z[:1])
        h3d.conv3d_k5_bwd_data(h3d.Slab(x), h3d.Slab(x.roll(1, 0)), wt, h3d.Slab(d), h3d.ACT_LEAKY, 0.01)
        assert ",8," in h3d.h3d_last_kernel()
        for n in (0, N - 1):
            h3d.conv3d_k5_fwd(h3d.Slab(x[n:n + 1].contiguous()), w, None, h3d.Slab(y1), h3d.ACT_LEAKY, 0.01)
            assert ",2," in h3d.h3d_last_kernel() and torch.equal(y1[0], y[n])
            h3d.conv3d_k5_bwd_data(h3d.Slab(x[n:n + 1].contiguous()), h3d.Slab(x.roll(1, 0)[n:n + 1].contiguous()), wt, h3d.Slab(d1), h3d.ACT_LEAKY, 0.01)
            assert ",2," in h3d.h3d_last_kernel() and torch.equal(d1[0], d[n])


@pytest.mark.parametrize("N,ci,co,D,H,W", [(1, 96, 16, 3, 7, 16), (1, 30, 40, 2, 9, 33)])
def test_k5_f32_in_less_workspace(N, ci, co, D, H, W):
    """What a larger volume of the same channels asks for does (the channels are then not summed in parts), and what the vector ALU's kernels
    need does: their packed filter (16 channels a block, every contraction channel), or the chunks' partial sums."""
    import torch
    import paper_2007_12856_amd as h3d
    print("k5 f32 workspace", N, ci, co, D, H, W, flush=True)
    rng = np.random.default_rng(ci)
    w = quantize(rng.uniform(-1, 1, (co, ci, 5, 5, 5)) / np.sqrt(40 * ci), "f32")
    wd, bd = to_dev(w, "f32"), to_dev(rng.uniform(-0.1, 0.1, co), "f32")
    xo, xg = slab_pair(rng.standard_normal((N, ci, D, H, W)), "f32")
    go, gg = slab_pair(rng.standard_normal((N, co, D, H, W)), "f32")
    so, sg = slab_pair(rng.standard_normal((N, co, D, H, W)), "f32")
    big = lambda c: h3d.Slab(torch.empty((N, c, 64, 64, W), device="cuda"))
    packed = lambda a, b: -(-(-(-a // 16) * 16 * b * 125 * 4) // 256) * 256
    zo = orc.convk_fwd(xo, w, from_dev(bd), orc.ACT_LEAKY, 0.01)
    dxo = orc.convk_bwd_data(go, so, w, orc.ACT_LEAKY, 0.01)

    class Sized:
        def __init__(self, n):
            self.n, self.buf = n, torch.full((n + 4096,), 171, dtype=torch.uint8, device="cuda")

        def get(self, nbytes):
            assert nbytes > self.n
            return self.buf.data_ptr(), self.n

    for op, ref, least, call in ((h3d.OP_FWD, zo, packed(co, ci), lambda t, k: h3d.conv3d_k5_fwd(xg, wd, bd, t, h3d.ACT_LEAKY, 0.01, k)),
                                 (h3d.OP_BWD_DATA, dxo, packed(ci, co), lambda t, k: h3d.conv3d_k5_bwd_data(gg, sg, wd, t, h3d.ACT_LEAKY, 0.01, k))):
        for n, kernel in ((h3d.h3d_conv3d_k5_workspace_bytes(op, big(ci), big(co)), "k5f_conv"), (least, "")):
            ws, t = Sized(n), dev_like(ref, "f32", float("nan"))
            call(t, ws)
            assert h3d.h3d_last_kernel().startswith(kernel)
            close(from_dev(t.t), ref.a, TOL["f32"])
            assert bool((ws.buf[n:] == 171).all())
        with pytest.raises(h3d.H3DError):
            call(dev_like(ref, "f32"), Sized(least - 256))
