"""GPU parity of the three convolution passes against the CPU oracle (relative L2 and an element-by-element bound), on
seeded inputs at sizes the oracle finishes in seconds: several tiles, ragged tails, odd channel
counts, boundary and interior shards, halo recompute.  All calls go through the C ABI."""
import numpy as np
import pytest

import oracle as orc
import synth
from helpers import TOL, cut, dev_like, elem_masked_bf, from_dev, quantize, close, rel_l2, slab_pair, to_dev

pytestmark = pytest.mark.gpu
SEED = synth.BASE_SEED

# (N, Cin, Cout, Dg, H, W)
SHAPES = [
    (1, 4, 16, 32, 32, 32),      # the single-layer fp32 configuration's shape
    (2, 3, 5, 6, 7, 9),          # nothing divides anything
    (1, 1, 32, 8, 20, 70),       # single input channel (U-Net first layer), W spans two 64-wide tiles raggedly
    (1, 17, 4, 5, 9, 33),
    (2, 16, 32, 8, 12, 40),
    (1, 32, 64, 6, 10, 36),
    (1, 64, 16, 4, 6, 66),
    (1, 8, 8, 1, 1, 1),          # degenerate volume
]


def _weights(cin, cout, dtype, stream):
    b = np.sqrt(3.0 / (27 * cin))
    w = quantize(synth.flat("uniform", SEED, stream, (cout, cin, 3, 3, 3), -b, b), dtype)
    bias = synth.round_f32(synth.flat("uniform", SEED, stream + 1, (cout,), -0.1, 0.1)).astype(np.float64)
    return w, bias


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", SHAPES)
def test_conv3d_three_passes_unsharded(shape, dtype):
    import torch
    import paper_2007_12856_amd as h3d
    N, Ci, Co, D, H, W = shape
    alpha = 0.01
    w, bias = _weights(Ci, Co, dtype, 10)
    xo, xg = slab_pair(synth.flat("uniform", SEED, 1, (N, Ci, D, H, W)), dtype)
    wd, bd = to_dev(w, dtype), to_dev(bias, "f32")
    # forward
    zo = orc.conv3d_fwd(xo, w, bias, act=orc.ACT_LEAKY, alpha=alpha)
    zg = h3d.conv3d_fwd(xg, wd, bd, dev_like(zo, dtype), h3d.ACT_LEAKY, alpha)
    close(from_dev(zg.t), zo.a, TOL[dtype])
    # backward passes take the ORACLE's z (rounded to storage) as the saved output on both sides
    zq_o, zq_g = slab_pair(zo.a, dtype)
    dzo, dzg = slab_pair(synth.flat("uniform", SEED, 2, (N, Co, D, H, W)), dtype)
    dxo = orc.conv3d_bwd_data(dzo, zq_o, w, act=orc.ACT_LEAKY, alpha=alpha)
    dxg = h3d.conv3d_bwd_data(dzg, zq_g, wd, dev_like(dxo, dtype), h3d.ACT_LEAKY, alpha)
    close(from_dev(dxg.t), dxo.a, TOL[dtype])
    dwo, dbo = orc.conv3d_bwd_filter(xo, dzo, zq_o, act=orc.ACT_LEAKY, alpha=alpha)
    dw = torch.full((Co, Ci, 3, 3, 3), 777.0, device="cuda")
    db = torch.full((Co,), 777.0, device="cuda")
    h3d.conv3d_bwd_filter(xg, dzg, zq_g, dw, db, h3d.ACT_LEAKY, alpha)
    # dW stays fp32: with exact bf16 products and fp32 accumulation the error is far below the bf16 bar
    tol_w = 1e-5 if dtype == "f32" else 2e-4
    close(from_dev(dw), dwo, tol_w, elem=elem_masked_bf(dtype))
    close(from_dev(db), dbo, tol_w, elem=elem_masked_bf(dtype))
    # deterministic split-spatial reduction: a second call returns identical bits
    dw2, db2 = torch.empty_like(dw), torch.empty_like(db)
    h3d.conv3d_bwd_filter(xg, dzg, zq_g, dw2, db2, h3d.ACT_LEAKY, alpha)
    assert torch.equal(dw, dw2) and torch.equal(db, db2)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("act", [orc.ACT_NONE, orc.ACT_RELU])
def test_conv3d_no_bias_and_other_activations(dtype, act):
    import paper_2007_12856_amd as h3d
    N, Ci, Co, D, H, W = 1, 8, 16, 4, 6, 20
    w, _ = _weights(Ci, Co, dtype, 20)
    xo, xg = slab_pair(synth.flat("normal", SEED, 3, (N, Ci, D, H, W)), dtype)
    zo = orc.conv3d_fwd(xo, w, None, act=act)
    zg = h3d.conv3d_fwd(xg, to_dev(w, dtype), None, dev_like(zo, dtype), act, 0.0)
    close(from_dev(zg.t), zo.a, TOL[dtype])
    dzo, dzg = slab_pair(synth.flat("normal", SEED, 4, (N, Co, D, H, W)), dtype)
    zq_o, zq_g = slab_pair(zo.a, dtype)
    dxo = orc.conv3d_bwd_data(dzo, zq_o, w, act=act)
    dxg = h3d.conv3d_bwd_data(dzg, zq_g, to_dev(w, dtype), dev_like(dxo, dtype), act, 0.0)
    close(from_dev(dxg.t), dxo.a, TOL[dtype])


# (N, Cin, Cout, D, H, W, halo): unmasked filter gradients (the activation's mask already applied upstream), shapes
# chosen to reach every workgroup layout of the matrix-core kernels: first-layer (Cin <= 4) with one and two
# row blocks, 16- and 32-channel workgroups, one and two row groups, 4- and 6-row tiles, ragged H / W / channels
BF_SHAPES = [
    (1, 4, 16, 3, 36, 40, 1),
    (2, 3, 24, 2, 20, 64, 0),
    (1, 1, 40, 3, 33, 32, 1),
    (1, 16, 32, 3, 12, 40, 1),
    (1, 12, 16, 2, 9, 32, 0),
    (1, 32, 64, 3, 50, 32, 1),
    (1, 48, 80, 2, 10, 72, 1),
    (1, 20, 16, 2, 8, 96, 0),
    (1, 24, 24, 5, 7, 33, 1),
    (1, 4, 16, 2, 20, 72, 1),
    (1, 2, 10, 3, 17, 128, 0),
    # more than 32 channels on both sides: the kernel on the 32x32x16 tile (64-, 32- and 16-voxel row segments, ragged
    # bands and channel blocks, a ragged last K-step, chunks of several strips that cross planes and samples)
    (2, 40, 48, 3, 20, 16, 1),
    (1, 72, 40, 2, 9, 32, 0),
    (1, 64, 64, 4, 34, 64, 1),
    (2, 40, 40, 5, 18, 24, 1),
    (1, 36, 130, 2, 6, 136, 0),
    (4, 130, 130, 5, 10, 16, 1),
]


@pytest.mark.parametrize("kernel", ["by shape", "32x32x16 tile"])
@pytest.mark.parametrize("shape", BF_SHAPES)
def test_conv3d_bwd_filter_unmasked_bf16(shape, kernel, monkeypatch):
    import torch
    import paper_2007_12856_amd as h3d
    N, Ci, Co, D, H, W, halo = shape
    if kernel == "32x32x16 tile":
        # the library gives volumes this small to the kernels with smaller workgroup tiles; H3D_BF_ROW32=1 lifts that
        # limit, so that the many-channel kernel is compared with the oracle at sizes the oracle finishes in seconds
        if not (Ci > 32 and Co > 32):
            pytest.skip("the kernel takes more than 32 channels on both sides")
        monkeypatch.setenv("H3D_BF_ROW32", "1")
    else:
        monkeypatch.delenv("H3D_BF_ROW32", raising=False)
    dtype = "bf16"
    # with halo: the middle slab of a volume two planes taller (the halo planes hold real neighbours);
    # without: the whole volume, zero beyond both ends
    Dg, off = (D + 2, 1) if halo else (D, 0)
    xo, xg = slab_pair(synth.flat("normal", SEED, 30, (N, Ci, D + 2 * halo, H, W)), dtype, (halo, halo), off, Dg)
    dzo, dzg = slab_pair(synth.flat("normal", SEED, 31, (N, Co, D, H, W)), dtype, (0, 0), off, Dg)
    dwo, dbo = orc.conv3d_bwd_filter(xo, dzo, None, act=orc.ACT_NONE)
    dw = torch.full((Co, Ci, 3, 3, 3), 777.0, device="cuda")
    db = torch.full((Co,), 777.0, device="cuda")
    h3d.conv3d_bwd_filter(xg, dzg, None, dw, db, h3d.ACT_NONE, 0.0)
    close(from_dev(dw), dwo, 2e-4)
    close(from_dev(db), dbo, 2e-4)
    dw2, db2 = torch.empty_like(dw), torch.empty_like(db)
    h3d.conv3d_bwd_filter(xg, dzg, None, dw2, db2, h3d.ACT_NONE, 0.0)
    assert torch.equal(dw, dw2) and torch.equal(db, db2)
    if kernel == "32x32x16 tile":
        assert h3d.h3d_last_kernel().startswith("bwd_filter_row32_kernel"), h3d.h3d_last_kernel()


def _row32_random_shapes(k=8):
    rng = np.random.default_rng(SEED + 77)
    out = []
    for _ in range(k):
        out.append((int(rng.integers(1, 4)), int(rng.integers(33, 81)), int(rng.integers(33, 81)), int(rng.integers(1, 6)),
                    int(rng.integers(1, 21)), int(rng.choice([16, 24, 32, 40, 48, 64, 72, 96])), int(rng.integers(0, 2))))
    return out


@pytest.mark.parametrize("shape", _row32_random_shapes())
def test_conv3d_bwd_filter_many_channels_random_shapes(shape, monkeypatch):
    """Seeded random shapes for the kernel on the 32x32x16 tile (test hook H3D_BF_ROW32, see above): ragged channel
    blocks, bands, K-steps and chunks in combinations nobody picked by hand."""
    import torch
    import paper_2007_12856_amd as h3d
    monkeypatch.setenv("H3D_BF_ROW32", "1")
    N, Ci, Co, D, H, W, halo = shape
    dtype = "bf16"
    Dg, off = (D + 2, 1) if halo else (D, 0)
    xo, xg = slab_pair(synth.flat("normal", SEED, 32, (N, Ci, D + 2 * halo, H, W)), dtype, (halo, halo), off, Dg)
    dzo, dzg = slab_pair(synth.flat("normal", SEED, 33, (N, Co, D, H, W)), dtype, (0, 0), off, Dg)
    dwo, dbo = orc.conv3d_bwd_filter(xo, dzo, None, act=orc.ACT_NONE)
    dw = torch.full((Co, Ci, 3, 3, 3), 777.0, device="cuda")
    db = torch.full((Co,), 777.0, device="cuda")
    h3d.conv3d_bwd_filter(xg, dzg, None, dw, db, h3d.ACT_NONE, 0.0)
    assert h3d.h3d_last_kernel().startswith("bwd_filter_row32_kernel"), h3d.h3d_last_kernel()
    close(from_dev(dw), dwo, 2e-4, f"dw {shape}")
    close(from_dev(db), dbo, 2e-4, f"db {shape}")


@pytest.mark.parametrize("shape", [(1, 40, 32, 3, 18, 48, 0), (2, 70, 9, 2, 5, 56, 1), (1, 33, 24, 1, 1, 64, 0), (1, 130, 5, 4, 20, 136, 1), (3, 64, 17, 5, 16, 72, 0)])
def test_conv3d_bwd_filter_few_output_channels(shape, monkeypatch):
    """Up to 32 output channels on the 32x32x16 tile (test hook H3D_BF_ROW32, see above): two wavefronts share a row's columns, planes walked in step by x."""
    import torch
    import paper_2007_12856_amd as h3d
    monkeypatch.setenv("H3D_BF_ROW32", "1")
    N, Ci, Co, D, H, W, halo = shape
    print("few output channels", shape, flush=True)
    Dg, off = (D + 2, 1) if halo else (D, 0)
    xo, xg = slab_pair(synth.flat("normal", SEED, 34, (N, Ci, D + 2 * halo, H, W)), "bf16", (halo, halo), off, Dg)
    dzo, dzg = slab_pair(synth.flat("normal", SEED, 35, (N, Co, D, H, W)), "bf16", (0, 0), off, Dg)
    dwo, dbo = orc.conv3d_bwd_filter(xo, dzo, None, act=orc.ACT_NONE)
    dw = torch.full((Co, Ci, 3, 3, 3), 777.0, device="cuda")
    db = torch.full((Co,), 777.0, device="cuda")
    h3d.conv3d_bwd_filter(xg, dzg, None, dw, db, h3d.ACT_NONE, 0.0)
    assert h3d.h3d_last_kernel() == "bwd_filter_row32_kernel<64,1,1>", h3d.h3d_last_kernel()
    close(from_dev(dw), dwo, 2e-4, f"dw {shape}")
    close(from_dev(db), dbo, 2e-4, f"db {shape}")


@pytest.mark.parametrize("shape", [(1, 20, 24, 3, 9, 72, 0), (2, 17, 40, 2, 5, 96, 1), (1, 33, 8, 4, 6, 160, 0), (1, 16, 12, 2, 7, 88, 1)])
def test_conv3d_bwd_filter_odd_number_of_column_tiles(shape):
    """Rolling kernel on three and five tiles of 32 columns: walked one by one with two blocks of input channels, as pairs with one."""
    import torch
    import paper_2007_12856_amd as h3d
    N, Ci, Co, D, H, W, halo = shape
    print("odd number of column tiles", shape, flush=True)
    Dg, off = (D + 2, 1) if halo else (D, 0)
    xo, xg = slab_pair(synth.flat("normal", SEED, 36, (N, Ci, D + 2 * halo, H, W)), "bf16", (halo, halo), off, Dg)
    dzo, dzg = slab_pair(synth.flat("normal", SEED, 37, (N, Co, D, H, W)), "bf16", (0, 0), off, Dg)
    dwo, dbo = orc.conv3d_bwd_filter(xo, dzo, None, act=orc.ACT_NONE)
    dw = torch.full((Co, Ci, 3, 3, 3), 777.0, device="cuda")
    db = torch.full((Co,), 777.0, device="cuda")
    h3d.conv3d_bwd_filter(xg, dzg, None, dw, db, h3d.ACT_NONE, 0.0)
    assert h3d.h3d_last_kernel().startswith("bwd_filter_roll_kernel"), h3d.h3d_last_kernel()
    close(from_dev(dw), dwo, 2e-4, f"dw {shape}")
    close(from_dev(db), dbo, 2e-4, f"db {shape}")


# (N, Cin, Cout, D, H, W, halo): layers with a handful of channels on one side and at most 16 on the other, wide
# enough for the tap-row-folding kernel: backward-data onto <= 8 channels (no fused mask), forward onto <= 8
THIN_SHAPES = [
    (1, 4, 16, 5, 9, 40, 1),
    (2, 3, 12, 3, 6, 66, 0),
    (1, 8, 16, 6, 10, 32, 1),
    (1, 1, 7, 2, 5, 130, 0),
    # at most 4 channels, W a multiple of 8, H >= 8: the row-streaming variant (several depth tiles with a ragged
    # last one, several row segments, one to three column tiles)
    (2, 4, 16, 7, 33, 136, 1),
    (1, 2, 9, 9, 8, 64, 0),
    (1, 3, 16, 4, 20, 72, 1),
    (1, 4, 12, 2, 70, 32, 1),
    # backward-data onto at most 4 channels from 17 to 32: two passes of the row-streaming kernel over channel halves
    (1, 1, 32, 5, 12, 72, 1),
    (2, 4, 24, 3, 9, 40, 0),
    (1, 2, 17, 4, 16, 136, 1),
]


@pytest.mark.parametrize("shape", THIN_SHAPES)
def test_conv3d_few_channels_bf16(shape):
    import paper_2007_12856_amd as h3d
    N, Cs, Cl, D, H, W, halo = shape      # Cs: the small channel count, Cl: the larger one
    dtype = "bf16"
    Dg, off = (D + 2, 1) if halo else (D, 0)
    # backward-data of a Cs -> Cl layer: dz has Cl channels and a halo, dx has Cs channels
    w, bias = _weights(Cs, Cl, dtype, 40)
    dzo, dzg = slab_pair(synth.flat("normal", SEED, 41, (N, Cl, D + 2 * halo, H, W)), dtype, (halo, halo), off, Dg)
    dxo = orc.conv3d_bwd_data(dzo, None, w, act=orc.ACT_NONE)
    dxg = h3d.conv3d_bwd_data(dzg, None, to_dev(w, dtype), dev_like(dxo, dtype), h3d.ACT_NONE, 0.0)
    close(from_dev(dxg.t), dxo.a, TOL[dtype])
    # forward of a Cl -> Cs layer with bias and leaky ReLU
    w2, bias2 = _weights(Cl, Cs, dtype, 42)
    xo, xg = slab_pair(synth.flat("normal", SEED, 43, (N, Cl, D + 2 * halo, H, W)), dtype, (halo, halo), off, Dg)
    zo = orc.conv3d_fwd(xo, w2, bias2, act=orc.ACT_LEAKY, alpha=0.01)
    zg = h3d.conv3d_fwd(xg, to_dev(w2, dtype), to_dev(bias2, "f32"), dev_like(zo, dtype), h3d.ACT_LEAKY, 0.01)
    close(from_dev(zg.t), zo.a, TOL[dtype])


# (N, channels in, channels out, D, H, W) of a layer whose forward and backward-data both have half a channel chunk: tiles of 4 x 8 x 32 and one
# more or less on every side, odd rows, a channel
@pytest.mark.parametrize("shape", [(1, 8, 8, 3, 4, 17), (2, 6, 8, 4, 8, 18), (1, 8, 5, 5, 9, 34), (1, 7, 8, 4, 7, 33), (2, 5, 7, 9, 17, 65), (1, 8, 1, 3, 16, 31)])
def test_conv3d_wide_kernel_with_half_a_chunk(shape):
    """At most 8 contraction and 32 result channels on a wide volume: the wide kernel, on a copy where the operand is masked or its rows are odd;
    the same bits as the general kernel, which a result at an odd address still gets."""
    import torch
    import paper_2007_12856_amd as h3d
    N, Ci, Co, D, H, W = shape
    w, bias = _weights(Ci, Co, "bf16", 90)
    xo, xg = slab_pair(synth.flat("normal", SEED, 92, (N, Ci, D, H, W)), "bf16")
    dzo, dzg = slab_pair(synth.flat("normal", SEED, 93, (N, Co, D, H, W)), "bf16")
    zo, zg = slab_pair(synth.flat("normal", SEED, 94, (N, Co, D, H, W)), "bf16")
    wd, bd = to_dev(w, "bf16"), to_dev(bias, "f32")
    thin = W >= 32 and W % 2 == 0
    for name, ref, call, c in (("fwd", orc.conv3d_fwd(xo, w, bias, act=orc.ACT_LEAKY, alpha=0.01), lambda o: h3d.conv3d_fwd(xg, wd, bd, o, h3d.ACT_LEAKY, 0.01), Co),
                               ("bwd", orc.conv3d_bwd_data(dzo, zo, w, act=orc.ACT_LEAKY, alpha=0.01), lambda o: h3d.conv3d_bwd_data(dzg, zg, wd, o, h3d.ACT_LEAKY, 0.01), Ci)):
        n = N * c * D * H * W
        got = []
        for shift in (0, 1):
            buf = torch.full((n + 2,), 3.0, dtype=torch.bfloat16, device="cuda")
            out = h3d.Slab(buf[shift:shift + n].view(N, c, D, H, W))
            call(out)
            assert torch.all(buf[:shift] == 3.0) and torch.all(buf[shift + n:] == 3.0)
            got.append(out.t.clone())
            if not (name == "fwd" and thin):
                assert ("wide" in h3d.h3d_last_kernel()) == (shift == 0), h3d.h3d_last_kernel()
        close(from_dev(got[0]), ref.a, TOL["bf16"])
        assert torch.equal(got[0], got[1])


# (N, channels in, channels out, D, H, W): half a chunk, one block of output channels, two blocks of which the last is cut, odd rows, and enough tiles for
# two blocks a workgroup
@pytest.mark.parametrize("shape", [(1, 8, 12, 5, 9, 34), (2, 16, 32, 4, 8, 32), (1, 24, 40, 6, 10, 36), (1, 16, 24, 3, 8, 33), (2, 16, 64, 36, 66, 100)])
def test_conv3d_wide_kernel_activations(shape):
    """z = y > 0 ? y : slope * y for any slope (above 1, where the larger of y and slope * y is the wrong one, and below 0) and for infinite sums (-inf * 0 is NaN): the wide kernel stores what the
    general kernel does, which a result at an odd address gets."""
    import torch
    import paper_2007_12856_amd as h3d
    N, Ci, Co, D, H, W = shape
    w, bias = _weights(Ci, Co, "bf16", 96)
    wd, bd = to_dev(w, "bf16"), to_dev(bias, "f32")
    xo, xg = slab_pair(synth.flat("normal", SEED, 97, (N, Ci, D, H, W)), "bf16")
    xi = h3d.Slab(xg.t.clone())
    xi.t[0, Ci - 1, D // 2, H // 2, W // 2] = float("inf")
    n = N * Co * D * H * W
    for act, alpha, slope in ((h3d.ACT_LEAKY, 2.0, 2.0), (h3d.ACT_LEAKY, -0.5, -0.5), (h3d.ACT_LEAKY, 0.25, 0.25), (h3d.ACT_LEAKY, 1.0, 1.0), (h3d.ACT_RELU, 0.0, 0.0)):
        for x in (xg, xi):
            got = []
            for shift in (0, 1):
                buf = torch.full((n + 2,), 3.0, dtype=torch.bfloat16, device="cuda")
                out = h3d.Slab(buf[shift:shift + n].view(N, Co, D, H, W))
                h3d.conv3d_fwd(x, wd, bd, out, act, alpha)
                assert ("wide" in h3d.h3d_last_kernel()) == (shift == 0), h3d.h3d_last_kernel()
                got.append(out.t.clone())
            assert torch.all((got[0] == got[1]) | (got[0].isnan() & got[1].isnan())), alpha
            if x is xi:
                around = got[0][0, :, D // 2 - 1:D // 2 + 2, H // 2 - 1:H // 2 + 2, W // 2 - 1:W // 2 + 2]      # weights of both signs: sums of both signs
                assert bool((around == float("inf")).any()) and bool(around.isnan().any()) == (slope == 0.0)
                assert bool((around == float("-inf")).any()) == (slope > 0.0)
            elif n < 10 ** 5:
                close(from_dev(got[0]), orc.conv3d_fwd(xo, w, bias, act=orc.ACT_LEAKY, alpha=slope).a, TOL["bf16"])


@pytest.mark.parametrize("shape,form", [((1, 8, 8, 9, 30, 41), "1,8,32,1,0,0,0"), ((1, 64, 16, 2, 33, 33), "2,4,32,1,0,0,1"), ((1, 40, 16, 2, 33, 13), "2,4,16,1,0,0,1"),
                                        ((1, 16, 16, 9, 17, 15), "1,8,16,1,0,0,0"), ((1, 24, 40, 9, 17, 15), "1,8,16,1,0,1,0")])
def test_conv3d_masked_odd_rows_without_room_for_the_copy(shape, form):
    """Masked backward-data of odd rows in a workspace without room for a prepared copy: the general kernel's masked forms, which have the bits of the
    call with room."""
    import torch
    import paper_2007_12856_amd as h3d

    class Fixed(h3d.Workspace):      # what the packed filter (and the sums of a split) take, whatever the call would like
        def get(self, nbytes):
            return super().get(self.size)

    N, Ci, Co, D, H, W = shape
    w, _ = _weights(Ci, Co, "bf16", 98)
    dzo, dzg = slab_pair(synth.flat("normal", SEED, 99, (N, Co, D, H, W)), "bf16")
    zo, zg = slab_pair(synth.flat("normal", SEED, 100, (N, Co, D, H, W)), "bf16")
    dxo = orc.conv3d_bwd_data(dzo, zo, w, act=orc.ACT_LEAKY, alpha=0.01)
    wd, ws = to_dev(w, "bf16"), Fixed()
    even = [h3d.Slab(torch.empty((N, c, D, H, W + 1), dtype=torch.bfloat16, device="cuda")) for c in (Co, Ci)]
    ws.size = h3d.h3d_conv3d_workspace_bytes(h3d.OP_FWD, *even)
    got = [h3d.conv3d_bwd_data(dzg, zg, wd, dev_like(dxo, "bf16"), h3d.ACT_LEAKY, 0.01, s).t for s in (h3d.Workspace(), ws)]
    assert h3d.h3d_last_kernel().startswith(f"conv3d_mfma_kernel<{form},"), h3d.h3d_last_kernel()
    close(from_dev(got[1]), dxo.a, TOL["bf16"])
    assert torch.equal(*got)


def _in_a_tall_tensor(t):
    """A copy of t, all of whose planes lie in a bf16 tensor whose samples are past 31-bit byte offsets, next to its end (a Slab), and that tensor."""
    import torch
    import paper_2007_12856_amd as h3d
    n, c, d, h, w = t.shape
    tall = torch.full((n, c, -(-2 ** 30 // (c * h * w)), h, w), 3.0, dtype=torch.bfloat16, device="cuda")
    p = tall.shape[2] - d - 1
    tall[:, :, p:p + d] = t
    return h3d.Slab(tall[:, :, p:p + d]), tall, p


def test_conv3d_first_layer_into_a_view_of_a_tall_tensor():
    """z is a run of planes of such a tensor: not the row-streaming kernel, which stores through 32-bit offsets; nothing around the run is written."""
    import torch
    import paper_2007_12856_amd as h3d
    Ci, Co, D, H, W = 4, 16, 4, 8, 32
    w, bias = _weights(Ci, Co, "bf16", 101)
    xo, xg = slab_pair(synth.flat("normal", SEED, 102, (1, Ci, D, H, W)), "bf16")
    zo = orc.conv3d_fwd(xo, w, bias, act=orc.ACT_LEAKY, alpha=0.01)
    wd, bd = to_dev(w, "bf16"), to_dev(bias, "f32")
    h3d.conv3d_fwd(xg, wd, bd, dev_like(zo, "bf16"), h3d.ACT_LEAKY, 0.01)
    roll = h3d.h3d_last_kernel()
    z, tall, p = _in_a_tall_tensor(torch.zeros((1, Co, D, H, W), device="cuda"))
    h3d.conv3d_fwd(xg, wd, bd, z, h3d.ACT_LEAKY, 0.01)
    assert "roll" in roll and "roll" not in h3d.h3d_last_kernel(), (roll, h3d.h3d_last_kernel())
    close(from_dev(z.t), zo.a, TOL["bf16"])
    assert torch.all(tall[:, :, :p] == 3.0) and torch.all(tall[:, :, p + D:] == 3.0)


def test_conv3d_masked_by_a_view_of_a_tall_tensor():
    """The saved output of a masked data gradient is a run of planes of such a tensor: copied where the workspace has room, on the direct kernel where not."""
    import torch
    import paper_2007_12856_amd as h3d
    N, Ci, Co, D, H, W = 1, 16, 24, 5, 9, 33
    w, _ = _weights(Ci, Co, "bf16", 103)
    dzo, dzg = slab_pair(synth.flat("normal", SEED, 104, (N, Co, D, H, W)), "bf16")
    zo, zg = slab_pair(synth.flat("normal", SEED, 105, (N, Co, D, H, W)), "bf16")
    dxo = orc.conv3d_bwd_data(dzo, zo, w, act=orc.ACT_LEAKY, alpha=0.01)
    z, _, _ = _in_a_tall_tensor(zg.t)
    even = [h3d.Slab(torch.empty((N, c, D, H, W + 1), dtype=torch.bfloat16, device="cuda")) for c in (Co, Ci)]

    class Fixed(h3d.Workspace):
        def get(self, nbytes):
            return super().get(h3d.h3d_conv3d_workspace_bytes(h3d.OP_FWD, *even))

    for ws, kernel in ((h3d.Workspace(), "conv3d_mfma_wide"), (Fixed(), "conv3d_direct")):
        dx = h3d.conv3d_bwd_data(dzg, z, to_dev(w, "bf16"), dev_like(dxo, "bf16"), h3d.ACT_LEAKY, 0.01, ws)
        assert h3d.h3d_last_kernel().startswith(kernel), h3d.h3d_last_kernel()
        close(from_dev(dx.t), dxo.a, TOL["bf16"])


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("cin,cout", [(4, 16), (3, 5), (16, 32)])
def test_conv3d_sharded_matches_oracle_and_unsharded_gpu(dtype, cin, cout):
    """Boundary and interior shards; halo planes outside the volume hold a canary that must not be read;
    the concatenated shard outputs equal the unsharded GPU output bit for bit (the accumulation
    order of a voxel does not depend on the slab it is computed in)."""
    import torch
    import paper_2007_12856_amd as h3d
    N, Dg, H, W, nshard = 2, 12, 10, 34, 3
    d = Dg // nshard
    full = (N, cin, Dg, H, W)
    w, bias = _weights(cin, cout, dtype, 30)
    wd, bd = to_dev(w, dtype), to_dev(bias, "f32")
    xfo, xfg = slab_pair(synth.slab("cosmo", SEED, 5, full, 0, Dg), dtype)
    zfo = orc.conv3d_fwd(xfo, w, bias, act=orc.ACT_LEAKY, alpha=0.01)
    zfg = h3d.conv3d_fwd(xfg, wd, bd, dev_like(zfo, dtype), h3d.ACT_LEAKY, 0.01)
    dzf = synth.slab("normal", SEED, 6, (N, cout, Dg, H, W), 0, Dg)
    dzfo, dzfg = slab_pair(dzf, dtype)
    zqo, zqg = slab_pair(zfo.a, dtype)
    dxfg = h3d.conv3d_bwd_data(dzfg, zqg, wd, dev_like(xfo, dtype), h3d.ACT_LEAKY, 0.01)
    dwf = torch.empty((cout, cin, 3, 3, 3), device="cuda")
    dbf = torch.empty((cout,), device="cuda")
    h3d.conv3d_bwd_filter(xfg, dzfg, zqg, dwf, dbf, h3d.ACT_LEAKY, 0.01)
    dw_sum = torch.zeros_like(dwf, dtype=torch.float64)
    db_sum = torch.zeros_like(dbf, dtype=torch.float64)
    dwo_sum = 0.0
    for s in range(nshard):
        off = s * d
        xs = cut("cosmo", SEED, 5, full, off, d, (1, 1))
        for pl, g in enumerate(range(off - 1, off + d + 1)):
            if g < 0 or g >= Dg:
                xs[:, :, pl] = 999.0          # canary outside the volume
        xo, xg = slab_pair(xs, dtype, (1, 1), off, Dg)
        zo = orc.conv3d_fwd(xo, w, bias, act=orc.ACT_LEAKY, alpha=0.01)
        zg = h3d.conv3d_fwd(xg, wd, bd, dev_like(zo, dtype), h3d.ACT_LEAKY, 0.01)
        close(from_dev(zg.t), zo.a, TOL[dtype])
        assert torch.equal(zg.t, zfg.t[:, :, off:off + d])
        # backward-data: dz and z carry the exchanged halo
        zs = np.full((N, cout, d + 2, H, W), 999.0)
        dzs = np.full((N, cout, d + 2, H, W), 999.0)
        for pl, g in enumerate(range(off - 1, off + d + 1)):
            if 0 <= g < Dg:
                zs[:, :, pl], dzs[:, :, pl] = zfo.a[:, :, g], dzf[:, :, g]
        zso, zsg = slab_pair(zs, dtype, (1, 1), off, Dg)
        dzo, dzg = slab_pair(dzs, dtype, (1, 1), off, Dg)
        dxo = orc.conv3d_bwd_data(dzo, zso, w, act=orc.ACT_LEAKY, alpha=0.01)
        dxg = h3d.conv3d_bwd_data(dzg, zsg, wd, dev_like(dxo, dtype), h3d.ACT_LEAKY, 0.01)
        close(from_dev(dxg.t), dxo.a, TOL[dtype])
        assert torch.equal(dxg.t, dxfg.t[:, :, off:off + d])
        # backward-filter partial of this shard
        dwo, dbo = orc.conv3d_bwd_filter(xo, dzo, zso, act=orc.ACT_LEAKY, alpha=0.01)
        dw, db = torch.empty_like(dwf), torch.empty_like(dbf)
        h3d.conv3d_bwd_filter(xg, dzg, zsg, dw, db, h3d.ACT_LEAKY, 0.01)
        close(from_dev(dw), dwo, TOL[dtype])
        close(from_dev(db), dbo, TOL[dtype])
        dw_sum += dw.double()
        db_sum += db.double()
        dwo_sum = dwo_sum + dwo
    close(dw_sum.cpu().numpy(), from_dev(dwf), 1e-5)
    close(db_sum.cpu().numpy(), from_dev(dbf), 1e-5)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("cin,cout,W,exact", [(4, 16, 40, True), (16, 32, 32, True), (24, 8, 36, True), (64, 128, 40, True),
                                              (64, 128, 8, False), (256, 256, 8, True)])      # (72 workgroups)
def test_main_halo_split_is_bit_exact(dtype, cin, cout, W, exact):
    """Sec. III-C: the planes that need no halo (main) and the two strips that do are computed by separate
    calls on plane-run views of the same buffers; together they must reproduce the whole-slab call bit for bit."""
    import torch
    import paper_2007_12856_amd as h3d
    N, D, H = 2, 9, 18
    w, bias = _weights(cin, cout, dtype, 50)
    wd, bd = to_dev(w, dtype), to_dev(bias, "f32")
    xo, xg = slab_pair(synth.flat("normal", SEED, 51, (N, cin, D + 2, H, W)), dtype, (1, 1), 3, D + 6)
    zo = orc.conv3d_fwd(xo, w, bias, act=orc.ACT_LEAKY, alpha=0.01)
    whole = h3d.conv3d_fwd(xg, wd, bd, dev_like(zo, dtype), h3d.ACT_LEAKY, 0.01)
    close(from_dev(whole.t), zo.a, TOL[dtype])
    parts = dev_like(zo, dtype)
    for p0, p1 in [(1, D - 1), (0, 1), (D - 1, D)]:          # main first, then the two strips
        h3d.conv3d_fwd(xg.planes(p0, p1, 1, 1), wd, bd, parts.planes(p0, p1), h3d.ACT_LEAKY, 0.01)
    if exact or dtype == "f32":
        assert torch.equal(parts.t, whole.t)
    else:
        close(from_dev(parts.t), zo.a, TOL[dtype])
    # backward-data on the same split
    dzo, dzg = slab_pair(synth.flat("normal", SEED, 52, (N, cout, D + 2, H, W)), dtype, (1, 1), 3, D + 6)
    dxo = orc.conv3d_bwd_data(dzo, None, w, act=orc.ACT_NONE)
    dx_whole = h3d.conv3d_bwd_data(dzg, None, wd, dev_like(dxo, dtype), h3d.ACT_NONE, 0.0)
    close(from_dev(dx_whole.t), dxo.a, TOL[dtype])
    dx_parts = dev_like(dxo, dtype)
    for p0, p1 in [(2, D - 2), (0, 2), (D - 2, D)]:
        h3d.conv3d_bwd_data(dzg.planes(p0, p1, 1, 1), None, wd, dx_parts.planes(p0, p1), h3d.ACT_NONE, 0.0)
    if exact or dtype == "f32":
        assert torch.equal(dx_parts.t, dx_whole.t)
    else:
        close(from_dev(dx_parts.t), dxo.a, TOL[dtype])
    # backward-filter: the strips' partial gradients add up to the whole slab's (different summation order)
    go, gg = slab_pair(synth.flat("normal", SEED, 53, (N, cout, D, H, W)), dtype, (0, 0), 3, D + 6)
    dwo, dbo = orc.conv3d_bwd_filter(xo, go, None, act=orc.ACT_NONE)
    dw = torch.zeros((cout, cin, 3, 3, 3), device="cuda")
    db = torch.zeros((cout,), device="cuda")
    for p0, p1 in [(1, D - 1), (0, 1), (D - 1, D)]:
        dwp, dbp = torch.empty_like(dw), torch.empty_like(db)
        h3d.conv3d_bwd_filter(xg.planes(p0, p1, 1, 1), gg.planes(p0, p1), None, dwp, dbp, h3d.ACT_NONE, 0.0)
        dw += dwp
        db += dbp
    tol_w = 1e-5 if dtype == "f32" else 2e-4
    close(from_dev(dw), dwo, tol_w)
    close(from_dev(db), dbo, tol_w)


@pytest.mark.parametrize("dtype,N,c,D,H,W", [("bf16", 2, 64, 9, 18, 32), ("f32", 2, 64, 9, 18, 32), ("bf16", 4, 256, 16, 8, 8), ("bf16", 2, 64, 9, 18, 8)])
def test_whole_samples_are_summed_in_parts_and_views_are_not(dtype, N, c, D, H, W):
    """Which calls may sum their channels in parts: the packed whole sample does; plane runs of it, one in a packed tensor of its own with the
    neighbours as halos, and its channels as a range of a wider tensor do not, and these agree bit for bit."""
    import torch
    import paper_2007_12856_amd as h3d
    print("whole and views", dtype, N, c, D, H, W, flush=True)
    g = torch.Generator(device="cuda").manual_seed(c + W)
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    x = torch.randn((N, c, D, H, W), generator=g, device="cuda").to(td)
    w = (0.05 * torch.randn((c, c, 3, 3, 3), generator=g, device="cuda")).to(td)

    def fwd(xs, zs):
        h3d.conv3d_fwd(xs, w, None, zs, h3d.ACT_LEAKY, 0.01)
        name = h3d.h3d_last_kernel()
        return zs.t, "split" in name or (name.startswith("conv3d_mfma_kernel<") and name.split(",")[5] == "1")

    whole, parted = fwd(h3d.Slab(x), h3d.Slab(torch.empty_like(x)))
    assert parted
    views = h3d.Slab(torch.empty_like(x))
    for p0, p1 in ((1, D - 1), (0, 1), (D - 1, D)):
        assert not fwd(h3d.Slab(x).planes(p0, p1, 1 if p0 else 0, 1 if p1 < D else 0), views.planes(p0, p1))[1]
    wide = torch.empty((N, 2 * c, D, H, W), dtype=td, device="cuda")
    ranged, parted = fwd(h3d.Slab(x), h3d.Slab(wide[:, c:]))
    assert not parted and torch.equal(ranged, views.t)
    if W > 16 or N * D * c > 8192:      # (narrow shards of fewer than 64 workgroups are summed in parts)
        inner = x[:, :, 1:D - 1].contiguous()
        shard, parted = fwd(h3d.Slab(x, 1, 1, 1, D), h3d.Slab(torch.empty_like(inner), 0, 0, 1, D))
        assert not parted and torch.equal(shard, views.t[:, :, 1:D - 1])
    # as many products summed in another order
    bar = 2.0 ** -8 if dtype == "bf16" else 2.0 ** -23 * (27 * c) ** 0.5
    assert float((views.t.double() - whole.double()).norm()) <= bar * float(whole.double().norm())


# (N, Cin, Cout, D, H, W, halo, d_offset, d_global): fp32 tensors on the matrix cores.  Both instances of the forward kernel
# (one and two blocks of 16 output channels per workgroup; 2-row tiles since these volumes are small), channel counts that fill neither the groups of 4 input
# channels nor the blocks of 16 output channels, two workgroups of output channels, W beyond one 32-column tile with a
# ragged tail, W not a multiple of 4 (no 16-byte stores), H beyond one 8-row tile, more planes than one workgroup's four,
# boundary and interior shards, and backward-filter chunks of several tiles
F32_SHAPES = [
    (1, 6, 16, 5, 11, 44, 0, 0, 5),
    (2, 5, 20, 3, 9, 37, 1, 0, 3),
    (1, 40, 48, 6, 20, 40, 1, 6, 18),
    (2, 40, 48, 6, 20, 40, 1, 12, 18),
    (1, 18, 70, 2, 8, 66, 0, 0, 2),
    (1, 33, 7, 9, 4, 16, 1, 0, 12),
    (2, 8, 40, 16, 100, 132, 0, 0, 16),     # enough 8-row tiles to fill the chip: the 8-row instances
    (2, 36, 12, 16, 100, 132, 0, 0, 16),
    # at most 4 channels on the output side of the correlation (thin form: the three kh taps share a product) or on the
    # input side of backward-filter (the three kw taps share a product)
    (1, 4, 16, 6, 20, 40, 1, 0, 6),
    (2, 20, 3, 5, 9, 37, 0, 0, 5),
    (2, 1, 2, 3, 10, 72, 1, 3, 9),
    (2, 16, 4, 16, 100, 132, 0, 0, 16),
    # volumes at most 16 voxels wide: 16-column tiles (forward / BD) and 8-row x 16-column tiles (BF)
    (2, 20, 24, 4, 12, 8, 1, 0, 4),
    (1, 3, 6, 5, 9, 12, 0, 0, 5),
    (4, 5, 6, 16, 256, 16, 0, 0, 16),
    # forms of one block and of 8 rows that the shapes above do not take
    (2, 5, 32, 16, 128, 128, 0, 0, 16),
    (1, 5, 32, 4, 128, 128, 0, 0, 4),
    (4, 5, 32, 16, 32, 16, 0, 0, 16),
    (1, 9, 40, 5, 34, 40, 1, 4, 16),
]


kernels_seen = set()


@pytest.mark.parametrize("shape", F32_SHAPES)
def test_conv3d_fp32_matrix_core_kernels(shape):
    """Sec. III-C FP / BD / BF in the paper's own precision (fp32 storage and arithmetic) against the fp64 oracle at the
    1e-5 bar, with the kernel that ran checked by name."""
    import torch
    import paper_2007_12856_amd as h3d
    N, Ci, Co, D, H, W, halo, off, Dg = shape
    alpha = 0.01
    w, bias = _weights(Ci, Co, "f32", 60)
    wd, bd = to_dev(w, "f32"), to_dev(bias, "f32")
    hl = (halo, halo)
    xs = synth.flat("normal", SEED, 61, (N, Ci, D + 2 * halo, H, W))
    dzs = synth.flat("normal", SEED, 62, (N, Co, D + 2 * halo, H, W))
    for pl in range(D + 2 * halo):                    # canaries in halo planes outside the volume: never read
        g = off - halo + pl
        if g < 0 or g >= Dg:
            xs[:, :, pl] = 999.0
            dzs[:, :, pl] = 999.0
    xo, xg = slab_pair(xs, "f32", hl, off, Dg)
    zo = orc.conv3d_fwd(xo, w, bias, act=orc.ACT_LEAKY, alpha=alpha)
    zg = h3d.conv3d_fwd(xg, wd, bd, dev_like(zo, "f32"), h3d.ACT_LEAKY, alpha)
    form = lambda c: "thin" if c <= 4 else ("1" if c <= 16 else "2")
    assert h3d.h3d_last_kernel().startswith("conv3d_f32_mfma_kernel<%s," % form(Co)), h3d.h3d_last_kernel()
    kernels_seen.add(h3d.h3d_last_kernel())
    close(from_dev(zg.t), zo.a, 1e-5)
    # backward passes: z and dz with the same halo (what the neighbours would have sent)
    zfull = synth.flat("normal", SEED, 63, (N, Co, D + 2 * halo, H, W))
    zso, zsg = slab_pair(zfull, "f32", hl, off, Dg)
    dzo, dzg = slab_pair(dzs, "f32", hl, off, Dg)
    dxo = orc.conv3d_bwd_data(dzo, zso, w, act=orc.ACT_LEAKY, alpha=alpha)
    dxg = h3d.conv3d_bwd_data(dzg, zsg, wd, dev_like(dxo, "f32"), h3d.ACT_LEAKY, alpha)
    assert h3d.h3d_last_kernel().startswith("conv3d_f32_mfma_kernel<%s," % form(Ci)), h3d.h3d_last_kernel()
    kernels_seen.add(h3d.h3d_last_kernel())
    close(from_dev(dxg.t), dxo.a, 1e-5)
    dwo, dbo = orc.conv3d_bwd_filter(xo, dzo, zso, act=orc.ACT_LEAKY, alpha=alpha)
    dw = torch.full((Co, Ci, 3, 3, 3), 777.0, device="cuda")
    db = torch.full((Co,), 777.0, device="cuda")
    h3d.conv3d_bwd_filter(xg, dzg, zsg, dw, db, h3d.ACT_LEAKY, alpha)
    assert h3d.h3d_last_kernel() == ("bwd_filter_f32_mfma_kernel<thin>" if Ci <= 4 else "bwd_filter_f32_mfma_kernel"), h3d.h3d_last_kernel()
    close(from_dev(dw), dwo, 1e-5)
    close(from_dev(db), dbo, 1e-5)
    dw2, db2 = torch.empty_like(dw), torch.empty_like(db)
    h3d.conv3d_bwd_filter(xg, dzg, zsg, dw2, db2, h3d.ACT_LEAKY, alpha)
    assert torch.equal(dw, dw2) and torch.equal(db, db2)
    # no activation, no saved output, no bias gradient wanted
    dwo_n, _ = orc.conv3d_bwd_filter(xo, dzo, None, act=orc.ACT_NONE)
    h3d.conv3d_bwd_filter(xg, dzg, None, dw2, None, h3d.ACT_NONE, 0.0)
    close(from_dev(dw2), dwo_n, 1e-5)


# (N, channels in, channels out, D, H, W, planes of the volume on either side of the shard, kernel forward, kernel backward-data) on 256 CUs: one block
# of several a workgroup (whole samples and shards, 2 and 8 rows, 32 and 16 columns, a last block of few channels); shapes where two blocks, split, are faster
@pytest.mark.parametrize("shape,fwd,bwd", [
    ((2, 64, 32, 16, 50, 80, 0), "1,2,2", "2,2,2"),
    ((1, 20, 40, 16, 66, 33, 1), "1,2,2", "1,2,2"),
    ((1, 24, 48, 16, 66, 12, 2), "1,2,1", "2,2,1"),
    ((1, 48, 24, 16, 66, 12, 1), "2,2,1", "1,2,1"),
    ((4, 16, 33, 12, 104, 24, 0), "1,8,2", "1,2,2"),
    ((1, 147, 128, 16, 37, 32, 0), "2,2,2> (split)", "1,2,2"),
    ((1, 254, 71, 16, 54, 16, 0), "2,2,1> (split)", "1,2,1"),
])
def test_conv3d_fp32_tile_forms(shape, fwd, bwd):
    """The tile form that the planner takes, by name, and its result (masked in the data gradient) against the tap-by-tap products in 64 bits."""
    import torch
    import paper_2007_12856_amd as h3d
    N, Ci, Co, D, H, W, beside = shape
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the forms are those of 256 CUs")
    g = torch.Generator(device="cuda").manual_seed(Ci * Co + W)
    halo, ends = (1, (beside, D + 2 * beside)) if beside else (0, (0, D))
    normal = lambda c, p: torch.randn((N, c, D + 2 * p, H, W), generator=g, device="cuda")
    slab = lambda t, p: h3d.Slab(t, p, p, *ends)
    x, dz, z = normal(Ci, halo), normal(Co, halo), normal(Co, halo)
    w = (torch.rand((Co, Ci, 3, 3, 3), generator=g, device="cuda") - 0.5) * 2 * (3.0 / (27 * Ci)) ** 0.5
    b = torch.rand((Co,), generator=g, device="cuda") - 0.5

    def products(t, w):      # of a tensor with its halo planes, or zeros for them
        t = torch.nn.functional.pad(t.double(), (1, 1, 1, 1) + ((0, 0) if halo else (1, 1)))
        out = torch.zeros((N, w.shape[0], D * H * W), dtype=torch.float64, device="cuda")
        for tap in range(27):
            i, j, k = tap // 9, tap // 3 % 3, tap % 3
            for n in range(N):
                out[n] += w[:, :, i, j, k].double() @ t[n, :, i:i + D, j:j + H, k:k + W].reshape(t.shape[1], -1)
        return out.view(N, -1, D, H, W)

    y, dx = (torch.empty((N, c, D, H, W), device="cuda") for c in (Co, Ci))
    h3d.conv3d_fwd(slab(x, halo), w, b, slab(y, 0), h3d.ACT_LEAKY, 0.01)
    name = lambda form: "conv3d_f32_mfma_kernel<%s%s" % (form, "" if ">" in form else ">")
    assert h3d.h3d_last_kernel() == name(fwd), h3d.h3d_last_kernel()
    want = products(x, w) + b.double().view(1, -1, 1, 1, 1)
    close(from_dev(y), torch.where(want > 0, want, 0.01 * want).cpu().numpy(), 1e-5)
    h3d.conv3d_bwd_data(slab(dz, halo), slab(z, halo), w, slab(dx, 0), h3d.ACT_LEAKY, 0.01)
    assert h3d.h3d_last_kernel() == name(bwd), h3d.h3d_last_kernel()
    close(from_dev(dx), products(torch.where(z > 0, dz, 0.01 * dz), w.transpose(0, 1).flip(2, 3, 4)).cpu().numpy(), 1e-5)


def _f32_random_shapes(k=12):
    rng = np.random.default_rng(SEED + 99)
    out = []
    for _ in range(k):
        ci = int(rng.choice([1, 2, 3, 4, 5, 7, 8, 12, 17, 24, 33]))
        co = int(rng.choice([1, 3, 4, 5, 9, 16, 17, 20, 32, 35]))
        d, halo = int(rng.integers(1, 8)), int(rng.integers(0, 2))
        out.append((int(rng.integers(1, 3)), ci, co, d, int(rng.integers(1, 23)), int(rng.choice([3, 8, 12, 16, 17, 31, 32, 40, 66])), halo,
                    int(rng.choice([0, 4])) if halo else 0))
    return out


@pytest.mark.parametrize("shape", _f32_random_shapes())
def test_conv3d_fp32_random_shapes(shape):
    """Seeded random shapes for the fp32 matrix-core kernels: channel counts on either side of the thin / one-block /
    two-block forms, widths on either side of the 16-column tiles, ragged rows, planes and halos in combinations nobody
    picked by hand; all three passes with the fused activation derivative, against the oracle at the fp32 bar."""
    import torch
    import paper_2007_12856_amd as h3d
    N, Ci, Co, D, H, W, halo, off = shape
    Dg = off + D + (4 if halo else 0)
    alpha = 0.01
    w, bias = _weights(Ci, Co, "f32", 70)
    wd, bd = to_dev(w, "f32"), to_dev(bias, "f32")
    hl = (halo, halo)
    xo, xg = slab_pair(synth.flat("normal", SEED, 71, (N, Ci, D + 2 * halo, H, W)), "f32", hl, off, Dg)
    zo = orc.conv3d_fwd(xo, w, bias, act=orc.ACT_LEAKY, alpha=alpha)
    zg = h3d.conv3d_fwd(xg, wd, bd, dev_like(zo, "f32"), h3d.ACT_LEAKY, alpha)
    assert h3d.h3d_last_kernel().startswith("conv3d_f32_mfma_kernel"), h3d.h3d_last_kernel()
    close(from_dev(zg.t), zo.a, 1e-5, f"fwd {shape}")
    zso, zsg = slab_pair(synth.flat("normal", SEED, 73, (N, Co, D + 2 * halo, H, W)), "f32", hl, off, Dg)
    dzo, dzg = slab_pair(synth.flat("normal", SEED, 72, (N, Co, D + 2 * halo, H, W)), "f32", hl, off, Dg)
    dxo = orc.conv3d_bwd_data(dzo, zso, w, act=orc.ACT_LEAKY, alpha=alpha)
    dxg = h3d.conv3d_bwd_data(dzg, zsg, wd, dev_like(dxo, "f32"), h3d.ACT_LEAKY, alpha)
    close(from_dev(dxg.t), dxo.a, 1e-5, f"bwd_data {shape}")
    dwo, dbo = orc.conv3d_bwd_filter(xo, dzo, zso, act=orc.ACT_LEAKY, alpha=alpha)
    dw = torch.full((Co, Ci, 3, 3, 3), 777.0, device="cuda")
    db = torch.full((Co,), 777.0, device="cuda")
    h3d.conv3d_bwd_filter(xg, dzg, zsg, dw, db, h3d.ACT_LEAKY, alpha)
    assert h3d.h3d_last_kernel().startswith("bwd_filter_f32_mfma_kernel"), h3d.h3d_last_kernel()
    close(from_dev(dw), dwo, 1e-5, f"dw {shape}")
    close(from_dev(db), dbo, 1e-5, f"db {shape}")


def test_conv3d_fp32_every_instance_was_run():
    """The shapes above reach the instances of the fp32 forward / backward-data kernel (channel-block form x tile rows x
    tile halves) (collected from the library's
    own report of the kernel it ran); skipped when that test was not run in this process."""
    if not kernels_seen:
        pytest.skip("test_conv3d_fp32_matrix_core_kernels did not run in this process")
    want = {"conv3d_f32_mfma_kernel<%s,%d,2>" % (cb, tr) for cb in ("1", "2", "thin") for tr in (2, 8)}
    want |= {"conv3d_f32_mfma_kernel<%s,1>" % k for k in ("1,8", "1,2", "2,2", "thin,2")}
    assert want <= kernels_seen, (want - kernels_seen, kernels_seen)


def test_plane_run_views_are_rejected_elsewhere():
    import paper_2007_12856_amd as h3d
    _, xg = slab_pair(synth.flat("normal", SEED, 54, (1, 2, 6, 4, 8)), "bf16")
    _, yg = slab_pair(np.zeros((1, 2, 3, 2, 4)), "bf16")
    import torch
    buf = torch.empty(2 * 2 * 4 * 8, dtype=torch.bfloat16, device="cuda")
    with pytest.raises(h3d.H3DError) as e:
        h3d.halo_pack(xg.planes(0, 4), h3d.FACE_D_LO, 1, buf)
    assert e.value.status == -2
    with pytest.raises(h3d.H3DError) as e:
        x4 = h3d.Slab(torch.zeros((2, 4, 6, 4, 8), dtype=torch.bfloat16, device="cuda"))      # (one sample: its first channels are packed memory)
        h3d.concat_c(x4.channels(0, 2), x4.channels(2, 4), h3d.Slab(torch.empty_like(x4.t)))
    assert e.value.status == -2


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_halo_recompute_two_stacked_convs(dtype):
    """A 2-plane halo serves two stacked convolutions (U-Net-shaped level): the first also produces
    its output's halo plane; beyond the global boundary that plane must be zero, not act(bias)."""
    import paper_2007_12856_amd as h3d
    Ci, Cm, Co, Dg, H, W, d = 1, 8, 16, 8, 12, 20, 4
    wa, ba = _weights(Ci, Cm, dtype, 40)
    wb, bb = _weights(Cm, Co, dtype, 42)
    for off in (0, 4):
        xs = cut("normal", SEED, 7, (1, Ci, Dg, H, W), off, d, (2, 2))
        xo, xg = slab_pair(xs, dtype, (2, 2), off, Dg)
        ao = orc.conv3d_fwd(xo, wa, ba, cout_halo=(1, 1), act=orc.ACT_RELU)
        ag = h3d.conv3d_fwd(xg, to_dev(wa, dtype), to_dev(ba, "f32"), dev_like(ao, dtype), h3d.ACT_RELU, 0.0)
        close(from_dev(ag.t), ao.a, TOL[dtype])
        outside = 0 if off == 0 else -1
        assert not from_dev(ag.t)[:, :, outside].any()
        aqo, aqg = slab_pair(ao.a, dtype, (1, 1), off, Dg)
        bo = orc.conv3d_fwd(aqo, wb, bb, act=orc.ACT_RELU)
        bg = h3d.conv3d_fwd(aqg, to_dev(wb, dtype), to_dev(bb, "f32"), dev_like(bo, dtype), h3d.ACT_RELU, 0.0)
        close(from_dev(bg.t), bo.a, TOL[dtype])


def test_error_paths_do_not_launch():
    import torch
    import paper_2007_12856_amd as h3d
    x = h3d.Slab(torch.zeros((1, 2, 4, 4, 4), device="cuda"), 0, 0, 4, 16)      # interior shard without halo
    z = x.like(3)
    w = torch.zeros((3, 2, 3, 3, 3), device="cuda")
    with pytest.raises(h3d.H3DError) as e:
        h3d.conv3d_fwd(x, w, None, z)
    assert e.value.status == -4
    zbad = h3d.Slab(torch.zeros((1, 3, 4, 4, 5), device="cuda"), 0, 0, 4, 16)
    with pytest.raises(h3d.H3DError) as e:
        h3d.conv3d_fwd(x, w, None, zbad)
    assert e.value.status == -1
    with pytest.raises(h3d.H3DError) as e:
        h3d.conv3d_fwd(h3d.Slab(torch.zeros((1, 2, 4, 4, 4), device="cuda")), w, None,
                       h3d.Slab(torch.zeros((1, 3, 4, 4, 4), device="cuda")), act=7)
    assert e.value.status == -1
    # workspace too small is reported, not overrun
    import ctypes
    xd, zd = h3d.Slab(torch.zeros((1, 2, 4, 4, 4), device="cuda")), h3d.Slab(torch.zeros((1, 3, 4, 4, 4), device="cuda"))
    st = h3d.lib().h3d_conv3d_fwd(h3d.handle(), ctypes.byref(xd.desc()), ctypes.c_void_p(w.data_ptr()), None,
                                  ctypes.byref(zd.desc()), 0, 0.0, None, 0, None)
    assert st == -3


def test_empty_shard():
    import torch
    import paper_2007_12856_amd as h3d
    x = h3d.Slab(torch.zeros((0, 2, 4, 4, 4), device="cuda"))
    z = h3d.Slab(torch.zeros((0, 3, 4, 4, 4), device="cuda"))
    w = torch.ones((3, 2, 3, 3, 3), device="cuda")
    h3d.conv3d_fwd(x, w, None, z)
    dw = torch.full((3, 2, 3, 3, 3), 5.0, device="cuda")
    db = torch.full((3,), 5.0, device="cuda")
    h3d.conv3d_bwd_filter(x, z, None, dw, db)
    torch.cuda.synchronize()
    assert not dw.any() and not db.any()
