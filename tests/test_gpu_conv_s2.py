"""GPU parity of the stride-2 3x3x3 convolution (Table I, fourth convolution) against the CPU oracle:
all three passes, unsharded and on depth shards with the halo sides each direction needs, fp32 and bf16,
odd H / W, channel counts that divide nothing, canaries on what must not be written."""
import numpy as np
import pytest

import oracle as orc
import synth
from helpers import TOL, cut, dev_like, elem_masked_bf, from_dev, quantize, close, rel_l2, slab_pair, to_dev

pytestmark = pytest.mark.gpu
SEED = synth.BASE_SEED

# (N, Cin, Cout, Dg, H, W)
SHAPES = [
    (1, 64, 128, 8, 8, 8),       # the layer's channel counts on a small volume
    (2, 3, 5, 4, 7, 9),          # odd H and W, nothing divides anything
    (1, 16, 32, 6, 12, 40),
    (1, 8, 16, 2, 2, 2),         # a single output voxel
    (1, 4, 16, 4, 16, 64),
]


def _weights(cin, cout, dtype, stream):
    b = np.sqrt(3.0 / (27 * cin))
    w = quantize(synth.flat("uniform", SEED, stream, (cout, cin, 3, 3, 3), -b, b), dtype)
    bias = synth.round_f32(synth.flat("uniform", SEED, stream + 1, (cout,), -0.1, 0.1)).astype(np.float64)
    return w, bias


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", SHAPES)
def test_stride2_three_passes_unsharded(shape, dtype):
    import torch
    import paper_2007_12856_amd as h3d
    N, Ci, Co, D, H, W = shape
    alpha = 0.01
    w, bias = _weights(Ci, Co, dtype, 310)
    wd, bd = to_dev(w, dtype), to_dev(bias, "f32")
    xo, xg = slab_pair(synth.flat("uniform", SEED, 301, (N, Ci, D, H, W)), dtype)
    yo = orc.conv3d_s2_fwd(xo, w, bias, orc.ACT_LEAKY, alpha)
    yg = h3d.conv3d_s2_fwd(xg, wd, bd, dev_like(yo, dtype), h3d.ACT_LEAKY, alpha)
    close(from_dev(yg.t), yo.a, TOL[dtype])
    yq_o, yq_g = slab_pair(yo.a, dtype)
    dyo, dyg = slab_pair(synth.flat("uniform", SEED, 302, yo.a.shape), dtype)
    dxo = orc.conv3d_s2_bwd_data(dyo, yq_o, w, xo, orc.ACT_LEAKY, alpha)
    dxg = h3d.conv3d_s2_bwd_data(dyg, yq_g, wd, dev_like(dxo, dtype), h3d.ACT_LEAKY, alpha)
    close(from_dev(dxg.t), dxo.a, TOL[dtype])
    dwo, dbo = orc.conv3d_s2_bwd_filter(xo, dyo, yq_o, orc.ACT_LEAKY, alpha)
    dw = torch.full((Co, Ci, 3, 3, 3), 777.0, device="cuda")
    db = torch.full((Co,), 777.0, device="cuda")
    h3d.conv3d_s2_bwd_filter(xg, dyg, yq_g, dw, db, h3d.ACT_LEAKY, alpha)
    tol_w = 1e-5 if dtype == "f32" else 2e-4
    close(from_dev(dw), dwo, tol_w, elem=elem_masked_bf(dtype))
    close(from_dev(db), dbo, tol_w, elem=elem_masked_bf(dtype))
    dw2, db2 = torch.empty_like(dw), torch.empty_like(db)
    h3d.conv3d_s2_bwd_filter(xg, dyg, yq_g, dw2, db2, h3d.ACT_LEAKY, alpha)
    assert torch.equal(dw, dw2) and torch.equal(db, db2)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("act", [orc.ACT_NONE, orc.ACT_RELU])
def test_stride2_no_bias_other_activations(dtype, act):
    import torch
    import paper_2007_12856_amd as h3d
    N, Ci, Co, D, H, W = 1, 8, 16, 4, 6, 20
    w, _ = _weights(Ci, Co, dtype, 320)
    wd = to_dev(w, dtype)
    xo, xg = slab_pair(synth.flat("normal", SEED, 303, (N, Ci, D, H, W)), dtype)
    yo = orc.conv3d_s2_fwd(xo, w, None, act)
    yg = h3d.conv3d_s2_fwd(xg, wd, None, dev_like(yo, dtype), act, 0.0)
    close(from_dev(yg.t), yo.a, TOL[dtype])
    yq_o, yq_g = slab_pair(yo.a, dtype)
    dyo, dyg = slab_pair(synth.flat("normal", SEED, 304, yo.a.shape), dtype)
    dxo = orc.conv3d_s2_bwd_data(dyo, yq_o, w, xo, act)
    dxg = h3d.conv3d_s2_bwd_data(dyg, yq_g, wd, dev_like(dxo, dtype), act, 0.0)
    close(from_dev(dxg.t), dxo.a, TOL[dtype])
    dwo, _ = orc.conv3d_s2_bwd_filter(xo, dyo, yq_o, act)
    dw = torch.full((Co, Ci, 3, 3, 3), 777.0, device="cuda")
    h3d.conv3d_s2_bwd_filter(xg, dyg, yq_g, dw, None, act, 0.0)
    close(from_dev(dw), dwo, (1e-5 if dtype == "f32" else 2e-4))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shard", [0, 1, 3])
def test_stride2_on_depth_shards(shard, dtype):
    """4-way depth partition of a 1 x 8 x 16 x 10 x 24 sample: forward and backward-filter read the lower halo
    of x, backward-data the upper halo of dy and y; outputs carry halos that must stay untouched."""
    import torch
    import paper_2007_12856_amd as h3d
    N, Ci, Co, Dg, H, W = 1, 8, 16, 16, 10, 24
    d, alpha = Dg // 4, 0.01
    off = shard * d
    w, bias = _weights(Ci, Co, dtype, 330)
    wd, bd = to_dev(w, dtype), to_dev(bias, "f32")
    full_x = (N, Ci, Dg, H, W)
    full_y = (N, Co, Dg // 2, H // 2, W // 2)
    # forward: x with halo 1/1 (the upper one is never read: poison it), y with halos 1/1 holding canaries
    xa = cut("uniform", SEED, 305, full_x, off, d, (1, 1))
    xa[:, :, -1] = np.nan
    xo, xg = slab_pair(xa, dtype, (1, 1), off, Dg)
    yo = orc.conv3d_s2_fwd(xo, w, bias, orc.ACT_LEAKY, alpha)
    yg = h3d.Slab(torch.full((N, Co, d // 2 + 2, H // 2, W // 2), 12345.0, device="cuda",
                             dtype=torch.float32 if dtype == "f32" else torch.bfloat16), 1, 1, off // 2, Dg // 2)
    h3d.conv3d_s2_fwd(xg, wd, bd, yg, h3d.ACT_LEAKY, alpha)
    got = from_dev(yg.t)
    close(got[:, :, 1:-1], yo.a, TOL[dtype])
    assert np.all(got[:, :, 0] == from_dev(torch.full((1,), 12345.0, device="cuda", dtype=yg.t.dtype))[0])
    assert np.all(got[:, :, -1] == got[0, 0, 0, 0, 0])
    # backward: dy and the saved y with halo 0/1 cut from the seeded full tensors; lower halos absent
    dya = cut("uniform", SEED, 306, full_y, off // 2, d // 2, (0, 1))
    ya = cut("normal", SEED, 307, full_y, off // 2, d // 2, (0, 1))
    dyo, dyg = slab_pair(dya, dtype, (0, 1), off // 2, Dg // 2)
    yso, ysg = slab_pair(ya, dtype, (0, 1), off // 2, Dg // 2)
    xin = orc.Slab(xo.interior, 0, 0, off, Dg)
    dxo = orc.conv3d_s2_bwd_data(dyo, yso, w, xin, orc.ACT_LEAKY, alpha)
    dxg = h3d.conv3d_s2_bwd_data(dyg, ysg, wd, dev_like(dxo, dtype), h3d.ACT_LEAKY, alpha)
    close(from_dev(dxg.t), dxo.a, TOL[dtype])
    dwo, dbo = orc.conv3d_s2_bwd_filter(xo, dyo, yso, orc.ACT_LEAKY, alpha)
    dw = torch.full((Co, Ci, 3, 3, 3), 777.0, device="cuda")
    db = torch.full((Co,), 777.0, device="cuda")
    h3d.conv3d_s2_bwd_filter(xg, dyg, ysg, dw, db, h3d.ACT_LEAKY, alpha)
    tol_w = 1e-5 if dtype == "f32" else 2e-4
    close(from_dev(dw), dwo, tol_w, elem=elem_masked_bf(dtype))
    close(from_dev(db), dbo, tol_w, elem=elem_masked_bf(dtype))


def test_stride2_errors_do_not_launch():
    import ctypes
    import torch
    import paper_2007_12856_amd as h3d
    w = torch.zeros((3, 2, 3, 3, 3), device="cuda")
    x = h3d.Slab(torch.zeros((1, 2, 4, 4, 4), device="cuda"), 0, 0, 4, 16)       # interior shard, no lower halo
    y = h3d.Slab(torch.zeros((1, 3, 2, 2, 2), device="cuda"), 0, 0, 2, 8)
    with pytest.raises(h3d.H3DError) as e:
        h3d.conv3d_s2_fwd(x, w, None, y)
    assert e.value.status == -4
    with pytest.raises(h3d.H3DError) as e:                                       # dy without its upper halo
        h3d.conv3d_s2_bwd_data(y, None, w, x)
    assert e.value.status == -4
    xodd = h3d.Slab(torch.zeros((1, 2, 3, 4, 4), device="cuda"))
    with pytest.raises(h3d.H3DError) as e:
        h3d.conv3d_s2_fwd(xodd, w, None, h3d.Slab(torch.zeros((1, 3, 1, 2, 2), device="cuda")))
    assert e.value.status == -2
    xs = h3d.Slab(torch.zeros((1, 2, 4, 4, 4), device="cuda"))
    with pytest.raises(h3d.H3DError) as e:                                       # wrong output extents
        h3d.conv3d_s2_fwd(xs, w, None, h3d.Slab(torch.zeros((1, 3, 2, 2, 3), device="cuda")))
    assert e.value.status == -1
    ys = h3d.Slab(torch.zeros((1, 3, 2, 2, 2), device="cuda"))
    st = h3d.lib().h3d_conv3d_s2_fwd(h3d.handle(), ctypes.byref(xs.desc()), ctypes.c_void_p(w.data_ptr()), None,
                                     ctypes.byref(ys.desc()), 0, 0.0, None, 0, None)
    assert st == -3


def test_stride2_empty_shard():
    import torch
    import paper_2007_12856_amd as h3d
    x = h3d.Slab(torch.zeros((1, 2, 0, 4, 4), device="cuda"), 0, 0, 0, 8)
    y = h3d.Slab(torch.zeros((1, 3, 0, 2, 2), device="cuda"), 0, 0, 0, 4)
    w = torch.zeros((3, 2, 3, 3, 3), device="cuda")
    h3d.conv3d_s2_fwd(x, w, None, y)
    dw = torch.full((3, 2, 3, 3, 3), 5.0, device="cuda")
    h3d.conv3d_s2_bwd_filter(x, y, None, dw, None)
    torch.cuda.synchronize()
    assert float(dw.abs().max()) == 0.0


@pytest.mark.parametrize("act", [orc.ACT_NONE, orc.ACT_LEAKY])
@pytest.mark.parametrize("shape", [
    (1, 33, 70, 4, 18, 70),      # 35 coarse columns: a second column tile of three; one channel / six channels past a block
    (2, 16, 40, 2, 10, 144),     # aligned rows (16-byte loads), three column tiles, the middle form of the forward kernel
    (1, 70, 130, 2, 6, 16),      # a second group of output channels, a third 32-channel stage of one partial half
    (1, 5, 24, 4, 70, 34),       # 35 coarse rows: three bands of the filter gradient, nine row tiles
    (3, 17, 65, 2, 3, 15),       # odd extents: rows that start at odd addresses, a group that ends past the last row
])
def test_stride2_bf16_tile_edges(shape, act):
    """The edges of the direct kernels' tiles, channel blocks and row groups, against the oracle (the bars of the tests above)."""
    import torch
    import paper_2007_12856_amd as h3d
    N, Ci, Co, D, H, W = shape
    w, bias = _weights(Ci, Co, "bf16", 340)
    wd, bd = to_dev(w, "bf16"), to_dev(bias, "f32")
    xo, xg = slab_pair(synth.flat("normal", SEED, 341, (N, Ci, D, H, W)), "bf16")
    yo = orc.conv3d_s2_fwd(xo, w, bias, act, 0.01)
    yg = h3d.conv3d_s2_fwd(xg, wd, bd, dev_like(yo, "bf16"), act, 0.01)
    assert h3d.h3d_last_kernel().startswith("s2_fwd_kernel")
    close(from_dev(yg.t), yo.a, TOL["bf16"])
    so, sg = slab_pair(synth.flat("normal", SEED, 342, yo.a.shape), "bf16")
    dyo, dyg = slab_pair(synth.flat("normal", SEED, 343, yo.a.shape), "bf16")
    dxo = orc.conv3d_s2_bwd_data(dyo, so, w, xo, act, 0.01)
    dxg = h3d.conv3d_s2_bwd_data(dyg, sg, wd, dev_like(dxo, "bf16"), act, 0.01)
    close(from_dev(dxg.t), dxo.a, TOL["bf16"])
    dwo, dbo = orc.conv3d_s2_bwd_filter(xo, dyo, so, act, 0.01)
    dw, db = torch.empty((Co, Ci, 3, 3, 3), device="cuda"), torch.empty((Co,), device="cuda")
    h3d.conv3d_s2_bwd_filter(xg, dyg, sg, dw, db, act, 0.01)
    close(from_dev(dw), dwo, 2e-4, elem=elem_masked_bf("bf16"))
    close(from_dev(db), dbo, 2e-4, elem=elem_masked_bf("bf16"))


@pytest.mark.parametrize("shape", [
    (1, 20, 16, 4, 16, 32),      # one chunk of 16 output channels: nothing is requested behind it
    (1, 36, 65, 4, 18, 80),      # five, the last with one channel; two column tiles, a second row tile and channel block
    (2, 8, 96, 2, 16, 144),      # six, three column tiles
    (1, 8, 33, 2, 16, 20),       # rows that are no multiple of eight: the column behind a tile by a load that runs on
])
def test_stride2_bwd_data_chunks(shape):
    """Backward-data over one to six chunks of output channels, with and without a mask, against the oracle."""
    import torch
    import paper_2007_12856_amd as h3d
    N, Ci, Co, D, H, W = shape
    w, _ = _weights(Ci, Co, "bf16", 350)
    wd = to_dev(w, "bf16")
    xo, _ = slab_pair(np.zeros((N, Ci, D, H, W)), "bf16")
    coarse = (N, Co, D // 2, H // 2, W // 2)
    so, sg = slab_pair(synth.flat("normal", SEED, 351, coarse), "bf16")
    dyo, dyg = slab_pair(synth.flat("normal", SEED, 352, coarse), "bf16")
    for act in (orc.ACT_NONE, orc.ACT_LEAKY):
        dxo = orc.conv3d_s2_bwd_data(dyo, so, w, xo, act, 0.01)
        dxg = h3d.conv3d_s2_bwd_data(dyg, sg, wd, dev_like(dxo, "bf16"), act, 0.01)
        assert h3d.h3d_last_kernel() == f"s2_bwd_data_kernel<{int(act != orc.ACT_NONE)},{int(W // 2 % 8 == 0)}>"
        close(from_dev(dxg.t), dxo.a, TOL["bf16"])


@pytest.mark.parametrize("shape", [(1, 32, 32, 4, 16, 64), (1, 20, 40, 4, 70, 70), (2, 16, 32, 4, 9, 33), (1, 64, 32, 2, 34, 130)])
def test_stride2_an_infinity_reaches_only_the_taps_that_read_it(shape):
    """bf16 backward-filter: an infinite voxel of x next to the end of a row, column or plane makes the entries of dw infinite whose sums
    contain it and no others (the kernel's rows and columns of g beyond the volume are zeros, and zero times infinity is not)."""
    import torch
    import paper_2007_12856_amd as h3d
    N, Ci, Co, D, H, W = shape
    gen = torch.Generator(device="cuda").manual_seed(H + W)
    x = torch.randn((N, Ci, D, H, W), device="cuda", generator=gen).bfloat16()
    dy = (torch.rand((N, Co, D // 2, (H + 1) // 2, (W + 1) // 2), device="cuda", generator=gen) + 0.5).bfloat16()
    dw, db = torch.empty((Co, Ci, 3, 3, 3), device="cuda"), torch.empty((Co,), device="cuda")
    for d, h, w in [(D - 1, H - 1, W - 1), (D - 1, H - 1, 0), (0, 0, W - 1), (1, H - 2, W - 2), (D // 2, H // 2, W // 2), (1, 31, 63)]:
        if h >= H or w >= W:
            continue
        xi = x.clone()
        xi[N - 1, 1, d, h, w] = float("inf")
        h3d.conv3d_s2_bwd_filter(h3d.Slab(xi), h3d.Slab(dy), None, dw, db)
        # tap k of an axis reads position q if 2 p + k - 1 = q for an output position p
        reads = [[any(2 * p + k - 1 == q for p in range((e + 1) // 2)) for k in range(3)] for q, e in ((d, D), (h, H), (w, W))]
        expect = torch.zeros((Co, Ci, 3, 3, 3), dtype=torch.bool)
        expect[:, 1] = torch.tensor([[[a and b and c for c in reads[2]] for b in reads[1]] for a in reads[0]])
        assert torch.equal(~torch.isfinite(dw).cpu(), expect), (d, h, w)


@pytest.mark.parametrize("shape,planes", [((1, 32, 1, 2, 2, 8), 0), ((2, 3, 1, 2, 2, 10), 0), ((2, 5, 1, 4, 16, 16), 1 << 18), ((1, 17, 5, 2, 6, 10), 1118482)])
def test_stride2_saved_output_stored_unlike_the_gradient(shape, planes):
    """bf16 backward passes whose saved output stores fewer elements a sample than a 16-byte load takes, or (behind `planes` planes of
    halo that nobody reads) more than 32-bit offsets reach, in the workspace that the size query names: it does not see the saved output."""
    import torch
    import paper_2007_12856_amd as h3d
    N, Ci, Co, D, H, W = shape
    print("s2 far mask", shape, planes, flush=True)
    w, _ = _weights(Ci, Co, "bf16", 350)
    # the upper shard of two: the lower halo planes exist, the upper ones do not
    xo, xg = slab_pair(synth.flat("normal", SEED, 351, (N, Ci, D + 1, H, W)), "bf16", (1, 0), D, 2 * D)
    coarse = (N, Co, D // 2, H // 2, W // 2)
    dya = np.zeros((N, Co, D // 2 + 1) + coarse[3:])
    dya[:, :, 1:] = synth.flat("normal", SEED, 352, coarse)
    dyo, dyg = slab_pair(dya, "bf16", (1, 0), D // 2, D)
    so, sg = slab_pair(synth.flat("normal", SEED, 353, coarse), "bf16", (0, 0), D // 2, D)
    if planes:
        tall = torch.zeros((N, Co, planes + D // 2) + coarse[3:], dtype=torch.bfloat16, device="cuda")
        tall[:, :, planes:] = sg.t
        sg = h3d.Slab(tall, planes, 0, D // 2, D)
        assert 64 * tall.stride(1) >= 1 << 30      # (a workgroup's offsets reach over 64 channels)
    else:
        assert sg.t[0].numel() < 8 <= dyg.t[0].numel()
    ws = h3d.Workspace()
    dxo = orc.conv3d_s2_bwd_data(dyo, so, w, orc.Slab(xo.interior, 0, 0, D, 2 * D), orc.ACT_LEAKY, 0.01)
    dxg = h3d.conv3d_s2_bwd_data(dyg, sg, to_dev(w, "bf16"), dev_like(dxo, "bf16"), h3d.ACT_LEAKY, 0.01, ws)
    close(from_dev(dxg.t), dxo.a, TOL["bf16"])
    dwo, dbo = orc.conv3d_s2_bwd_filter(xo, dyo, so, orc.ACT_LEAKY, 0.01)
    dw, db = torch.empty((Co, Ci, 3, 3, 3), device="cuda"), torch.empty((Co,), device="cuda")
    ws = h3d.Workspace()
    h3d.conv3d_s2_bwd_filter(xg, dyg, sg, dw, db, h3d.ACT_LEAKY, 0.01, ws)
    close(from_dev(dw), dwo, 2e-4, elem=elem_masked_bf("bf16"))
    close(from_dev(db), dbo, 2e-4, elem=elem_masked_bf("bf16"))


@pytest.mark.parametrize("shape,fwd,filt", [
    # N, Cin, Cout, D, H, W; does forward / the filter gradient run on the direct kernels?
    ((1, 1, 16, 12, 64, 62), True, True),
    ((1, 1, 40, 12, 64, 64), True, False),
    ((1, 1, 4, 64, 96, 128), False, False),
    ((1, 1, 8, 24, 128, 130), False, False),
    ((1, 1, 64, 24, 128, 120), True, False),
    ((1, 1, 64, 26, 128, 120), False, False),
    ((2, 2, 16, 16, 56, 64), True, False),
    ((1, 3, 48, 16, 64, 160), True, True),
    ((1, 4, 16, 8, 160, 160), True, False),
    ((1, 4, 24, 8, 160, 160), True, True),
    ((1, 16, 16, 16, 32, 32), True, True),      # bands of four rows
    ((1, 16, 40, 4, 66, 64), True, True),       # bands of eight, the last of one row
])
def test_stride2_routes_of_few_input_channels(shape, fwd, filt):
    """Either side of the sizes from which the rewriting is the faster route for a first layer, and the band heights of small layers."""
    import torch
    import paper_2007_12856_amd as h3d
    N, Ci, Co, D, H, W = shape
    w, bias = _weights(Ci, Co, "bf16", 360)
    xo, xg = slab_pair(synth.flat("normal", SEED, 361, (N, Ci, D, H, W)), "bf16")
    yo = orc.conv3d_s2_fwd(xo, w, bias, orc.ACT_LEAKY, 0.01)
    yg = h3d.conv3d_s2_fwd(xg, to_dev(w, "bf16"), to_dev(bias, "f32"), dev_like(yo, "bf16"), h3d.ACT_LEAKY, 0.01)
    assert h3d.h3d_last_kernel().startswith("s2_fwd_kernel") == fwd
    close(from_dev(yg.t), yo.a, TOL["bf16"])
    so, sg = slab_pair(synth.flat("normal", SEED, 362, yo.a.shape), "bf16")
    dyo, dyg = slab_pair(synth.flat("normal", SEED, 363, yo.a.shape), "bf16")
    dwo, dbo = orc.conv3d_s2_bwd_filter(xo, dyo, so, orc.ACT_LEAKY, 0.01)
    dw, db = torch.empty((Co, Ci, 3, 3, 3), device="cuda"), torch.empty((Co,), device="cuda")
    h3d.conv3d_s2_bwd_filter(xg, dyg, sg, dw, db, h3d.ACT_LEAKY, 0.01)
    assert h3d.h3d_last_kernel().startswith("s2_bwd_filter_kernel") == filt
    close(from_dev(dw), dwo, 2e-4, elem=elem_masked_bf("bf16"))
    close(from_dev(db), dbo, 2e-4, elem=elem_masked_bf("bf16"))
