"""Seeded sweep of small random shapes through the three convolution passes (with and without the fused activation
mask, with and without halos, packed and as plane-run views) and the transposed convolution, against the oracle.
The shapes are drawn so that every kernel family is reached: first-layer kernels (Cin <= 4), the few-channel
kernel (<= 8 output channels), 16/32-channel workgroups, narrow (W <= 16) and wide volumes, ragged H / W / channels."""
import numpy as np
import pytest

import oracle as orc
import synth
from helpers import TOL, dev_like, from_dev, quantize, close, rel_l2, slab_pair, to_dev

pytestmark = pytest.mark.gpu
SEED = synth.BASE_SEED


def _cases(n, seed):
    rng = np.random.default_rng(seed)
    chans = [1, 2, 3, 4, 5, 8, 12, 16, 17, 24, 32, 33, 40, 48, 64, 72]
    widths = [4, 8, 12, 16, 24, 32, 33, 40, 48, 64, 72]
    out = []
    for i in range(n):
        cin, cout = int(rng.choice(chans)), int(rng.choice(chans))
        W = int(rng.choice(widths))
        H = int(rng.integers(2, 13)) if W > 16 else int(rng.integers(2, 20))
        D = int(rng.integers(1, 6))
        N = int(rng.integers(1, 3))
        halo = int(rng.integers(0, 2))
        # keep the oracle's direct loops under a second per case
        if N * D * H * W * cin * cout > 3_000_000:
            N, D = 1, min(D, 2)
        out.append((i, N, cin, cout, D, H, W, halo, bool(rng.integers(0, 2))))
    return out


@pytest.mark.parametrize("case", _cases(36, 2007), ids=lambda c: "c%d_%dx%d-%d_%dx%dx%d_h%d_m%d" % (c[0], c[1], c[2], c[3], c[4], c[5], c[6], c[7], c[8]))
def test_conv_sweep_bf16(case):
    import torch
    import paper_2007_12856_amd as h3d
    i, N, cin, cout, D, H, W, halo, masked = case
    dtype = "bf16"
    b = np.sqrt(3.0 / (27 * cin))
    w = quantize(synth.flat("uniform", SEED, 1000 + i, (cout, cin, 3, 3, 3), -b, b), dtype)
    bias = synth.round_f32(synth.flat("uniform", SEED, 2000 + i, (cout,), -0.1, 0.1)).astype(np.float64)
    Dg, off = (D + 2, 1) if halo else (D, 0)
    xo, xg = slab_pair(synth.flat("normal", SEED, 3000 + i, (N, cin, D + 2 * halo, H, W)), dtype, (halo, halo), off, Dg)
    wd, bd = to_dev(w, dtype), to_dev(bias, "f32")
    act = orc.ACT_LEAKY if masked else orc.ACT_NONE
    zo = orc.conv3d_fwd(xo, w, bias, act=act, alpha=0.01)
    zg = h3d.conv3d_fwd(xg, wd, bd, dev_like(zo, dtype), act, 0.01)
    close(from_dev(zg.t), zo.a, TOL[dtype])
    # the backward passes take ANY saved output as the activation mask: a seeded one with the halo dz is read at
    zm_o, zm_g = slab_pair(synth.flat("normal", SEED, 6000 + i, (N, cout, D + 2 * halo, H, W)), dtype, (halo, halo), off, Dg)
    zq_o, zq_g = slab_pair(zm_o.interior, dtype, (0, 0), off, Dg)
    # gradient of the layer's output with a halo of its own (neighbouring shards' planes), as backward-data needs it
    go, gg = slab_pair(synth.flat("normal", SEED, 4000 + i, (N, cout, D + 2 * halo, H, W)), dtype, (halo, halo), off, Dg)
    if masked:
        dxo = orc.conv3d_bwd_data(go, zm_o, w, act=act, alpha=0.01)
        dxg = h3d.conv3d_bwd_data(gg, zm_g, wd, dev_like(dxo, dtype), act, 0.01)
    else:
        dxo = orc.conv3d_bwd_data(go, None, w, act=orc.ACT_NONE)
        dxg = h3d.conv3d_bwd_data(gg, None, wd, dev_like(dxo, dtype), h3d.ACT_NONE, 0.0)
    close(from_dev(dxg.t), dxo.a, TOL[dtype])
    g0o, g0g = slab_pair(go.interior, dtype, (0, 0), off, Dg)
    dwo, dbo = orc.conv3d_bwd_filter(xo, g0o, zq_o if masked else None, act=act, alpha=0.01)
    dw = torch.full((cout, cin, 3, 3, 3), 7.0, device="cuda")
    db = torch.full((cout,), 7.0, device="cuda")
    h3d.conv3d_bwd_filter(xg, g0g, zq_g if masked else None, dw, db, act, 0.01)
    close(from_dev(dw), dwo, 2e-4)
    close(from_dev(db), dbo, 2e-4)
    # the same forward on a plane-run view of the middle planes (when there are at least three)
    if D >= 3:
        part = dev_like(zo, dtype)
        part.t.zero_()
        h3d.conv3d_fwd(xg.planes(1, D - 1, 1, 1), wd, bd, part.planes(1, D - 1), act, 0.01)
        close(from_dev(part.t[:, :, 1:D - 1]), zo.a[:, :, 1:D - 1], TOL[dtype])
        assert float(part.t[:, :, 0].abs().max()) == 0.0 and float(part.t[:, :, D - 1].abs().max()) == 0.0


@pytest.mark.parametrize("case", [(0, 1, 8, 12, 2, 3, 8), (1, 2, 33, 7, 1, 5, 16), (2, 1, 64, 64, 2, 4, 24), (3, 1, 128, 32, 1, 2, 40),
                                  (4, 1, 96, 48, 2, 2, 8), (5, 2, 16, 16, 3, 6, 32)])
def test_deconv_sweep_bf16(case):
    import torch
    import paper_2007_12856_amd as h3d
    i, N, cin, cout, d, H, W = case
    dtype = "bf16"
    b = np.sqrt(3.0 / (8 * cin))
    w = quantize(synth.flat("uniform", SEED, 5000 + i, (cin, cout, 2, 2, 2), -b, b), dtype)
    bias = synth.round_f32(synth.flat("uniform", SEED, 5100 + i, (cout,), -0.1, 0.1)).astype(np.float64)
    xo, xg = slab_pair(synth.flat("normal", SEED, 5200 + i, (N, cin, d, H, W)), dtype, (0, 0), 1, d + 3)
    yo = orc.deconv2_fwd(xo, w, bias)
    yg = h3d.deconv2_fwd(xg, to_dev(w, dtype), to_dev(bias, "f32"), dev_like(yo, dtype))
    close(from_dev(yg.t), yo.a, TOL[dtype])
    dyo, dyg = slab_pair(synth.flat("normal", SEED, 5300 + i, yo.a.shape), dtype, (0, 0), yo.d_offset, yo.d_global)
    dxo = orc.deconv2_bwd_data(dyo, w)
    dxg = h3d.deconv2_bwd_data(dyg, to_dev(w, dtype), dev_like(dxo, dtype))
    close(from_dev(dxg.t), dxo.a, TOL[dtype])
    dwo, dbo = orc.deconv2_bwd_filter(xo, dyo)
    dw, db = torch.empty((cin, cout, 2, 2, 2), device="cuda"), torch.empty((cout,), device="cuda")
    h3d.deconv2_bwd_filter(xg, dyg, dw, db)
    close(from_dev(dw), dwo, 2e-4)
    close(from_dev(db), dbo, 2e-4)


@pytest.mark.parametrize("N,cin,cout,d,H,W,fast", [(1, 17, 65, 2, 3, 8, True), (2, 64, 96, 1, 5, 40, True), (1, 70, 128, 2, 3, 33, True), (1, 20, 129, 3, 2, 31, True),
                                                   (1, 9, 200, 2, 4, 16, False), (1, 15, 66, 2, 4, 16, False), (1, 16, 66, 2, 4, 16, True), (1, 16, 72, 2, 5, 14, True),
                                                   (1, 15, 72, 2, 5, 14, False), (2, 7, 65, 16, 48, 64, False), (2, 8, 65, 16, 48, 64, True), (1, 130, 66, 1, 3, 8, False)])
def test_deconv_forward_of_more_than_64_output_channels(N, cin, cout, d, H, W, fast):
    """Groups of 64 output channels, the last one with few of them, whole and ragged rows; nothing is written around the result."""
    import torch
    import paper_2007_12856_amd as h3d
    b = np.sqrt(3.0 / (8 * cin))
    w = quantize(synth.flat("uniform", SEED, 6000 + cout, (cin, cout, 2, 2, 2), -b, b), "bf16")
    bias = synth.round_f32(synth.flat("uniform", SEED, 6100 + cout, (cout,), -0.1, 0.1)).astype(np.float64)
    xo, xg = slab_pair(synth.flat("normal", SEED, 6200 + cout, (N, cin, d, H, W)), "bf16")
    yo = orc.deconv2_fwd(xo, w, bias)
    n = yo.a.size
    buf = torch.full((n + 64,), 3.0, dtype=torch.bfloat16, device="cuda")
    y = h3d.Slab(buf[32:32 + n].view(yo.a.shape), 0, 0, yo.d_offset, yo.d_global)
    h3d.deconv2_fwd(xg, to_dev(w, "bf16"), to_dev(bias, "f32"), y)
    assert h3d.h3d_last_kernel().startswith("deconv_fw_mfma_kernel") == fast, h3d.h3d_last_kernel()
    close(from_dev(y.t), yo.a, TOL["bf16"])
    assert torch.all(buf[:32] == 3.0) and torch.all(buf[32 + n:] == 3.0)


@pytest.mark.parametrize("cin,cout", [(17, 65), (64, 96), (128, 200)])
def test_deconv_forward_at_scratch_limits(cin, cout):
    """A workspace at an address of a float only, or with no more room than the direct kernel's filter: such calls run on the direct kernel; with less they are
    refused, as is a misaligned workspace of at most 64 output channels."""
    import torch
    import paper_2007_12856_amd as h3d
    xo, xg = slab_pair(synth.flat("normal", SEED, 6500 + cout, (1, cin, 2, 3, 8)), "bf16")
    b = np.sqrt(3.0 / (8 * cin))
    w = quantize(synth.flat("uniform", SEED, 6600 + cout, (cin, cout, 2, 2, 2), -b, b), "bf16")
    yo = orc.deconv2_fwd(xo, w, np.zeros(cout))
    wd, y = to_dev(w, "bf16"), dev_like(yo, "bf16")
    lib, xd, yd = h3d.lib(), xg.desc(), y.desc()
    direct, fragments = cin * -(-cout // 8) * 8 * 32, -(-cout // 4) * (8 if cin > 64 else 4) * 1024
    size = lib.h3d_deconv2_workspace_bytes(h3d.handle(), h3d.OP_FWD, xd, yd)
    assert size >= max(direct, fragments)
    buf = torch.empty(size + 16, dtype=torch.uint8, device="cuda")

    def call(shift, nbytes, yd=yd):
        st = lib.h3d_deconv2_fwd(h3d.handle(), xd, wd.data_ptr(), None, yd, buf.data_ptr() + shift, nbytes, None)
        torch.cuda.synchronize()
        return st

    for shift, nbytes in ((0, size), (4, size), (0, direct), (0, fragments)):
        fast = shift == 0 and nbytes >= fragments
        y.t.fill_(3.0)
        assert call(shift, nbytes) == (0 if fast or nbytes >= direct else -3), h3d.h3d_last_error()
        if fast or nbytes >= direct:
            assert h3d.h3d_last_kernel().startswith("deconv_fw_mfma_kernel" if fast else "deconv2_fwd"), (shift, nbytes, h3d.h3d_last_kernel())
            close(from_dev(y.t), yo.a, TOL["bf16"])
    assert call(0, min(direct, fragments) - 1) == -3
    assert call(4, size, h3d.Slab(y.t[:, :64].contiguous()).desc()) == -3


@pytest.mark.parametrize("N,cin,cout,d,H,W,blocks", [(1, 129, 5, 2, 3, 8, 3), (2, 128, 78, 1, 5, 40, 4), (2, 128, 79, 1, 5, 40, 2), (1, 97, 110, 2, 3, 33, 2), (1, 70, 156, 2, 2, 34, 2),
                                                     (1, 40, 159, 3, 2, 31, 1), (1, 33, 310, 1, 2, 5, 1), (1, 20, 311, 1, 2, 5, 0), (1, 300, 17, 1, 4, 9, 4), (1, 1025, 3, 1, 2, 3, 0)])
def test_deconv_backward_data_in_groups_of_input_channels(N, cin, cout, d, H, W, blocks):
    """Blocks of 32 input channels that do not fit in one workgroup, the last group with few channels or none of a block; nothing is written around the result."""
    import torch
    import paper_2007_12856_amd as h3d
    b = np.sqrt(3.0 / (8 * cin))
    w = quantize(synth.flat("uniform", SEED, 6300 + cout, (cin, cout, 2, 2, 2), -b, b), "bf16")
    dyo, dyg = slab_pair(synth.flat("normal", SEED, 6400 + cout, (N, cout, 2 * d, 2 * H, 2 * W)), "bf16")
    dxo = orc.deconv2_bwd_data(dyo, w)
    n = dxo.a.size
    buf = torch.full((n + 64,), 3.0, dtype=torch.bfloat16, device="cuda")
    dx = h3d.Slab(buf[32:32 + n].view(dxo.a.shape), 0, 0, dxo.d_offset, dxo.d_global)
    h3d.deconv2_bwd_data(dyg, to_dev(w, "bf16"), dx)
    assert h3d.h3d_last_kernel() == (f"deconv_bd_mfma_kernel<{blocks},0>" if blocks else "deconv2_bwd_data"), h3d.h3d_last_kernel()
    close(from_dev(dx.t), dxo.a, TOL["bf16"])
    assert torch.all(buf[:32] == 3.0) and torch.all(buf[32 + n:] == 3.0)


@pytest.mark.parametrize("cin,cout", [(17, 66), (20, 40)])
def test_deconv_on_views_of_tall_tensors(cin, cout):
    """y (dy) is a run of planes of a tensor whose samples are past 31-bit byte offsets, on which neither matrix-core kernel runs; nothing is written around the run."""
    import torch
    import paper_2007_12856_amd as h3d
    d, H, W = 2, 3, 8
    g = torch.Generator(device="cuda").manual_seed(cin)
    x = h3d.Slab(torch.randn((1, cin, d, H, W), generator=g, device="cuda").bfloat16())
    w = (torch.rand((cin, cout, 2, 2, 2), generator=g, device="cuda") - 0.5).bfloat16()
    packed = h3d.Slab(torch.empty((1, cout, 2 * d, 2 * H, 2 * W), dtype=torch.bfloat16, device="cuda"))
    h3d.deconv2_fwd(x, w, None, packed)
    assert h3d.h3d_last_kernel().startswith("deconv_fw_mfma_kernel")
    tall = torch.full((1, cout, -(-2 ** 30 // (cout * 4 * H * W)), 2 * H, 2 * W), 3.0, dtype=torch.bfloat16, device="cuda")
    p0 = tall.shape[2] - 2 * d - 1
    view = h3d.Slab(tall[:, :, p0:p0 + 2 * d])
    h3d.deconv2_fwd(x, w, None, view)
    assert h3d.h3d_last_kernel() == "deconv2_fwd"
    close(from_dev(view.t), from_dev(packed.t), TOL["bf16"])
    assert torch.all(tall[:, :, :p0] == 3.0) and torch.all(tall[:, :, p0 + 2 * d:] == 3.0)
    dx = [h3d.Slab(torch.empty_like(x.t)) for _ in range(2)]
    h3d.deconv2_bwd_data(packed, w, dx[0])
    assert h3d.h3d_last_kernel().startswith("deconv_bd_mfma_kernel")
    view.t.copy_(packed.t)
    h3d.deconv2_bwd_data(view, w, dx[1])
    assert h3d.h3d_last_kernel() == "deconv2_bwd_data"
    close(from_dev(dx[1].t), from_dev(dx[0].t), TOL["bf16"])


@pytest.mark.parametrize("case", [(0, 1, 33, 20, 2, 5, 7, 0), (1, 2, 16, 17, 1, 3, 33, 1), (2, 1, 70, 64, 3, 4, 45, 2), (3, 1, 128, 24, 1, 2, 3, 0),
                                  (4, 1, 5, 9, 2, 1, 40, 1), (5, 3, 100, 34, 2, 9, 100, 0), (6, 1, 1, 1, 1, 2, 4, 2)])
def test_deconv_ragged_rows_bf16(case):
    """Rows that are no whole aligned 16-byte pieces (any width, data at an odd address), between NaNs: what a piece reads beyond its
    row or tensor must not reach a result."""
    import torch
    import paper_2007_12856_amd as h3d
    i, N, cin, cout, d, H, W, shift = case
    print("deconv ragged", case, flush=True)

    def moved(s, even=False):
        k = shift & ~1 if even else shift
        flat = torch.full((s.t.numel() + 32,), float("nan"), dtype=s.t.dtype, device="cuda")[k:k + s.t.numel()]
        return h3d.Slab(flat.view(s.t.shape).copy_(s.t), s.halo_lo, s.halo_hi, s.d_offset, s.d_global)

    b = np.sqrt(3.0 / (8 * cin))
    w = quantize(synth.flat("uniform", SEED, 5600 + i, (cin, cout, 2, 2, 2), -b, b), "bf16")
    bias = synth.round_f32(synth.flat("uniform", SEED, 5700 + i, (cout,), -0.1, 0.1)).astype(np.float64)
    xo, xg = slab_pair(synth.flat("normal", SEED, 5800 + i, (N, cin, d, H, W)), "bf16")
    xg = moved(xg)
    yo = orc.deconv2_fwd(xo, w, bias)
    yg = moved(dev_like(yo, "bf16"), even=True)      # (odd result addresses keep the general kernel)
    h3d.deconv2_fwd(xg, to_dev(w, "bf16"), to_dev(bias, "f32"), yg)
    ragged = h3d.h3d_last_kernel().startswith("deconv_fw_mfma_kernel") and h3d.h3d_last_kernel().endswith(",0>")
    assert ragged == (cin >= 16)      # (volumes of less than 49152 voxels)
    close(from_dev(yg.t), yo.a, TOL["bf16"])
    dyo, dyg = slab_pair(synth.flat("normal", SEED, 5900 + i, yo.a.shape), "bf16", (0, 0), yo.d_offset, yo.d_global)
    dxo = orc.deconv2_bwd_data(dyo, w)
    dxg = h3d.deconv2_bwd_data(moved(dyg, even=True), to_dev(w, "bf16"), moved(dev_like(dxo, "bf16")))
    close(from_dev(dxg.t), dxo.a, TOL["bf16"])
    dwo, dbo = orc.deconv2_bwd_filter(xo, dyo)
    dw, db = torch.empty((cin, cout, 2, 2, 2), device="cuda"), torch.empty((cout,), device="cuda")
    h3d.deconv2_bwd_filter(xg, moved(dyg), dw, db)
    # pieces of as many voxels as divide the width, and the plane into whole units of 8 where they are the longest
    piece = 4 if W % 4 == 0 and H * W % 8 == 0 else 2 if W % 2 == 0 else 1
    assert h3d.h3d_last_kernel() == "deconv_bf_flat_kernel<bf16,%d,%d>" % (128 if cin > 64 else 64 if cin > 32 else 32, piece)
    close(from_dev(dw), dwo, 2e-4)
    close(from_dev(db), dbo, 2e-4)


@pytest.mark.parametrize("cin,cout", [(20, 40), (40, 24), (33, 72)])
@pytest.mark.parametrize("N,D,H,W", [(1, 3, 9, 16), (1, 5, 17, 8), (24, 9, 17, 16), (48, 5, 9, 8), (16, 2, 70, 16)])
def test_narrow_rows_by_sixteen_bytes_equal_the_general_staging(cin, cout, N, D, H, W):
    """8 or 16 columns, at a 16-byte address (whole rows staged by 16-byte loads) and at one that is not (dwords): the products and
    their order are the same, so the bits are.  With channels split over workgroups and without, planes in rows of tiles, halos."""
    import torch
    import paper_2007_12856_amd as h3d
    print("narrow rows", cin, cout, N, D, H, W, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(cin + W)
    x = torch.randn((N, cin, D + 2, H, W), device="cuda", generator=gen).bfloat16()
    w = (0.1 * torch.randn((cout, cin, 3, 3, 3), device="cuda", generator=gen)).bfloat16()
    bias = torch.randn(cout, device="cuda", generator=gen)
    flat = torch.full((x.numel() + 64,), float("nan"), dtype=x.dtype, device="cuda")
    outs = []
    for shift in (0, 2):
        xs = flat[32 + shift:32 + shift + x.numel()].view(x.shape).copy_(x)
        assert (xs.data_ptr() % 16 == 0) == (shift == 0)
        y = torch.full((N, cout, D, H, W), float("nan"), dtype=x.dtype, device="cuda")
        h3d.conv3d_fwd(h3d.Slab(xs, 1, 1, 1, D + 2), w, bias, h3d.Slab(y, 0, 0, 1, D + 2), h3d.ACT_LEAKY, 0.01)
        assert h3d.h3d_last_kernel().startswith("conv3d_mfma_kernel<") and h3d.h3d_last_kernel().endswith(",0>" if shift else ",1>")
        outs.append(y)
        flat.fill_(float("nan"))
    assert torch.equal(outs[0], outs[1]) and bool(torch.isfinite(outs[0]).all())
    # and one voxel of the last row, column and plane against its definition
    n, d, h, v = N - 1, D - 1, H - 1, W - 1
    patch = torch.zeros((cin, 3, 3, 3), dtype=torch.float64, device="cuda")
    patch[:, :, :2, :2] = x[n, :, d:d + 3, h - 1:, v - 1:].double()
    ref = (w.double() * patch).sum(dim=(1, 2, 3, 4)) + bias.double()
    ref = torch.where(ref > 0, ref, 0.01 * ref)
    assert float((outs[0][n, :, d, h, v].double() - ref).abs().max()) <= 2.0 ** -8 * float(ref.abs().max())


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("case", [(1, 1, 1, 1, 2, 4, 0, 0), (1, 33, 17, 2, 3, 4, 1, 0), (2, 16, 16, 3, 8, 16, 0, 1), (1, 65, 15, 2, 5, 6, 0, 2), (3, 128, 33, 1, 7, 9, 3, 0),
                                  (1, 129, 16, 2, 16, 20, 0, 1), (2, 64, 40, 9, 3, 12, 0, 0), (1, 8, 8, 70, 2, 2, 1, 1)])
def test_deconv_filter_gradient_of_any_rows(case, dtype):
    """The filter gradient's tiles run along a plane whatever its width: one plane's last unit of voxels must not take the next plane's
    (or the next channel's, or what lies behind the tensor).  Odd addresses, halos, NaN around the tensors and in their halo planes, an infinity behind a plane's end."""
    import torch
    import paper_2007_12856_amd as h3d
    N, cin, cout, d, H, W, shift, halo = case
    print("deconv filter gradient", case, dtype, flush=True)
    td = {"bf16": torch.bfloat16, "f32": torch.float32}[dtype]
    rng = np.random.default_rng(1000 * cin + W)
    xa, ya = rng.standard_normal((N, cin, d, H, W)) + 0.3, rng.standard_normal((N, cout, 2 * d, 2 * H, 2 * W)) + 0.1

    def placed(a, hw):
        shape = (a.shape[0], a.shape[1], a.shape[2] + 2 * hw) + a.shape[3:]
        flat = torch.full((int(np.prod(shape)) + 64,), float("nan"), dtype=td, device="cuda")
        t = flat[32 + shift:32 + shift + int(np.prod(shape))].view(shape)
        t[:, :, hw:hw + a.shape[2]] = to_dev(quantize(a, dtype), dtype)
        return h3d.Slab(t, hw, hw, a.shape[2], 3 * a.shape[2])

    xg, yg = placed(xa, halo), placed(ya, 2 * halo)
    dwo, dbo = orc.deconv2_bwd_filter(orc.Slab(quantize(xa, dtype)), orc.Slab(quantize(ya, dtype)))
    dw, db = torch.full((cin, cout, 2, 2, 2), float("nan"), device="cuda"), torch.full((cout,), float("nan"), device="cuda")
    h3d.deconv2_bwd_filter(xg, yg, dw, db)
    assert h3d.h3d_last_kernel().startswith("deconv_bf_flat_kernel")
    # sums of at most 4096 products in fp32, each partial sum rounded once: a few units of 2^-24 of what was added up
    n = N * d * H * W
    scale = np.abs(quantize(xa, dtype)).max() * np.abs(quantize(ya, dtype)).max() * n ** 0.5
    assert np.abs(from_dev(dw) - dwo).max() <= 2e-6 * scale and np.abs(from_dev(db) - dbo).max() <= 2e-6 * 8 ** 0.5 * scale
    if cin > 1:      # an infinity in the last channel stays there
        xg.t[:, cin - 1, halo] = float("inf")
        h3d.deconv2_bwd_filter(xg, yg, dw, db)
        assert bool(torch.isfinite(dw[:cin - 1]).all()) and bool(torch.isfinite(db).all())


@pytest.mark.parametrize("masked", [False, True])
@pytest.mark.parametrize("N,cin,cout,D,H,W", [(2, 65, 65, 7, 12, 33), (1, 80, 70, 1, 9, 40), (3, 66, 72, 2, 20, 16), (1, 70, 65, 5, 17, 7), (1, 5, 3, 1, 1, 1), (2, 17, 16, 3, 4, 32)])
def test_f32_filter_gradient_walks_every_run_of_planes(N, cin, cout, D, H, W, masked):
    """fp32 backward-filter: chunks that begin and end within a run of planes (65 channels on both sides: three tiles a chunk), runs of one
    plane, rows wider than a tile and narrower than one; halos that are stored and ones that lie outside the volume."""
    import torch
    import paper_2007_12856_amd as h3d
    print("f32 filter gradient", N, cin, cout, D, H, W, masked, flush=True)
    rng = np.random.default_rng(cin + D)
    for off, dg in ((0, D), (2, D + 5)):
        halo = (1, 1) if off else (0, 0)
        xo, xg = slab_pair(rng.standard_normal((N, cin, D + sum(halo), H, W)), "f32", halo, off, dg)
        dzo, dzg = slab_pair(rng.standard_normal((N, cout, D, H, W)), "f32", (0, 0), off, dg)
        zo, zg = slab_pair(rng.standard_normal((N, cout, D, H, W)), "f32", (0, 0), off, dg)
        act = orc.ACT_LEAKY if masked else orc.ACT_NONE
        dwo, dbo = orc.conv3d_bwd_filter(xo, dzo, zo if masked else None, act=act, alpha=0.01)
        dw, db = torch.full((cout, cin, 3, 3, 3), float("nan"), device="cuda"), torch.full((cout,), float("nan"), device="cuda")
        h3d.conv3d_bwd_filter(xg, dzg, zg if masked else None, dw, db, act, 0.01)
        close(from_dev(dw), dwo, TOL["f32"], "dw")
        close(from_dev(db), dbo, TOL["f32"], "db")


@pytest.mark.parametrize("N,ci,co,D,H,W,split", [(1, 100, 33, 3, 4, 17, True), (2, 64, 40, 5, 9, 35, True), (1, 256, 8, 6, 17, 32, True), (1, 48, 70, 9, 8, 66, True),
                                                 (1, 40, 64, 4, 8, 30, True), (1, 17, 9, 33, 64, 64, False), (1, 16, 64, 4, 8, 32, False)])
def test_wide_rows_of_few_tiles_with_split_channels(N, ci, co, D, H, W, split):
    """Volumes of few tiles: the input channels are split over workgroups whose sums a second kernel adds (rows of odd length and masked ones through
    the operand copies).  A shard of the same numbers is not split: the two agree to a rounding of bf16."""
    import torch
    import paper_2007_12856_amd as h3d
    print("wide split", N, ci, co, D, H, W, flush=True)
    rng = np.random.default_rng(ci + W)
    w = quantize(rng.uniform(-1, 1, (co, ci, 3, 3, 3)) / np.sqrt(9 * ci), "bf16")
    wd, bd = to_dev(w, "bf16"), to_dev(rng.uniform(-0.1, 0.1, co), "f32")
    xo, xg = slab_pair(rng.standard_normal((N, ci, D, H, W)), "bf16")
    zo = orc.conv3d_fwd(xo, w, from_dev(bd), act=orc.ACT_LEAKY, alpha=0.01)
    zg = h3d.conv3d_fwd(xg, wd, bd, dev_like(zo, "bf16", float("nan")), h3d.ACT_LEAKY, 0.01)
    assert h3d.h3d_last_kernel().endswith("(split)") == split, h3d.h3d_last_kernel()
    close(from_dev(zg.t), zo.a, TOL["bf16"], "z")
    pad = torch.zeros((N, ci, D + 2, H, W), dtype=torch.bfloat16, device="cuda")
    pad[:, :, 1:-1] = xg.t
    zs = h3d.conv3d_fwd(h3d.Slab(pad, 1, 1, 1, D + 2), wd, bd, h3d.Slab(torch.empty_like(zg.t), 0, 0, 1, D + 2), h3d.ACT_LEAKY, 0.01)
    assert not h3d.h3d_last_kernel().endswith("(split)")
    close(from_dev(zs.t), from_dev(zg.t), TOL["bf16"], "shard")
    go, gg = slab_pair(rng.standard_normal((N, co, D, H, W)), "bf16")
    so, sg = slab_pair(rng.standard_normal((N, co, D, H, W)), "bf16")
    for a, z, zd in ((orc.ACT_NONE, None, None), (orc.ACT_LEAKY, so, sg)):
        dxo = orc.conv3d_bwd_data(go, z, w, act=a, alpha=0.01)
        close(from_dev(h3d.conv3d_bwd_data(gg, zd, wd, dev_like(dxo, "bf16", float("nan")), a, 0.01).t), dxo.a, TOL["bf16"], "dx")


@pytest.mark.parametrize("N,ci,co,D,H,W,split", [(1, 70, 9, 3, 5, 33, True), (2, 36, 40, 5, 7, 16, True), (1, 256, 24, 4, 3, 18, True), (1, 40, 6, 1, 1, 1, False),
                                                 (1, 32, 16, 4, 8, 16, False), (1, 64, 3, 6, 9, 20, False)])
def test_f32_few_tiles_with_split_channels(N, ci, co, D, H, W, split):
    """fp32 volumes of few tiles: channel groups split over workgroups, an uneven last split, rows that end within a store of four."""
    import torch
    import paper_2007_12856_amd as h3d
    print("f32 split", N, ci, co, D, H, W, flush=True)
    rng = np.random.default_rng(ci + W)
    w = quantize(rng.uniform(-1, 1, (co, ci, 3, 3, 3)) / np.sqrt(9 * ci), "f32")
    wd, bd = to_dev(w, "f32"), to_dev(rng.uniform(-0.1, 0.1, co), "f32")
    xo, xg = slab_pair(rng.standard_normal((N, ci, D, H, W)), "f32")
    zo = orc.conv3d_fwd(xo, w, from_dev(bd), act=orc.ACT_LEAKY, alpha=0.01)
    zg = h3d.conv3d_fwd(xg, wd, bd, dev_like(zo, "f32", float("nan")), h3d.ACT_LEAKY, 0.01)
    assert h3d.h3d_last_kernel().endswith("(split)") == split, h3d.h3d_last_kernel()
    close(from_dev(zg.t), zo.a, TOL["f32"], "z")
    wt = quantize(rng.uniform(-1, 1, (ci, co, 3, 3, 3)) / np.sqrt(9 * ci), "f32")      # a layer co -> ci: its data gradient has co channels
    so, sg = slab_pair(rng.standard_normal((N, ci, D, H, W)), "f32")
    dxo = orc.conv3d_bwd_data(xo, so, wt, act=orc.ACT_LEAKY, alpha=0.01)
    dxg = h3d.conv3d_bwd_data(xg, sg, to_dev(wt, "f32"), dev_like(dxo, "f32", float("nan")), h3d.ACT_LEAKY, 0.01)
    assert h3d.h3d_last_kernel().endswith("(split)") == split, h3d.h3d_last_kernel()
    close(from_dev(dxg.t), dxo.a, TOL["f32"], "dx")


@pytest.mark.parametrize("N,ci,co,D,H,W,split", [(5, 144, 72, 8, 9, 16, True), (8, 144, 128, 8, 16, 8, True), (64, 40, 32, 1, 4, 5, False), (8, 112, 128, 9, 8, 7, True), (65, 80, 40, 4, 16, 3, False)])
def test_narrow_volumes_split_from_64_workgroups_on(N, ci, co, D, H, W, split):
    """Narrow volumes between 64 and 256 workgroups: channels split where it pays; an uneven last split; more workgroups than 256 stay whole."""
    import torch
    import paper_2007_12856_amd as h3d
    print("narrow split", N, ci, co, D, H, W, flush=True)
    rng = np.random.default_rng(ci + W)
    w = quantize(rng.uniform(-1, 1, (co, ci, 3, 3, 3)) / np.sqrt(9 * ci), "bf16")
    wd, bd = to_dev(w, "bf16"), to_dev(rng.uniform(-0.1, 0.1, co), "f32")
    xo, xg = slab_pair(rng.standard_normal((N, ci, D, H, W)), "bf16")
    zo = orc.conv3d_fwd(xo, w, from_dev(bd), act=orc.ACT_LEAKY, alpha=0.01)
    zg = h3d.conv3d_fwd(xg, wd, bd, dev_like(zo, "bf16", float("nan")), h3d.ACT_LEAKY, 0.01)
    assert (h3d.h3d_last_kernel().split(",")[5] == "1") == split, h3d.h3d_last_kernel()
    close(from_dev(zg.t), zo.a, TOL["bf16"], "z")


@pytest.mark.parametrize("dtype,N,ci,co,D,H,W,larger", [("bf16", 1, 100, 33, 3, 4, 17, 64), ("bf16", 1, 64, 64, 16, 32, 32, 64), ("bf16", 8, 144, 128, 8, 16, 8, 128),
                                                        ("f32", 2, 36, 40, 5, 7, 16, 128), ("f32", 1, 70, 36, 3, 5, 33, 64)])
def test_the_workspace_of_a_larger_volume_does_for_a_smaller_one(dtype, N, ci, co, D, H, W, larger):
    """Calls that would sum their channels in parts, in a workspace sized by a layer of the same channels that does not: one chain of sums."""
    import torch
    import paper_2007_12856_amd as h3d
    print("larger workspace", dtype, N, ci, co, D, H, W, flush=True)
    rng = np.random.default_rng(ci + W)
    w = quantize(rng.uniform(-1, 1, (co, ci, 3, 3, 3)) / np.sqrt(9 * ci), dtype)
    wd, bd = to_dev(w, dtype), to_dev(rng.uniform(-0.1, 0.1, co), "f32")
    xo, xg = slab_pair(rng.standard_normal((N, ci, D, H, W)), dtype)
    go, gg = slab_pair(rng.standard_normal((N, co, D, H, W)), dtype)
    so, sg = slab_pair(rng.standard_normal((N, co, D, H, W)), dtype)
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    big = lambda c: h3d.Slab(torch.empty((N, c, larger, 64, 16 if W <= 16 else 64), dtype=td, device="cuda"))

    class Sized:
        def __init__(self, op, a, b):
            self.n = h3d.h3d_conv3d_workspace_bytes(op, big(a), big(b))
            self.buf = torch.full((self.n + 4096,), 171, dtype=torch.uint8, device="cuda")

        def get(self, nbytes):
            assert nbytes > self.n, "the smaller volume asks for more"
            return self.buf.data_ptr(), self.n

    zo = orc.conv3d_fwd(xo, w, from_dev(bd), act=orc.ACT_LEAKY, alpha=0.01)
    dxo = orc.conv3d_bwd_data(go, so, w, act=orc.ACT_LEAKY, alpha=0.01)
    for ws, ref, call in ((Sized(h3d.OP_FWD, ci, co), zo, lambda t, k: h3d.conv3d_fwd(xg, wd, bd, t, h3d.ACT_LEAKY, 0.01, k)),
                          (Sized(h3d.OP_FWD, co, ci), dxo, lambda t, k: h3d.conv3d_bwd_data(gg, sg, wd, t, h3d.ACT_LEAKY, 0.01, k))):
        t = dev_like(ref, dtype, float("nan"))
        call(t, ws)
        assert "split" not in h3d.h3d_last_kernel()
        close(from_dev(t.t), ref.a, TOL[dtype])
        assert bool((ws.buf[ws.n:] == 171).all())


@pytest.mark.parametrize("dtype,cin,cout,d,H,W,shift,kernel", [
    ("f32", 20, 24, 4, 16, 32, 4, "deconv2_bwd_filter"), ("bf16", 20, 24, 4, 16, 30, 4, "deconv2_bwd_filter"), ("f32", 20, 24, 4, 16, 32, 0, "deconv_bf_flat_kernel")])
def test_deconv_filter_gradient_in_a_workspace_at_an_odd_address(dtype, cin, cout, d, H, W, shift, kernel):
    """fp32 tensors and ragged rows in a workspace that is no multiple of 16: the direct kernel, as for one too small for the matrix cores' sums."""
    import torch
    import paper_2007_12856_amd as h3d

    class Moved:
        def get(self, nbytes):
            self.buf = torch.empty(int(nbytes) + 16, dtype=torch.uint8, device="cuda")
            return self.buf.data_ptr() + shift, int(nbytes)

    rng = np.random.default_rng(cin)
    xo, xg = slab_pair(rng.standard_normal((1, cin, d, H, W)), dtype)
    dyo, dyg = slab_pair(rng.standard_normal((1, cout, 2 * d, 2 * H, 2 * W)), dtype)
    dwo, dbo = orc.deconv2_bwd_filter(xo, dyo)
    dw, db = torch.full((cin, cout, 2, 2, 2), float("nan"), device="cuda"), torch.full((cout,), float("nan"), device="cuda")
    h3d.deconv2_bwd_filter(xg, dyg, dw, db, Moved())
    assert h3d.h3d_last_kernel().startswith(kernel)
    close(from_dev(dw), dwo, 2e-5)
    close(from_dev(db), dbo, 2e-5)
