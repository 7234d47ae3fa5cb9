"""The C-ABI library loads without a GPU and exports every symbol the header declares."""
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_symbols():
    text = open(os.path.join(ROOT, "include", "h3d.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(h3d_[a-z0-9_]+)\s*\(", text)))


def test_header_symbols_are_exported_and_bound():
    import paper_2007_12856_amd as h3d
    if not os.path.exists(h3d.LIB_PATH):
        from paper_2007_12856_amd import build
        build.build()
    lib = ctypes.CDLL(h3d.LIB_PATH)
    names = declared_symbols()
    assert len(names) >= 20
    for name in names:
        assert hasattr(lib, name), f"{name} declared in include/h3d.h but not exported"
        assert name in h3d._SIGNATURES, f"{name} has no Python binding"
        assert callable(getattr(h3d, name)), name


def test_descriptor_layout_matches_header():
    import paper_2007_12856_amd as h3d
    # void* + 8 x int32 + 2 x int64 with natural alignment
    assert ctypes.sizeof(h3d.h3d_tensor) == 8 + 8 * 4 + 4 * 8
    assert h3d.h3d_tensor.d_offset.offset == 40 and h3d.h3d_tensor.dtype.offset == 8 and h3d.h3d_tensor.c_stride.offset == 56


def test_missing_library_fails_loudly(monkeypatch):
    import paper_2007_12856_amd as h3d
    monkeypatch.setattr(h3d, "_lib", None)
    monkeypatch.setattr(h3d, "LIB_PATH", "/nonexistent/libh3d.so")
    with pytest.raises(RuntimeError):
        h3d.lib()


def _desc(h3d, n, c, d, h, w, halo=0, d_offset=None, d_global=None):
    """A bf16 descriptor without data: what the size queries take."""
    off = d if d_offset is None else d_offset
    return h3d.h3d_tensor(None, h3d.BF16, n, c, d, h, w, halo, halo, off, 3 * d if d_global is None else d_global, 0, 0)


def test_k5_filter_gradient_of_a_channel_whose_padded_copy_is_too_long():
    """5x5x5 backward-filter of rows of 97 columns reads copies with rows of 104.  32-bit offsets reach blocks of 32 channels below 2^25
    elements each: x as it is (33.52e6) and the padded dz (33.55e6) pass, the padded x (35.94e6, four planes taller) does not, so the
    query must not ask for room for its copy (2.3e9 bytes); a shard of 51 planes does get it."""
    import paper_2007_12856_amd as h3d
    lib, handle = h3d.lib(), ctypes.cast(ctypes.create_string_buffer(4096), ctypes.c_void_p)      # (a query reads no field of the handle)
    limit = 1 << 25
    for d, fits in ((56, False), (51, True)):
        x, z = _desc(h3d, 1, 32, d, 5760, 97, halo=2), _desc(h3d, 1, 32, d, 5760, 97)
        assert (d + 4) * 5760 * 97 < limit and d * 5760 * 104 < limit and ((d + 4) * 5760 * 104 < limit) == fits
        need = lib.h3d_conv3d_k5_workspace_bytes(handle, h3d.OP_BWD_FILTER, ctypes.byref(x), ctypes.byref(z))
        assert (need > 2 * 32 * (d + 4) * 5760 * 104) == fits
        # forward reads x where it lies
        assert lib.h3d_conv3d_k5_workspace_bytes(handle, h3d.OP_FWD, ctypes.byref(x), ctypes.byref(z)) == 1 * 2 * 125 * 1024


def test_a_failed_kernel_setup_is_reported_to_every_handle():
    """Without a device the dynamic LDS limit of the 5x5x5 kernel cannot be raised.  Each call says so on its own handle: the first failure
    is not kept for the process."""
    import subprocess
    import sys
    script = """
import ctypes, sys
sys.path.insert(0, %r)
import paper_2007_12856_amd as h3d
lib = h3d.lib()
none = ctypes.c_void_p()
assert lib.h3d_create(ctypes.byref(none)) != 0          # no device is visible to this process: nothing below can run on one
t = lambda c: h3d.h3d_tensor(1 << 20, h3d.BF16, 1, c, 4, 16, 32, 0, 0, 0, 4, 0, 0)
x, z = t(16), t(32)
for attempt in range(2):
    handle = ctypes.cast(ctypes.create_string_buffer(4096), ctypes.c_void_p)
    need = lib.h3d_conv3d_k5_workspace_bytes(handle, h3d.OP_FWD, ctypes.byref(x), ctypes.byref(z))
    st = lib.h3d_conv3d_k5_fwd(handle, ctypes.byref(x), ctypes.c_void_p(1 << 20), None, ctypes.byref(z), 0, 0.0, ctypes.c_void_p(1 << 20), need, None)
    text = lib.h3d_last_error(handle)
    assert st != 0 and b"LDS limit" in text, (attempt, st, text)
""" % ROOT
    env = dict(os.environ, HIP_VISIBLE_DEVICES="-1", ROCR_VISIBLE_DEVICES="-1")
    r = subprocess.run([sys.executable, "-c", script], env=env, capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr


def test_an_unmasked_data_gradient_asks_for_no_copies():
    """64 -> 64 channels on 64 x 256 x 256: with an activation the workspace has room for a slab of the masked gradient, without one it is the
    packed filter alone, and the wrapper asks for that."""
    import paper_2007_12856_amd as h3d
    lib, handle = h3d.lib(), ctypes.cast(ctypes.create_string_buffer(4096), ctypes.c_void_p)
    dz, dx = _desc(h3d, 1, 64, 64, 256, 256, halo=1), _desc(h3d, 1, 64, 64, 256, 256)
    packed = 64 * 64 * 27 * 2
    need = lambda op: lib.h3d_conv3d_workspace_bytes(handle, op, ctypes.byref(dz), ctypes.byref(dx))
    assert need(h3d.OP_BWD_DATA) > 100 << 20 and packed <= need(h3d.OP_FWD) <= 2 * packed

    class Asked(Exception):
        pass

    class Slab:
        def __init__(self, d):
            self.d = d

        def desc(self):
            return self.d

    class Workspace:
        def get(self, nbytes):
            raise Asked(nbytes)

    saved, h3d._handle = h3d._handle, handle
    try:
        for z, act, op in ((None, h3d.ACT_LEAKY, h3d.OP_FWD), (Slab(dz), h3d.ACT_NONE, h3d.OP_FWD), (Slab(dz), h3d.ACT_RELU, h3d.OP_BWD_DATA)):
            with pytest.raises(Asked) as e:
                h3d.conv3d_bwd_data(Slab(dz), z, None, Slab(dx), act, 0.01, Workspace())
            assert e.value.args[0] == need(op)
    finally:
        h3d._handle = saved
