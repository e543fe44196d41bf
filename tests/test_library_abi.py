"""Host-side tests of the C-ABI library: it loads, exports every entry point the header
declares, and rejects invalid arguments with the documented codes before anything is launched.
No compute call is made here."""
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "tfla_mlstm.h")


@pytest.fixture(scope="module")
def tfla():
    import paper_2503_14376_amd as pkg
    if not os.path.exists(pkg.lib_path()):
        from paper_2503_14376_amd import build
        build.build(verbose=False)
    pkg.load_library()
    return pkg


def declared_symbols():
    text = open(HEADER).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"TFLA_API\s+[\w\s\*]+?\b(tfla_\w+)\s*\(", text)))


def test_header_declares_the_entry_points():
    names = declared_symbols()
    for need in ("tfla_mlstm_fwd", "tfla_mlstm_bwd", "tfla_mlstm_workspace_bytes", "tfla_mlstm_check"):
        assert need in names, names


def test_library_exports_every_declared_symbol(tfla):
    lib = ctypes.CDLL(tfla.lib_path())
    for name in declared_symbols():
        assert hasattr(lib, name), name
    from paper_2503_14376_amd import binding
    assert sorted(binding.EXPORTS) == declared_symbols()


def test_every_kernel_is_built_once(tfla):
    # A kernel descriptor's name stands in its code object a fixed number of times; a kernel that more than one unit
    # instantiates is there in as many copies.
    with open(tfla.lib_path(), "rb") as f:
        names = re.findall(rb"_ZN4tfla\w+?\.kd", f.read())
    count = {n: names.count(n) for n in set(names)}
    assert any(b"grads_kernel_bf16" in n for n in count)
    least = min(count.values())
    assert [n for n, c in count.items() if c != least] == []


def test_missing_library_fails_loudly(tfla, monkeypatch):
    from paper_2503_14376_amd import binding
    monkeypatch.setattr(binding, "_lib", None)
    monkeypatch.setattr(binding, "_LIB_PATH", "/nonexistent/libtfla_mlstm.so")
    with pytest.raises(ImportError):
        binding.load_library()


OK_ARGS = dict(direction=0, B=2, NH=8, T=8192, dqk=256, dhv=512, chunk=256, variant=0, dtype=1)


def _check(tfla, **kw):
    a = dict(OK_ARGS); a.update(kw)
    return tfla.check(a["direction"], a["B"], a["NH"], a["T"], a["dqk"], a["dhv"], a["chunk"], a["variant"], a["dtype"])


def test_check_accepts_the_benchmark_configurations(tfla):
    import workloads as wl
    for w in wl.CONFIGS.values():
        for direction in (0, 1):
            assert tfla.check(direction, w.B, w.NH, w.T, w.dqk, w.dhv, w.chunk, w.variant, w.dtype) == 0, w.name
            assert tfla.workspace_bytes(direction, w.B, w.NH, w.T, w.dqk, w.dhv, w.chunk, w.variant, w.dtype) > 0
    for L in wl.C2_CHUNKS:
        assert _check(tfla, variant=1, chunk=L) == 0


@pytest.mark.parametrize("kw,code", [
    (dict(B=0), -2), (dict(NH=-1), -2), (dict(T=0), -2), (dict(dqk=100), -2), (dict(dqk=4), -2), (dict(dhv=1032), -2), (dict(dqk=2048), -2),
    (dict(dtype=0, dhv=1024), -2), (dict(B=4096, NH=16), -2),
    (dict(chunk=0), -3), (dict(chunk=32), -3), (dict(chunk=96), -3), (dict(chunk=4096), -3),
    (dict(T=64 * 8192, chunk=64), -3),
    (dict(variant=2), -4), (dict(dtype=7), -4), (dict(direction=3), -4),
])
def test_check_rejects_invalid_dimensions(tfla, kw, code):
    assert _check(tfla, **kw) == code
    a = dict(OK_ARGS); a.update(kw)
    assert tfla.workspace_bytes(*[a[k] for k in ("direction", "B", "NH", "T", "dqk", "dhv", "chunk", "variant", "dtype")]) == 0


def test_ragged_sequence_lengths_are_accepted_and_need_more_workspace(tfla):
    assert _check(tfla, T=8192 + 64, chunk=256) == 0
    assert _check(tfla, T=1, chunk=64) == 0
    a = dict(OK_ARGS); a.pop("direction")
    for direction in (0, 1):
        whole = tfla.workspace_bytes(direction, **a)
        ragged = tfla.workspace_bytes(direction, **dict(a, T=8192 - 1))
        # the same number of chunks plus padded copies of the inputs and per-step outputs
        assert ragged > whole + 16 * 8192 * (256 + 256 + 512) * 2


def test_head_dimensions_between_the_kernel_widths_are_accepted(tfla):
    # any multiple of 8 up to 1024 runs zero-padded to the next width of the kernels, with more workspace
    for dqk, dhv in ((32, 32), (96, 192), (8, 504), (1024, 1024), (520, 1000)):
        assert _check(tfla, dqk=dqk, dhv=dhv) == 0
    a = dict(OK_ARGS); a.pop("direction")
    for direction in (0, 1):
        assert tfla.workspace_bytes(direction, **dict(a, dqk=192)) > tfla.workspace_bytes(direction, **a)


def test_status_strings(tfla):
    seen = set()
    for code in range(0, -7, -1):
        s = tfla.status_string(code)
        assert s and s not in seen
        seen.add(s)
    assert tfla.status_string(-99)      # unknown codes still give a printable string
    assert tfla.load_library().tfla_version() >= 1


def test_workspace_grows_with_the_problem(tfla):
    small = tfla.workspace_bytes(1, 1, 1, 512, 64, 64, 64, 0, 1)
    big = tfla.workspace_bytes(1, 2, 8, 8192, 256, 512, 256, 0, 1)
    assert 0 < small < big
    # the backward workspace holds both chunk-state sets (bf16): at least 2 * BH*Nc*dqk*dhv*2 bytes
    assert big >= 2 * 16 * 32 * 256 * 512 * 2
    assert big % 256 == 0


# (B, NH, T, dqk, dhv, chunk, variant, dtype), bytes forward and backward that callers may have planned their buffers with
PLANNED = [
    ((2, 8, 8192, 256, 512, 256, 0, 1), 215488512, 417373440),
    ((1, 8, 512, 256, 512, 256, 0, 1), 12763648, 19074048),         # 128-wide dQ / dK blocks at d_hv = 512
    ((1, 8, 512, 512, 512, 128, 1, 1), 33784320, 51614720),
    ((1, 4, 300, 1024, 512, 128, 0, 1), 65710592, 91792384),
    ((1, 1, 5000, 1024, 512, 2048, 0, 1), 58061312, 107551744),
    ((1, 8, 1000, 256, 512, 128, 0, 1), 55067392, 86586624),
    ((2, 16, 3000, 96, 192, 128, 0, 1), 194683904, 300718080),
    ((4, 64, 2048, 64, 64, 256, 0, 1), 50880512, 71336960),
    ((1, 1, 64, 64, 64, 64, 0, 1), 44288, 53504),
    ((4, 4, 4096, 1024, 1024, 256, 0, 1), 1413221376, 2020347648),
    ((2, 8, 1024, 128, 256, 64, 1, 0), 36836352, 103949824),
    ((3, 8, 1000, 256, 264, 128, 0, 0), 241291008, 556245248),
]


@pytest.mark.parametrize("dims,fwd,bwd", PLANNED)
def test_workspace_sizes_do_not_grow(tfla, dims, fwd, bwd):
    # the forward size is exact: it decides what the entry point with the static scratch memory accepts
    assert tfla.workspace_bytes(0, *dims) == fwd
    assert 0 < tfla.workspace_bytes(1, *dims) <= bwd


def _call_fwd(lib, q=1, k=1, v=1, i=1, f=1, C0=0, n0=0, m0=0, H=1, ws=256, ws_bytes=1 << 40, **kw):
    """tfla_mlstm_fwd with fake (never dereferenced) pointers: only the host-side validation runs."""
    a = dict(OK_ARGS); a.update(kw)
    P = lambda x: ctypes.c_void_p(x * 4096) if x else None
    return lib.tfla_mlstm_fwd(P(q), P(k), P(v), P(i), P(f), P(C0), P(n0), P(m0), a["B"], a["NH"], a["T"], a["dqk"],
                              a["dhv"], a["chunk"], a["variant"], a["dtype"], 1e-6, P(H), None, None, None, None, None,
                              ctypes.c_void_p(ws) if ws else None, ws_bytes, None)


def test_forward_argument_validation_happens_before_any_launch(tfla):
    lib = tfla.load_library()
    assert _call_fwd(lib, q=0) == -1
    assert _call_fwd(lib, H=0) == -1
    assert _call_fwd(lib, f=0) == -1
    assert _call_fwd(lib, dqk=100) == -2
    assert _call_fwd(lib, chunk=100) == -3
    assert _call_fwd(lib, variant=5) == -4
    assert _call_fwd(lib, C0=1) == -6              # initial state only partly given
    assert _call_fwd(lib, C0=1, n0=1) == -6
    assert _call_fwd(lib, ws=0) == -5              # no workspace
    assert _call_fwd(lib, ws=4096 + 8) == -5       # misaligned workspace
    assert _call_fwd(lib, ws=4096, ws_bytes=1024) == -5   # too small


def test_backward_argument_validation_happens_before_any_launch(tfla):
    lib = tfla.load_library()
    P = lambda x: ctypes.c_void_p(x * 4096) if x else None
    a = OK_ARGS

    def call(n_out=1, m_out=1, dH=1, dq=1, d_f=1, C0=0, ws=4096, ws_bytes=1 << 40, chunk=256, variant=0,
             fws=0, fws_bytes=0):
        return lib.tfla_mlstm_bwd(P(1), P(1), P(1), P(1), P(1), P(C0), None, None, P(n_out), P(m_out), P(dH), None,
                                  a["B"], a["NH"], a["T"], a["dqk"], a["dhv"], chunk, variant, a["dtype"], 1e-6,
                                  P(dq), P(1), P(1), P(1), P(d_f), None, P(fws) if fws else None, fws_bytes,
                                  P(1) if ws else None, ws_bytes, None)
    assert call(dH=0) == -1
    assert call(dq=0) == -1
    assert call(d_f=0) == -1
    assert call(n_out=0) == -1                     # the exponential-gate backward needs n and m of the forward
    assert call(m_out=0) == -1
    assert call(chunk=48) == -3
    assert call(C0=1) == -6
    assert call(ws=0) == -5
    assert call(ws_bytes=4096) == -5
    assert call(fws=2, fws_bytes=1024) == -5       # a forward workspace that is too small to be one


def test_step_argument_validation_happens_before_any_launch(tfla):
    lib = tfla.load_library()
    P = lambda x: ctypes.c_void_p(x * 4096) if x else None

    def call(q=1, C=1, n=2, m=3, h=1, C_out=1, n_out=4, m_out=5, dqk=256, dhv=512, variant=0, dtype=1, B=2, NH=8):
        return lib.tfla_mlstm_step(P(q), P(1), P(1), P(1), P(1), P(C), P(n), P(m), B, NH, dqk, dhv, variant, dtype, 1e-6,
                                   P(h), P(C_out), P(n_out), P(m_out), None)
    assert call(q=0) == -1
    assert call(C=0) == -1
    assert call(h=0) == -1
    assert call(n_out=0) == -1                     # the exponential-gate step returns n and m
    assert call(dqk=96) == -2
    assert call(dhv=2048) == -2
    assert call(B=0) == -2
    assert call(variant=3) == -4
    assert call(dtype=2) == -4
    assert call(n=2, m=0) == -6                    # state only partly given
    assert call(n=4, n_out=4) == -6                # n_out must not alias n
    assert call(m=5, m_out=5) == -6


def test_layer_argument_validation_happens_before_any_launch(tfla):
    lib = tfla.load_library()
    P = lambda x: ctypes.c_void_p(x * 4096) if x else None
    a = OK_ARGS
    cf = ctypes.c_float

    def fwd(Y=1, H=1, q=1, norm=0, cap=15.0, neps=1e-6, ws=1, ws_bytes=1 << 40, chunk=256):
        return lib.tfla_mlstm_layer_fwd(P(q), P(1), P(1), P(1), P(1), P(1), P(1), None, None, None, None,
                                        a["B"], a["NH"], a["T"], a["dqk"], a["dhv"], chunk, a["variant"], a["dtype"],
                                        cf(1e-6), cf(cap), norm, cf(neps), P(Y), P(H), None, None, None, None, None,
                                        P(ws), ws_bytes, None)
    assert fwd(Y=0) == -1
    assert fwd(H=0) == -1
    assert fwd(q=0) == -1
    assert fwd(norm=7) == -4
    assert fwd(cap=-1.0) == -2
    assert fwd(neps=-1.0) == -2
    assert fwd(chunk=100) == -3
    assert fwd(ws=0) == -5
    assert fwd(ws_bytes=1024) == -5

    def bwd(H=1, dY=1, dq=1, n_out=1, norm=1, ws=1, ws_bytes=1 << 40, fws=0, fws_bytes=0):
        return lib.tfla_mlstm_layer_bwd(P(1), P(1), P(1), P(1), P(1), P(1), P(1), P(1), None, None, None,
                                        P(H), P(n_out), P(1), P(dY), None,
                                        a["B"], a["NH"], a["T"], a["dqk"], a["dhv"], a["chunk"], a["variant"], a["dtype"],
                                        cf(1e-6), cf(15.0), norm, cf(1e-6), P(dq), P(1), P(1), P(1), P(1), P(1), P(1), P(1),
                                        None, P(fws), fws_bytes, P(ws), ws_bytes, None)
    assert bwd(H=0) == -1
    assert bwd(dY=0) == -1
    assert bwd(dq=0) == -1
    assert bwd(n_out=0) == -1
    assert bwd(norm=-1) == -4
    assert bwd(ws=0) == -5
    # the layer's backward workspace is larger than the cell's: the cell's size alone is refused
    args9 = (a["B"], a["NH"], a["T"], a["dqk"], a["dhv"], a["chunk"], a["variant"], a["dtype"])
    cell = lib.tfla_mlstm_workspace_bytes(1, *args9)
    layer = lib.tfla_mlstm_layer_workspace_bytes(1, *args9)
    assert layer >= cell + a["B"] * a["NH"] * a["T"] * a["dhv"] * 2
    assert lib.tfla_mlstm_layer_workspace_bytes(0, *args9) == lib.tfla_mlstm_workspace_bytes(0, *args9)
    assert bwd(ws_bytes=cell) == -5
    assert bwd(fws=1, fws_bytes=1024) == -5
    assert lib.tfla_mlstm_layer_workspace_bytes(1, a["B"], a["NH"], a["T"], 100, a["dhv"], a["chunk"], 0, 1) == 0

    def gain(h=1, gb=1, dhv=128, dtype=1, norm=0, neps=1e-6, T=512):
        return lib.tfla_transfer_gain(P(h), P(1), 2, 3, T, dhv, dtype, norm, cf(neps), P(gb), P(1), None)
    assert gain(h=0) == -1
    assert gain(gb=0) == -1
    assert gain(dhv=100) == -2
    assert gain(dhv=4096) == -2
    assert gain(T=0) == -2
    assert gain(dtype=3) == -4
    assert gain(norm=2) == -4
    assert gain(neps=-1.0) == -2


def test_layer_step_argument_validation(tfla):
    lib = tfla.load_library()
    P = lambda x: ctypes.c_void_p(x * 4096) if x else None
    cf = ctypes.c_float

    def call(y=1, h=1, norm=0, cap=0.0, dqk=256, n_out=1):
        return lib.tfla_mlstm_layer_step(P(1), P(1), P(1), P(1), P(1), None, None, None, P(1), None, None, 2, 8, dqk, 512,
                                         0, 1, cf(1e-6), cf(cap), norm, cf(1e-6), P(y), P(h), P(1), P(n_out), P(1), None)
    assert call(y=0) == -1
    assert call(h=0) == -1
    assert call(n_out=0) == -1
    assert call(norm=3) == -4
    assert call(cap=-2.0) == -2
    assert call(dqk=100) == -2


def test_tile_width_override_changes_workspace_layout_not_validity(tfla):
    lib = tfla.load_library()
    assert lib.tfla_tile_width(96) == -4 and lib.tfla_tile_width(-1) == -4
    a = dict(OK_ARGS); a.pop("direction")
    try:
        auto = tfla.workspace_bytes(1, **a)
        assert lib.tfla_tile_width(64) == 0
        narrow = tfla.workspace_bytes(1, **a)
        # narrower column blocks: more partial row-dot buffers (one per block of the dQ / dK kernels)
        assert narrow > auto
        assert lib.tfla_tile_width(256) == 0
        assert tfla.workspace_bytes(1, **a) == auto
    finally:
        assert lib.tfla_tile_width(0) == 0
    assert tfla.workspace_bytes(1, **a) == auto


def test_error_type_carries_status_and_entry_point(tfla):
    """every binding wrapper raises TflaError(status, entry point): the message names both"""
    e = tfla.TflaError(-4, "tfla_transfer_gain")
    assert e.status == -4 and "tfla_transfer_gain" in str(e) and "unknown variant" in str(e)
    # no wrapper passes anything but (status, name) to the constructor
    src = open(os.path.join(ROOT, "paper_2503_14376_amd", "binding.py")).read()
    for m in re.finditer(r"raise TflaError\(([^)]*)\)", src):
        assert len(m.group(1).split(",")) == 2, m.group(0)


def test_static_entry_point_rejects_before_touching_the_gpu(tfla):
    """tfla_mlstm_fwd_static validates dimensions, the size limit and the pointers before its first HIP call,
    so these codes come back on a machine without a GPU as well"""
    lib = tfla.load_library()
    P = lambda x: ctypes.c_void_p(x * 4096) if x else None
    cf = ctypes.c_float
    assert tfla.static_scratch_bytes() == 64 << 20

    def call(B=1, NH=2, T=256, dqk=64, dhv=128, chunk=64, q=1, H=1, variant=0, dtype=1):
        return lib.tfla_mlstm_fwd_static(P(q), P(1), P(1), P(1), P(1), None, None, None, B, NH, T, dqk, dhv, chunk,
                                         variant, dtype, cf(1e-6), P(H), None, None, None, None, None, None)
    assert call(B=2, NH=8, T=8192, dqk=256, dhv=512, chunk=256) == -7      # needs ~140 MB of scratch memory
    assert "static" in tfla.status_string(-7)
    assert call(chunk=48) == -3
    assert call(dqk=0) == -2
    assert call(variant=5) == -4
    assert call(q=0) == -1
    assert call(H=0) == -1
