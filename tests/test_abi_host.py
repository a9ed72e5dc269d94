"""Host-side checks of the C-ABI library that need no GPU: it loads, exports every
symbol the public header declares, and rejects bad arguments before launching anything."""
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "hbitlinear.h")


@pytest.fixture(scope="module")
def L():
    from paper_2504_18415_amd import hbl
    if not os.path.exists(hbl.LIB_PATH):
        from paper_2504_18415_amd import build
        build.build_library()
    return hbl.lib()


def declared_functions():
    src = open(HEADER).read()
    src = re.sub(r"/\*.*?\*/", "", src, flags=re.S)
    return sorted(set(re.findall(r"\b(hbl_[a-z0-9_]+)\s*\(", src)))


def test_every_declared_symbol_is_exported(L):
    from paper_2504_18415_amd import hbl
    names = declared_functions()
    assert len(names) >= 12
    for n in names:
        assert hasattr(L, n), n
    assert sorted(hbl.EXPORTS) == names
    for n in hbl.TEST_EXPORTS:                      # test-suite exports: csrc/hbl_test_exports.h, not the public header
        assert hasattr(L, n) and n not in names, n
    test_hdr = open(os.path.join(ROOT, "paper_2504_18415_amd", "csrc", "hbl_test_exports.h")).read()
    test_hdr = re.sub(r"/\*.*?\*/", "", test_hdr, flags=re.S)
    assert sorted(set(re.findall(r"\b(hbl_[a-z0-9_]+)\s*\(", test_hdr))) == sorted(hbl.TEST_EXPORTS)


def test_status_text(L):
    for st in range(0, -8, -1):
        assert L.hbl_strerror(st) and L.hbl_strerror(st) != b"unknown status"
    assert L.hbl_strerror(-99) == b"unknown status"


def test_size_queries(L):
    assert L.hbl_packed_bytes(4096, 16384) == 4096 * 16384 // 4 + 4 * 4096   # 2 bits per weight + int32 row sums
    assert L.hbl_packed_bytes(256, 256) == 16384 + 1024
    ws = L.hbl_workspace_bytes(8192, 16384, 4096, 4)
    assert ws >= 8192 * 16384 + 4 * 8192 and ws % 256 == 0
    assert L.hbl_workspace_bytes(17, 256, 256, 8) >= 17 * 256 + 4 * 17
    assert L.hbl_workspace_bytes(17, 256, 0, 8) == 256 and L.hbl_workspace_bytes(17, 256, -32, 8) == 256
    # the sizes that were told when a mid-size batch on a long K left partial tiles (4 slices of [T, N] int32 here) still are
    assert L.hbl_workspace_bytes(256, 16384, 4096, 4) >= 256 * 16384 + 4 * 256 * 4096 * 4
    assert L.hbl_workspace_bytes(256, 4096, 4096, 4) < 256 * 4096 + 256 * 4096 * 4
    assert L.hbl_ternarize_workspace_bytes(4096, 16384) >= 8
    assert L.hbl_ternarize_workspace_bytes(4096, 16384) <= 4096 * 16384 // 16


def test_argument_errors_before_any_launch(L):
    from paper_2504_18415_amd import hbl
    P = ctypes.c_void_p(0x10000)       # never dereferenced: every call below fails validation first
    NUL = ctypes.c_void_p(0)
    ok_ws = 1 << 30

    def fwd(fn=L.hbl_hbitlinear_forward, x=P, dt=hbl.BF16, T=4, K=256, w=P, N=64, sc=P, g=1, bits=4, y=P, ws=P,
            wsb=ok_ws):
        return fn(x, dt, T, K, w, N, sc, g, bits, 1e-5, y, ws, wsb, None)

    assert fwd(bits=5) == hbl.E_BITS
    assert fwd(dt=7) == hbl.E_DTYPE
    assert fwd(K=192) == hbl.E_SHAPE                      # Hadamard needs a power of two
    assert fwd(K=64) == hbl.E_SHAPE
    assert fwd(K=32768) == hbl.E_SHAPE
    assert fwd(K=200) == hbl.E_SHAPE
    assert fwd(N=48) == hbl.E_SHAPE
    assert fwd(T=-1) == hbl.E_SHAPE
    assert fwd(g=3) == hbl.E_SHAPE                        # 64 rows do not split into 3 groups
    assert fwd(N=96, g=3) != hbl.E_SHAPE
    assert fwd(x=NUL) == hbl.E_NULL
    assert fwd(w=NUL) == hbl.E_NULL
    assert fwd(sc=NUL) == hbl.E_NULL
    assert fwd(y=NUL) == hbl.E_NULL
    assert fwd(ws=NUL) == hbl.E_NULL
    assert fwd(x=ctypes.c_void_p(0x10004)) == hbl.E_ALIGN
    assert fwd(ws=ctypes.c_void_p(0x10010)) == hbl.E_ALIGN
    assert fwd(wsb=100) == hbl.E_WORKSPACE
    assert fwd(T=0, x=NUL, y=NUL) == hbl.OK              # empty batch is a no-op
    assert fwd(fn=L.hbl_plain_bitlinear_forward, K=384, wsb=100) == hbl.E_WORKSPACE   # K=384 is fine without Hadamard
    assert L.hbl_fwht_quant(P, hbl.BF16, 4, 256, 3, 1e-5, 1, 0, P, P, P, None) == hbl.E_BITS
    assert L.hbl_fwht_quant(P, hbl.BF16, 4, 256, 8, 1e-5, 1, 8, P, P, P, None) == hbl.E_BITS   # offset 8 is INT4 only
    assert L.hbl_fwht_quant(NUL, hbl.BF16, 4, 256, 4, 1e-5, 1, 0, P, P, P, None) == hbl.E_NULL
    ln = lambda g=P, had=1, K=256, bits=4: L.hbl_ln_bitlinear_forward(P, hbl.BF16, 4, K, g, 1e-6, had, P, 64, P, 1, bits,
                                                                    1e-5, P, P, ok_ws, None)
    assert ln(g=NUL) == hbl.E_NULL
    assert ln(g=ctypes.c_void_p(0x10004)) == hbl.E_ALIGN
    assert ln(K=384) == hbl.E_SHAPE
    assert ln(K=384, had=0, bits=7) == hbl.E_BITS
    assert L.hbl_ln_fwht_quant(P, hbl.BF16, 4, 256, NUL, 1e-6, 4, 1e-5, 1, 0, P, P, P, None) == hbl.E_NULL
    assert L.hbl_ln_fwht_quant(P, hbl.BF16, 4, 256, P, 1e-6, 8, 1e-5, 1, 8, P, P, P, None) == hbl.E_BITS
    assert L.hbl_fwht(P, hbl.BF16, 4, 384, P, hbl.F32, None) == hbl.E_SHAPE     # power of two only
    assert L.hbl_fwht(P, hbl.BF16, 4, 256, P, 5, None) == hbl.E_DTYPE
    assert L.hbl_fwht(P, hbl.BF16, 4, 256, NUL, hbl.F32, None) == hbl.E_NULL
    assert L.hbl_fwht(NUL, hbl.BF16, 0, 256, NUL, hbl.F32, None) == hbl.OK
    assert L.hbl_gemm_i32(P, 4, 100, P, 64, P, None) == hbl.E_SHAPE
    assert L.hbl_pack_ternary_2bit(P, 33, 256, P, None) == hbl.E_SHAPE
    assert L.hbl_pack_ternary_2bit(NUL, 32, 256, P, None) == hbl.E_NULL
    assert L.hbl_ternarize_weights_absmean(P, 0, 5, 1e-5, P, P, P, 8, None) == hbl.E_SHAPE
    assert L.hbl_ternarize_weights_absmean(P, 4, 4, 1e-5, P, P, P, 0, None) == hbl.E_WORKSPACE


def test_grouped_call_argument_errors_before_any_launch(L):
    from paper_2504_18415_amd import hbl
    P, NUL = 0x10000, 0

    def prob(x=P, dt=hbl.BF16, bits=4, had=1, T=4, K=256, N=64, w=P, sc=P, g=1, y=P):
        return hbl.Problem(x, dt, bits, had, 0, T, K, N, w, sc, g, y)

    def call(ps, ws=P, wsb=1 << 30):
        arr = (hbl.Problem * max(len(ps), 1))(*ps)
        return L.hbl_bitlinear_forward_grouped(arr, len(ps), 1e-5, ctypes.c_void_p(ws), wsb, None)

    assert call([]) == hbl.OK
    assert L.hbl_bitlinear_forward_grouped(None, 2, 1e-5, ctypes.c_void_p(P), 1 << 30, None) == hbl.E_NULL
    assert L.hbl_bitlinear_forward_grouped(None, -1, 1e-5, ctypes.c_void_p(P), 1 << 30, None) == hbl.E_SHAPE
    assert call([prob(), prob(bits=3)]) == hbl.E_BITS
    assert call([prob(), prob(dt=9)]) == hbl.E_DTYPE
    assert call([prob(K=384)]) == hbl.E_SHAPE            # Hadamard needs a power of two
    assert call([prob(K=384, had=0)], wsb=100) == hbl.E_WORKSPACE
    assert call([prob(y=NUL)]) == hbl.E_NULL
    assert call([prob()], ws=NUL) == hbl.E_NULL
    assert call([prob()], ws=P + 16) == hbl.E_ALIGN
    assert call([prob(x=P + 4)]) == hbl.E_ALIGN
    assert call([prob(T=0, x=NUL, y=NUL)], ws=NUL, wsb=0) == hbl.OK     # nothing to do
    arr = (hbl.Problem * 2)(prob(T=8, K=4096, N=4096), prob(T=200, K=1024, N=256))
    need = L.hbl_grouped_workspace_bytes(arr, 2)
    assert need >= 8 * 4096 + 200 * 1024 and need % 256 == 0
    assert need >= L.hbl_workspace_bytes(8, 4096, 4096, 4) + L.hbl_workspace_bytes(200, 1024, 256, 4)
    assert call(list(arr), wsb=need - 256) == hbl.E_WORKSPACE


def test_binding_fails_loudly_without_library(monkeypatch, tmp_path):
    from paper_2504_18415_amd import hbl
    monkeypatch.setattr(hbl, "_lib", None)
    monkeypatch.setattr(hbl, "LIB_PATH", str(tmp_path / "missing.so"))
    with pytest.raises(ImportError):
        hbl.lib()


@pytest.fixture()
def build_in(monkeypatch, tmp_path):
    """The build with its outputs under tmp_path and compilers that only write their output file; returns (module, commands run)."""
    from paper_2504_18415_amd import build
    ran = []

    def run(cmd, verbose):
        ran.append(cmd)
        with open(cmd[cmd.index("-o") + 1], "w") as f:
            f.write("built")
    monkeypatch.setattr(build, "PKG", str(tmp_path))
    monkeypatch.setattr(build, "OBJ_DIR", str(tmp_path / "_build"))
    monkeypatch.setattr(build, "LIB", str(tmp_path / "libhbitlinear.so"))
    monkeypatch.setattr(build, "HOST_CALL", str(tmp_path / os.path.basename(build.HOST_CALL)))
    monkeypatch.setattr(build, "_run", run)
    return build, ran


def test_library_is_built_without_the_native_half(build_in, monkeypatch, tmp_path, capsys):
    """The module is optional: where it cannot be compiled the library is linked all the same, and no module of another build stays."""
    build, ran = build_in
    run = build._run

    def without_gxx(cmd, verbose):
        if any("host_call" in word for word in cmd):
            raise RuntimeError("no compiler")
        run(cmd, verbose)
    monkeypatch.setattr(build, "_run", without_gxx)
    for old in ("_host_call.so", os.path.basename(build.HOST_CALL)):
        (tmp_path / old).write_text("of another build")
    assert build.build_library() == build.LIB and os.path.exists(build.LIB)
    assert not [f for f in os.listdir(tmp_path) if "host_call" in f] and "no compiler" in capsys.readouterr().err
    monkeypatch.setattr(build, "_host_call_command", lambda out: (_ for _ in ()).throw(ImportError("no torch")))
    os.remove(build.LIB)
    assert build.build_library(incremental=True) == build.LIB and os.path.exists(build.LIB)


def test_native_half_is_built_again_for_another_torch(build_in, monkeypatch):
    build, ran = build_in
    hosts = lambda: sum(any("host_call" in word for word in cmd) for cmd in ran)
    build.build_library()
    assert hosts() == 1 and open(build.HOST_CALL).read() == "built"
    build.build_library(incremental=True)
    assert hosts() == 1                                                          # nothing changed
    import torch
    monkeypatch.setattr(torch, "__version__", "0.0.0+another")
    build.build_library(incremental=True)
    assert hosts() == 2
    assert "cpython" in os.path.basename(build.HOST_CALL)                        # and another Python does not see this file


def test_native_half_of_another_torch_is_not_used(L, monkeypatch):
    from paper_2504_18415_amd import hbl, _host_call
    monkeypatch.setattr(hbl, "_call", None)
    monkeypatch.setattr(_host_call, "built_for", "0.0.0+another")
    hbl._bind_native(L)
    assert hbl._call is None
    monkeypatch.undo()
    hbl._bind_native(L)
    assert hbl._call is _host_call


def test_short_arrays_never_reach_the_library(L, monkeypatch):
    """Head states and transform into callers' arrays: what would be read or written out of range is refused before any launch."""
    import torch
    from paper_2504_18415_amd import hbl

    class NoLaunch:
        hbl_kv_packed_bytes = L.hbl_kv_packed_bytes

        def __getattr__(self, name):
            raise AssertionError(name + " was called")
    monkeypatch.setattr(hbl, "_lib", NoLaunch())
    monkeypatch.setattr(hbl, "_call", None)
    monkeypatch.setattr(hbl, "_dev_check", lambda *ts: None)                    # (CPU tensors stand in for device ones)
    x = torch.zeros(4, 64)
    packed, scales = torch.zeros(4, 32, dtype=torch.uint8), torch.zeros(4)
    for call in (lambda: hbl.kv_dequant(packed, scales, 64, 4, out_dtype=torch.float16),          # two bytes where four are written
                 lambda: hbl.kv_dequant(packed, scales, 64, 4, out=torch.zeros(4, 32)), lambda: hbl.kv_dequant(packed[:3], scales, 64, 4),
                 lambda: hbl.kv_dequant(packed, scales, 128, 4), lambda: hbl.kv_dequant(packed, scales.to(torch.bfloat16), 64, 4),
                 lambda: hbl.kv_quant_absmax(x, 4, packed=packed[:3], scales=scales), lambda: hbl.kv_quant_absmax(x, 8, packed=packed),
                 lambda: hbl.kv_quant_absmax(x, 4, scales=scales[:3]), lambda: hbl.kv_quant_absmax(x, 4, scales=scales.to(torch.bfloat16)),
                 lambda: hbl.fwht(torch.zeros(4, 128), out=torch.zeros(3, 128))):
        with pytest.raises(ValueError):
            call()


def test_outputs_are_plain_tensors_whatever_the_input_is(L, monkeypatch):
    """Outputs that the binding allocates: plain tensors, also for a Parameter or another subclass."""
    torch = pytest.importorskip("torch")
    from paper_2504_18415_amd import hbl

    class Tagged(torch.Tensor):
        pass

    monkeypatch.setattr(hbl, "_dev_check", lambda *tensors: None)
    monkeypatch.setattr(hbl, "_stream", lambda: 0)
    x, packed = torch.zeros((2, 128)), torch.zeros(32 * 128 // 4 + 4 * 32, dtype=torch.uint8)
    for t in (x, torch.nn.Parameter(x), x.as_subclass(Tagged)):
        sizes = []
        y = hbl._forward(lambda *args: sizes.append(args[-2]) or 0, "stub", t, packed, 32, torch.ones(1), 4, 1e-5, None, None)
        assert type(y) is torch.Tensor and y.shape == (2, 32) and y.dtype == torch.bfloat16 and not y.requires_grad
        assert sizes == [hbl.workspace_bytes(2, 128, 32, 4)]


def test_small_batch_launch_plan(L):
    """Host logic of the decode path as the calls take it: kernel, K splits and grid sizes for the 7B layer and a few odd
    shapes."""
    from paper_2504_18415_amd import hbl
    layer = lambda B, h=4096, m=16384: [(B, h, 3 * h, False), (B, h, h, True), (B, h, 2 * m, False), (B, m, h, True)]
    # batch <= 16: streaming form; 2048 wave-units of 32 weight tiles = 512 workgroups = two per CU, no reduction
    for B in (1, 8, 16):
        for bits in (4, 8):
            assert hbl.grouped_plan(layer(B), bits) == ("stream", [1, 1, 1, 4], 96 + 32 + 256 + 128, 0)
    # 17 to 32 tokens of records, more tiles than fit at once: shared form; only the K = 16384 problem is split, over
    # workgroups: one arrival counter per group of four row tiles of it
    assert hbl.grouped_plan(layer(32)) == ("stream", [1, 1, 1, 4], 512, 4096 // 128)
    # everything else above 16 tokens is the mid-size kernel's: more tokens, INT8, fewer tiles
    for shapes, bits in ((layer(33), 4), (layer(64), 4), (layer(32), 8), (layer(24, 2048, 8192), 4), ([(32, 16384, 4096, True)], 4),
                         ([(40, 8192, 160, True)], 4), ([(20, 256, 32768, True), (20, 512, 32768, True)], 4)):
        assert hbl.grouped_plan(shapes, bits) == ("mid", [0] * len(shapes), 0, 0)
    # ... but for short rows of bytes that do not fit at once
    assert hbl.grouped_plan([(32, 1024, 16448, True), (17, 512, 16448, True)], 8) == ("stream", [1, 1], 2 * 129, 0)
    # a single small problem is split down to 8 tiles per wave to reach more CUs
    assert hbl.grouped_plan([(4, 4096, 4096, True)]) == ("stream", [4], 128, 0)
    # W_down alone: 128 row tiles and 128 K blocks - the 8 waves of a wider workgroup share a row tile's K range
    for T in (8, 16):
        assert hbl.grouped_plan([(T, 16384, 4096, True)]) == ("stream", [8], 128, 0)
    assert hbl.grouped_plan([(4, 128, 96, False)]) == ("stream", [1], 1, 0)        # one K block: nothing to split
    # as many split row groups as a slot has arrival counters; with more the group runs without the split
    assert hbl.grouped_plan([(32, 8192, 128 * 2048, True)]) == ("stream", [2], 2 * 2048, 2048)
    assert hbl.grouped_plan([(32, 8192, 128 * 2049, True)]) == ("stream", [1], 2049, 0)
    with pytest.raises(hbl.HblError):
        hbl.grouped_plan([(65, 4096, 4096, True)])
    with pytest.raises(hbl.HblError):
        hbl.grouped_plan([(4, 4096 + 128, 4096, True)])


def test_one_launch_only_where_it_is_no_slower(L):
    """One launch for one to four tokens repeats the quantisation in every workgroup: it is taken up to as many workgroups
    per CU as measured no slower than two launches, not wherever it fits the chip at once."""
    from paper_2504_18415_amd import hbl
    fused = lambda T, K, N, had, dt=hbl.BF16: hbl.forward_route(T, K, N, 4, had, dt) == "fused"
    for N in (96, 4096, 12288):                                    # the projections of a decode step, batch 1
        assert fused(1, 4096, min(N, 8192), True) and fused(1, 4096, N, False) and fused(1, 1024, N, False)
    assert fused(1, 16384, 4096, True) and fused(1, 4096, 32768, False) and fused(4, 2048, 4096, True)
    for T, K, N, had in [(1, 1024, 32768, True), (2, 512, 65536, True), (4, 2048, 32768, True), (1, 512, 131072, False),
                         (2, 640, 32768, False), (3, 512, 12288, False), (3, 1024, 32768, False), (4, 512, 32, False),
                         (4, 640, 12288, False), (4, 1024, 8192, False), (4, 2048, 12288, False)]:
        for dt in (hbl.BF16, hbl.F32):
            assert not fused(T, K, N, had, dt), (T, K, N, had, dt)   # 1.05 to 1.6 times the two launches
    assert hbl.forward_route(1, 4096, 4096, 8) == "stream" and hbl.forward_route(1, 4096, 4096, 4, norm=True) == "stream"
    with pytest.raises(hbl.HblError):
        hbl.forward_route(0, 4096, 4096)


def test_one_launch_for_short_rows_with_the_norm(L):
    """With the norm every workgroup repeats more, so its lines lie closer; without it they are where they were."""
    from paper_2504_18415_amd import hbl
    one = lambda T, K, N, bits, had, norm: hbl.forward_route(T, K, N, bits, had, hbl.BF16, norm) == "fused_bytes"
    for norm in (False, True):                                     # the same on both
        for T, K, N, bits, had in ((16, 1920, 8192, 4, False), (12, 2560, 8192, 4, False), (9, 3456, 8192, 4, False), (8, 1536, 16384, 4, False),
                                   (8, 2048, 8192, 4, False), (7, 1024, 16384, 4, True), (12, 3072, 4096, 4, False), (8, 2048, 4096, 4, True), (16, 3584, 8192, 8, False),
                                   (8, 2944, 16384, 8, False), (5, 3584, 16384, 8, False), (3, 1024, 32768, 4, True), (16, 1024, 8192, 8, True),
                                   (4, 2048, 16384, 4, False)):
            if norm or not (T <= 4 and bits == 4):                 # (without the norm those are fused_small.hip's or two launches)
                assert one(T, K, N, bits, had, norm), (T, K, N, bits, had, norm)
    for T, K, N, bits, had in ((16, 2048, 4128, 4, False), (12, 2688, 4128, 4, False), (9, 3584, 4128, 4, False), (16, 2432, 32, 4, False), (8, 1664, 8224, 4, False),
                               (8, 1024, 8224, 4, True), (5, 2048, 4128, 4, True), (8, 3072, 8224, 8, False)):   # up to 1.21 times the two launches
        assert one(T, K, N, bits, had, False) and not one(T, K, N, bits, had, True), (T, K, N, bits, had)


def test_one_plain_token_of_more_than_4096_features(L):
    """Rows of up to 8192 by eight waves, two workgroups of 32 output rows a CU; longer ones by sixteen, 16 rows, two where LDS has
    room for them."""
    from paper_2504_18415_amd import hbl
    route = lambda K, N, dt=hbl.BF16: hbl.forward_route(1, K, N, 4, False, dt)
    for dt in (hbl.BF16, hbl.F32):
        assert route(4224, 16384, dt) == "fused" and route(4224, 16416, dt) == "stream"
        assert route(5376, 12288, dt) == route(8192, 8192, dt) == "fused" and route(8192, 8224, dt) == "stream"
        assert route(11008, 4096, dt) == route(16256, 4096, dt) == "fused" and route(11008, 4128, dt) != "fused"
    assert route(8320, 8192) == "fused" and route(8320, 8224) != "fused" and route(8320, 4128, hbl.F32) != "fused"


def test_single_calls_of_up_to_16_tokens_stream_or_not(L):
    """Long K ranges that few waves share: the mid-size kernel up to 128 workgroups of the streaming one, where it is the
    faster; beyond them records stream, bytes from 192 on."""
    from paper_2504_18415_amd import hbl
    route = lambda K, N, bits: hbl.forward_route(8, K, N, bits, hadamard=False)
    assert route(11008, 8192, 4) == "mid" and route(11008, 8224, 4) == "stream"      # 86 K-blocks: two pieces
    assert route(16256, 16384, 4) == "mid" and route(16256, 16512, 4) == "stream"    # 127: one
    assert route(16256, 24448, 8) == "mid" and route(16256, 24576, 8) == "stream"
    assert route(4096, 4096, 4) == route(4096, 4096, 8) == "stream" and route(16384, 4096, 4) == "stream"


def test_routes_of_17_to_64_tokens_against_many_output_rows(L):
    """More than 512 tiles of 64 x 64: records of up to 32 tokens stream in the shared form where it is the faster, short rows
    of bytes take the int8 kernel's narrow tiles; everything else is the mid-size kernel's."""
    from paper_2504_18415_amd import hbl
    route = lambda T, K, N, bits: hbl.forward_route(T, K, N, bits, hadamard=False)
    for T in (17, 32):
        assert route(T, 512, 32768, 4) == "mid" and route(T, 512, 32800, 4) == "stream"
        assert route(T, 8064, 131072, 4) == "stream" and route(T, 8192, 45056, 4) == "stream"
        assert route(T, 8192, 45088, 4) == "mid" and route(T, 12288, 40960, 4) == "mid"
    for T in (17, 32, 33, 64):
        for K, bits in ((128, 8), (384, 8), (384, 4)):
            assert route(T, K, 32768, bits) == "mid" and route(T, K, 32800, bits) == "prefill"
        assert route(T, 512, 65536, 8) == ("prefill" if T <= 32 else "mid") and route(T, 1024, 65568, 8) == "prefill"
        assert route(T, 1152, 32800, 8) == "mid"
    assert route(33, 512, 131072, 4) == route(64, 4096, 131072, 4) == "mid"


def test_route_names_the_kernel_that_runs_for_large_byte_tiles(L):
    """Bytes of more than 64 tokens: while all 128 x 64 tiles are resident at once, and up to 384 tiles of 128 x 128 where rows are
    512 to 1536 long, they are the mid-size kernel's, and the route says so.  Beyond that short rows take the small tile."""
    from paper_2504_18415_amd import hbl
    def tile(T, K, N, bits=8):
        t = hbl.gemm_tile(T, K, N, hbl.CODES_INT8 if bits == 8 else hbl.CODES_UINT4_PLUS8)
        assert hbl.forward_route(T, K, N, bits, hadamard=False) == ("mid" if t == hbl.TILE_MID else "prefill"), (T, K, N, bits)
        return t
    for bits, K in ((8, 8192), (8, 2048), (8, 640), (8, 128), (4, 384)):
        for T, N in ((2048, 2048), (1000, 2208), (2048, 2048), (64 + 1, 32768), (291, 12384)):   # at most 512 of 128 x 64
            assert tile(T, K, N, bits) == hbl.TILE_MID, (T, K, N, bits)
    for K in (512, 1024, 1536):
        assert tile(1536, K, 4096) == hbl.TILE_MID and tile(1536, K, 4128) != hbl.TILE_MID       # 384 tiles and 396
    assert tile(1536, 1664, 4096) == hbl.TILE_HALF and tile(346, 14464, 11424) == hbl.TILE_HALF
    for K, bits in ((128, 8), (384, 8), (384, 4)):
        assert tile(1536, K, 4096, bits) == hbl.TILE_SMALL
    for K in (128, 256, 384):
        assert tile(1099, K, 6912) == tile(2048, K, 8192) == tile(8192, K, 8192) == hbl.TILE_SMALL
    assert tile(1099, 1024, 6912) == tile(1536, 1024, 8192) == hbl.TILE_SMALL != tile(1099, 1152, 6912)      # 486, 768 tiles
    assert tile(1536, 512, 8224) == tile(2048, 512, 8192) == hbl.TILE_HALF                                   # 780, 1024
    assert tile(8192, 16384, 4096) == hbl.TILE_WIDE
    assert hbl.forward_route(2048, 2048, 2048, 4, hadamard=False) == "prefill"                   # records: prefill tiles
    for T, K, N, form in ((0, 512, 64, hbl.CODES_INT8), (4, 384, 64, hbl.CODES_BF6), (4, 100, 64, hbl.CODES_INT8)):
        with pytest.raises(hbl.HblError):
            hbl.gemm_tile(T, K, N, form)


def test_tiles_of_code_records(L):
    """At most two small workgroups a CU: one tile of 128 x 128 with four stages, then 192 x 128 with two or four, then 128 x 128 with
    two; beyond that the least estimate, on both sides of where it changes."""
    from paper_2504_18415_amd import hbl
    tile = lambda T, K, N: hbl.gemm_tile(T, K, N, hbl.CODES_BF6)
    assert tile(1000, 640, 2080) == hbl.TILE_SMALL and tile(512, 640, 2048) == hbl.TILE_MID
    assert tile(2048, 640, 2048) == hbl.TILE_SMALL and tile(2049, 640, 2048) == hbl.TILE_NARROW                # 256 tiles and 272
    assert tile(2049, 3072, 2048) == hbl.TILE_NARROW and tile(2049, 3200, 2048) == hbl.TILE_NARROW_DEEP
    assert tile(2048, 640, 3072) == hbl.TILE_NARROW and tile(2048, 640, 3104) == hbl.TILE_SMALL_FLAT           # 256 of 192 x 128, 272
    assert tile(2048, 512, 4096) == hbl.TILE_SMALL_FLAT and tile(4096, 512, 4096) == hbl.TILE_HALF             # 512, 1024
    assert tile(8192, 16384, 4096) == tile(8192, 4096, 12288) == hbl.TILE_WIDE


def test_kv_quant_argument_errors_before_any_launch(L):
    from paper_2504_18415_amd import hbl
    E = {n: getattr(hbl, n) for n in ("E_NULL", "E_SHAPE", "E_BITS", "E_DTYPE", "E_ALIGN")}
    assert L.hbl_kv_packed_bytes(10, 128, 8) == 1280 and L.hbl_kv_packed_bytes(10, 128, 4) == 640
    assert L.hbl_kv_packed_bytes(10, 128, 3) == 480 and L.hbl_kv_packed_bytes(10, 96, 4) == 0
    assert L.hbl_kv_packed_bytes(10, 128, 5) == 0
    a = 4096   # a non-null, 16-byte aligned stand-in address: every call below must fail before touching it
    q = lambda x, dt, rows, d, bits, p, s: L.hbl_kv_quant_absmax(x, dt, rows, d, bits, 1e-5, p, s, None)
    assert q(a, hbl.BF16, 4, 128, 5, a, a) == E["E_BITS"]
    assert q(a, 7, 4, 128, 4, a, a) == E["E_DTYPE"]
    assert q(a, hbl.BF16, 4, 96, 4, a, a) == E["E_SHAPE"]
    assert q(a, hbl.BF16, -1, 128, 4, a, a) == E["E_SHAPE"]
    assert q(a, hbl.BF16, 1 << 31, 128, 4, a, a) == E["E_SHAPE"]
    assert q(None, hbl.BF16, 4, 128, 4, a, a) == E["E_NULL"]
    assert q(a, hbl.BF16, 4, 128, 4, a, None) == E["E_NULL"]
    assert q(a + 4, hbl.BF16, 4, 128, 4, a, a) == E["E_ALIGN"]
    assert q(None, hbl.BF16, 0, 128, 4, None, None) == 0                      # no rows: nothing to do
    dq = lambda p, s, rows, d, bits, o, dt: L.hbl_kv_dequant(p, s, rows, d, bits, o, dt, None)
    assert dq(a, a, 4, 128, 2, a, hbl.BF16) == E["E_BITS"]
    assert dq(a, a, 4, 128, 3, a, 9) == E["E_DTYPE"]
    assert dq(a, a, 4, 1024, 3, a, hbl.F32) == E["E_SHAPE"]
    assert dq(a, None, 4, 128, 3, a, hbl.F32) == E["E_NULL"]
    assert dq(a, a, 4, 128, 3, a + 8, hbl.F32) == E["E_ALIGN"]
    assert dq(None, None, 0, 128, 3, None, hbl.F32) == 0


def test_trace_calls_without_a_gpu(L):
    """The timing trace is host state: opening, nesting and closing it needs no device (events are created
    lazily only when a count is asked for, so keep it to the error paths here)."""
    n = ctypes.c_int(-1)
    assert L.hbl_trace_end(None, None, 0, ctypes.byref(n)) == -2          # no open trace
    assert L.hbl_trace_begin(0) == -2 and L.hbl_trace_begin(-5) == -2


def test_raw_accumulator_exports_reject_bad_arguments(L):
    P = ctypes.c_void_p(0x10000)
    NUL = ctypes.c_void_p(0)
    f = L.hbl_gemm_i32_bf6
    assert f(P, 128, 256, P, 64, P, P, 1 << 30, NUL) == -2                 # records need K >= 512
    assert f(P, 128, 1024, P, 48, P, P, 1 << 30, NUL) == -2                # N not a multiple of 32
    assert f(NUL, 128, 1024, P, 64, P, P, 1 << 30, NUL) == -1
    assert f(P, 128, 1024, P, 64, P, P, 16, NUL) == -5                     # workspace too small
    assert f(P, 0, 1024, P, 64, P, P, 0, NUL) == 0                         # empty batch
    g = L.hbl_test_gemm_i32_tile
    assert g(P, 6, 32, 1024, P, 64, P, 1, NUL) == -2                       # prefill tiles: T > 64
    assert g(P, 8, 128, 1024, P, 64, P, 1, NUL) == -3                      # code form
    assert g(P, 6, 128, 1024, P, 64, P, 7, NUL) == -2                      # tile
    assert g(P, 0, 128, 1024, P, 64, P, 3, NUL) == -2                      # the mid-size kernel: records only here
