"""Host-side tests of the C-ABI library that need no GPU: the library loads, exports every symbol the
header declares, and rejects bad arguments with the documented status before any HIP call."""
import ctypes as C
import os
import re

import numpy as np
import pytest

import oracle
import paper_2503_17513_amd as pme

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
OK, NULL, SHAPE, ORDER, ALIGN, WORKSPACE, DTYPE, HIP, PATH, COLD = range(10)
FAKE = 0x10000   # a non-null, 64 KiB aligned address that is never dereferenced: every call below fails validation


def test_header_symbols_are_exported():
    with open(os.path.join(ROOT, "include", "pme.h")) as f:
        text = f.read()
    declared = set(re.findall(r"\b(pme_[a-z0-9_]+)\s*\(", text))
    assert declared == set(pme.EXPORTS)
    L = pme.lib()
    for name in declared:
        assert hasattr(L, name), name
    assert pme.version() >= 100
    assert L.pme_status_string(OK) == b"ok"
    for s in range(1, 10):
        assert L.pme_status_string(s) not in (b"ok", b"unknown status")


def test_factor_order_matches_oracle():
    for M in (80, 2176, 8704, 8448, 15360, 64, 8960, 9728, 10240, 12288, 18432, 19968, 22016, 24, 40):
        assert pme.factor_order(M) == oracle.factor_order(M)
    for bad in (7, 100, 11264, 0, -4):
        with pytest.raises(pme.PmeError) as e:
            pme.factor_order(bad)
        assert e.value.status == ORDER


def test_base_block_matches_oracle():
    for b in oracle.SUPPORTED_BASE:
        assert np.array_equal(pme.base_block(b), oracle.paley_block(b))
    out = np.zeros((16, 16), np.int8)
    assert pme.lib().pme_base_block(16, out.ctypes.data) == ORDER
    assert pme.lib().pme_base_block(20, None) == NULL


def test_rotate_argument_errors():
    f = pme.lib().pme_hadamard_expand_quant
    good = dict(x=FAKE, xt=1, T=4, d=64, ldx=64, d_e=80, qx=FAKE, sx=FAKE, stream=None)

    def call(**kw):
        a = dict(good, **kw)
        return f(a["x"], a["xt"], a["T"], a["d"], a["ldx"], a["d_e"], a["qx"], a["sx"], a["stream"])

    assert call(x=None) == NULL
    assert call(qx=None) == NULL
    assert call(sx=None) == NULL
    assert call(xt=5) == DTYPE
    assert call(T=-1) == SHAPE
    assert call(d=0) == SHAPE
    assert call(d=81) == SHAPE            # d > d_e
    assert call(ldx=63) == SHAPE          # pitch smaller than d
    assert call(d_e=81, d=64) == SHAPE    # odd d_e
    assert call(d_e=100) == ORDER
    assert call(d_e=11264, d=64) == ORDER
    assert call(x=FAKE + 1) == ALIGN
    assert call(xt=0, x=FAKE + 2) == ALIGN
    assert call(qx=FAKE + 2) == ALIGN
    assert call(sx=FAKE + 2) == ALIGN
    assert call(T=0, x=None, qx=None, sx=None) == OK      # empty input: no-op


def test_gemm_argument_errors():
    f = pme.lib().pme_w4a4_gemm

    def call(qx=FAKE, sx=FAKE, qw=FAKE, sw=FAKE, T=4, d_e=80, N=8, y=FAKE, ldy=8):
        return f(qx, sx, qw, sw, T, d_e, N, y, ldy, None)

    assert call(qx=None) == NULL
    assert call(qw=None) == NULL
    assert call(sx=None) == NULL
    assert call(sw=None) == NULL
    assert call(y=None) == NULL
    assert call(T=-2) == SHAPE
    assert call(N=-1) == SHAPE
    assert call(d_e=0) == SHAPE
    assert call(d_e=81) == SHAPE
    assert call(ldy=7) == SHAPE
    assert call(qx=FAKE + 1) == ALIGN
    assert call(qw=FAKE + 3) == ALIGN
    assert call(y=FAKE + 1) == ALIGN
    assert call(T=0) == OK
    assert call(N=0, ldy=0) == OK
    g = pme.lib().pme_w4a4_gemm_i32
    assert g(FAKE, FAKE, 4, 80, 8, None, None) == NULL
    assert g(FAKE, FAKE, 4, 81, 8, FAKE, None) == SHAPE


def test_expanded_linear_argument_errors():
    f = pme.lib().pme_expanded_linear
    need = pme.workspace_bytes(4, 64, 80, 8)
    assert need == 256 + 256 + 256
    # codes + MXFP4 scale bytes (the larger of the two scale kinds) + zero points of the asymmetric variant
    assert pme.workspace_bytes(2048, 2048, 2176, 3072) == 2048 * 1088 + 2048 * 68 + 2048 * 4
    assert pme.workspace_bytes(4, 81, 80, 8) == 0

    def call(x=FAKE, xt=1, T=4, d=64, ldx=64, d_e=80, qw=FAKE, sw=FAKE, N=8, y=FAKE, ldy=8, ws=FAKE, wsb=need):
        return f(x, xt, T, d, ldx, d_e, qw, sw, N, y, ldy, ws, wsb, None)

    assert call(wsb=need - 1) == WORKSPACE
    assert call(ws=None) == NULL
    assert call(ws=FAKE + 64) == ALIGN
    assert call(qw=None) == NULL
    assert call(d_e=100) == ORDER
    assert call(xt=9) == DTYPE
    assert call(ldy=4) == SHAPE
    assert call(T=0, x=None, ws=None, wsb=0) == OK


def test_mxfp4_and_weight_argument_errors():
    L = pme.lib()
    f = L.pme_hadamard_expand_quant_mxfp4
    assert f(None, 1, 4, 64, 64, 96, FAKE, FAKE, None) == NULL
    assert f(FAKE, 1, 4, 64, 64, 96, None, FAKE, None) == NULL
    assert f(FAKE, 1, 4, 64, 64, 96, FAKE, None, None) == NULL
    assert f(FAKE, 1, 4, 64, 64, 80, FAKE, FAKE, None) == SHAPE           # d_e not a multiple of 32
    assert f(FAKE, 1, 4, 64, 64, 100, FAKE, FAKE, None) == ORDER
    assert f(FAKE, 3, 4, 64, 64, 96, FAKE, FAKE, None) == DTYPE
    assert f(None, 1, 0, 64, 64, 96, None, None, None) == OK
    g = L.pme_mxfp4_gemm
    assert g(None, FAKE, FAKE, FAKE, 4, 96, 8, FAKE, 8, None) == NULL
    assert g(FAKE, None, FAKE, FAKE, 4, 96, 8, FAKE, 8, None) == NULL
    assert g(FAKE, FAKE, FAKE, None, 4, 96, 8, FAKE, 8, None) == NULL
    assert g(FAKE, FAKE, FAKE, FAKE, 4, 80, 8, FAKE, 8, None) == SHAPE
    assert g(FAKE, FAKE, FAKE, FAKE, 4, 96, 8, FAKE, 7, None) == SHAPE
    assert g(FAKE + 1, FAKE, FAKE, FAKE, 4, 96, 8, FAKE, 8, None) == ALIGN
    assert g(FAKE, FAKE, FAKE, FAKE, 0, 96, 8, FAKE, 8, None) == OK
    h = L.pme_expanded_linear_mxfp4
    need = pme.workspace_bytes(4, 64, 96, 8)
    assert h(FAKE, 1, 4, 64, 64, 96, FAKE, FAKE, 8, FAKE, 8, FAKE, need - 1, None) == WORKSPACE
    assert h(FAKE, 1, 4, 64, 64, 96, FAKE, None, 8, FAKE, 8, FAKE, need, None) == NULL
    assert h(FAKE, 1, 4, 64, 64, 80, FAKE, FAKE, 8, FAKE, 8, FAKE, need, None) == SHAPE
    w = L.pme_expand_quantize_weights
    assert w(None, 0, 8, 64, 64, 80, FAKE, FAKE, None) == NULL
    assert w(FAKE, 0, 8, 64, 60, 80, FAKE, FAKE, None) == SHAPE
    r = L.pme_weight_rowsum
    assert r(None, 8, 80, FAKE, None) == NULL
    assert r(FAKE, 8, 81, FAKE, None) == SHAPE
    a = L.pme_w4a4_gemm_asym
    assert a(FAKE, FAKE, None, FAKE, FAKE, FAKE, 4, 80, 8, FAKE, 8, None) == NULL
    assert a(FAKE, FAKE, FAKE, FAKE, FAKE, None, 4, 80, 8, FAKE, 8, None) == NULL
    q = L.pme_hadamard_expand_quant_asym
    assert q(FAKE, 1, 4, 64, 64, 80, FAKE, FAKE, None, None) == NULL


def test_expanded_linear_asym_argument_errors():
    f = pme.lib().pme_expanded_linear_asym
    need = pme.workspace_bytes(4, 64, 80, 8)

    def call(x=FAKE, xt=1, T=4, d=64, ldx=64, d_e=80, qw=FAKE, sw=FAKE, wsum=FAKE, N=8, y=FAKE, ldy=8, ws=FAKE, wsb=need):
        return f(x, xt, T, d, ldx, d_e, qw, sw, wsum, N, y, ldy, ws, wsb, None)

    assert call(wsum=None) == NULL
    assert call(wsum=FAKE + 2) == ALIGN
    assert call(wsb=need - 1) == WORKSPACE
    assert call(ws=FAKE + 128) == ALIGN
    assert call(d_e=11264) == ORDER
    assert call(ldy=7) == SHAPE
    assert call(T=0) == OK


def test_probe_copy_errors():
    f = pme.lib().pme_probe_copy
    assert f(None, FAKE, 16, None) == NULL
    assert f(FAKE, FAKE, 24, None) == SHAPE
    assert f(FAKE + 8, FAKE, 32, None) == ALIGN
    assert f(FAKE, FAKE, 0, None) == OK


def test_probe_mfma_errors():
    f = pme.lib().pme_probe_mfma
    n = 512 * 256
    assert f(0, None, n, 10, None, None) == NULL
    assert f(4, FAKE, n, 10, None, None) == DTYPE
    assert f(-1, FAKE, n, 10, None, None) == DTYPE
    assert f(0, FAKE, n - 1, 10, None, None) == SHAPE
    assert f(1, FAKE, n, -1, None, None) == SHAPE
    assert f(0, FAKE + 2, n, 10, None, None) == ALIGN


def test_binding_has_no_fallback():
    # The binding refuses host tensors instead of computing anything itself.
    import torch
    x = torch.zeros(2, 64)
    with pytest.raises(ValueError):
        pme.hadamard_expand_quant(x, 80)


def test_gemm_plan_names_the_kernel_without_launching():
    """pme_gemm_plan is a dry run of the dispatch: it needs no GPU and names the instantiation a profiler would print."""
    assert pme.gemm_plan(4096, 15360, 4096) == "k_gemm_mfma<256, 256, 2, 2, 128, 2, 0, 1, false>"
    assert pme.gemm_plan(4096, 15360, 4096, variant=1) == "k_gemm_mfma<256, 256, 2, 2, 128, 2, 1, 1, false>"
    assert pme.gemm_plan(2048, 2176, 3072) == "k_gemm_mfma<128, 192, 2, 2, 64, 3, 0, 1, true>"
    assert pme.gemm_plan(2048, 8704, 2048) == "k_gemm_mfma<128, 128, 2, 2, 128, 3, 0, 1, true>"
    assert pme.gemm_plan(8, 8448, 2048) == "k_gemm_decode"
    assert pme.gemm_plan(4096, 15360, 4096, variant=2).startswith("k_mxgemm_mfma<256, 256, ")
    assert pme.gemm_plan(8, 8448, 2048, variant=2) == "k_mxgemm_decode"
    assert pme.gemm_plan(16, 80, 64) == "k_gemm_generic"                 # d_e not a multiple of 128
    # the x256 accumulator of the matrix-core kernels: 256 * 64 * d_e < 2^31 holds below d_e = 2^17 only
    assert pme.gemm_plan(300, (1 << 17) - 128, 256).startswith("k_gemm_mfma<")
    assert pme.gemm_plan(300, 1 << 17, 256) == "k_gemm_generic"
    assert pme.gemm_plan(8, (1 << 17) - 128, 256) == "k_gemm_decode"
    assert pme.gemm_plan(8, 1 << 17, 256) == "k_gemm_generic"
    f = pme.lib().pme_gemm_plan
    buf = C.create_string_buffer(64)
    assert f(0, 8, 256, 8, None, 64) == NULL
    assert f(3, 8, 256, 8, buf, 64) == DTYPE
    assert f(0, 0, 256, 8, buf, 64) == SHAPE
    assert f(0, 8, 255, 8, buf, 64) == SHAPE
    assert f(2, 8, 80, 8, buf, 64) == SHAPE                              # MXFP4 needs whole blocks of 32
    try:
        pme.set_path(pme.PATH_MFMA)
        assert f(0, 16, 80, 64, buf, 64) == PATH                         # forced matrix-core path, shape it does not take
    finally:
        pme.set_path(pme.PATH_AUTO)


# (T, d_e, N) and the int4 kernel that measured faster, in us from the caches / from memory
PLANS = [
    # few tokens by up to 4096 channels: the streaming kernel up to 4 below d_e = 15000, up to 8 below 11000 and up to 12 below 10000, where
    # the K-split tiles lose with weights from memory, and wherever K is no whole number of 256 codes or shorter than 8192 (streaming
    # and 8 or 16 x 32: 1 x 12288 x 2048 7.0 / 7.1 and 6.5 / 7.8, 2 x 14848 x 2048 8.2 / 8.2 and 7.1 / 8.7, 10 x 8448 x 2048 6.4 / 6.5 and
    # 5.2 / 7.1, 12 x 8704 x 4096 7.4 / 7.5 and 6.2 / 7.9, 12 x 8704 x 2048 6.9 / 6.9 and 5.2 / 7.4)
    (1, 8448, 2048, "k_gemm_decode"), (8, 8448, 2048, "k_gemm_decode"), (4, 8704, 4096, "k_gemm_decode"),
    (8, 10240, 2048, "k_gemm_decode"), (9, 7680, 2048, "k_gemm_decode"), (20, 4352, 2048, "k_gemm_decode"),
    (16, 1024, 3072, "k_gemm_decode"), (58, 1024, 5056, "k_gemm_decode"), (1, 12288, 2048, "k_gemm_decode"), (2, 12288, 2112, "k_gemm_decode"), (2, 14848, 2048, "k_gemm_decode"),
    (4, 14848, 2048, "k_gemm_decode"), (9, 8448, 2048, "k_gemm_decode"), (10, 8448, 2048, "k_gemm_decode"), (12, 8704, 4096, "k_gemm_decode"), (12, 9984, 2048, "k_gemm_decode"),
    # beyond these lines 8 x 32 and 16 x 32, K split (8 x 11008 x 2048 7.5 / 7.6 and 6.1 / 7.8, 1 x 15360 x 4096 9.4 / 9.5 and 7.9 / 9.9,
    # 1 x 22016 x 3072 12.2 / 12.8 and 9.8 / 13.0, 1 x 32768 x 2048 14.3 / 14.4 and 11.8 / 14.4, 8 x 15104 x 2048 9.4 / 9.5 and 7.2 / 9.4,
    # 5 x 15360 x 1024 9.0 / 9.1 and 6.6 / 9.1, 10 x 15104 x 2048 9.8 / 9.8 and 7.3 / 9.9, 11 x 10240 x 2048 8.1 / 8.2 and 5.8 / 8.4,
    # 16 x 8448 x 2048 7.1 / 7.3 and 5.2 / 7.4)
    (8, 11008, 2048, "k_gemm_kslice<8, 32, 8, 3, 0>"), (5, 11008, 2048, "k_gemm_kslice<8, 32, 8, 3, 0>"), (1, 15104, 2048, "k_gemm_kslice<8, 32, 8, 3, 0>"), (1, 15360, 4096, "k_gemm_kslice<8, 32, 8, 3, 0>"), (1, 22016, 3072, "k_gemm_kslice<8, 32, 8, 3, 0>"),
    (1, 32768, 2048, "k_gemm_kslice<8, 32, 8, 3, 0>"), (2, 15104, 2048, "k_gemm_kslice<8, 32, 8, 3, 0>"), (8, 15104, 2048, "k_gemm_kslice<8, 32, 8, 3, 0>"), (3, 15360, 1356, "k_gemm_kslice<8, 32, 8, 3, 0>"), (5, 15360, 1024, "k_gemm_kslice<8, 32, 8, 3, 0>"), (2, 15360, 3072, "k_gemm_kslice<8, 32, 8, 3, 0>"),
    (10, 15104, 2048, "k_gemm_kslice<16, 32, 8, 3, 0>"), (9, 10240, 2048, "k_gemm_kslice<16, 32, 8, 3, 0>"), (11, 10240, 2048, "k_gemm_kslice<16, 32, 8, 3, 0>"), (13, 8448, 2048, "k_gemm_kslice<16, 32, 8, 3, 0>"), (16, 8448, 2048, "k_gemm_kslice<16, 32, 8, 3, 0>"),
    (12, 8704, 4160, "k_gemm_kslice<32, 32, 8, 2, 0>"),
    # from a second round of 4096 channels, or with more tokens, 32 x 32 and larger (1 x 12288 x 5120: 8.3 / 10.0, streaming 12.8 / 12.8;
    # 12 x 8704 x 4160: 6.4 / 7.9, 11.7 / 11.9; 32 x 15360 x 4096: 9.0 / 13.4, 18.8 / 19.2)
    (1, 12288, 5120, "k_gemm_kslice<32, 32, 8, 2, 0>"), (4, 8704, 6144, "k_gemm_kslice<32, 32, 8, 2, 0>"),
    (32, 15360, 4096, "k_gemm_kslice<32, 32, 8, 2, 0>"), (48, 8704, 6144, "k_gemm_kslice<64, 32, 8, 3, 0>"),
    # small outputs: each K-split tile, and the 64 x 64 tile where K is short or the tiles many
    (333, 9728, 2048, "k_gemm_kslice<64, 64, 8, 2, 0>"), (517, 8704, 2048, "k_gemm_kslice<96, 64, 4, 3, 0>"),
    (900, 15360, 2048, "k_gemm_kslice<128, 64, 4, 3, 0>"), (768, 15360, 4096, "k_gemm_kslice<128, 128, 4, 2, 0>"),
    (64, 1024, 14336, "k_gemm_mfma<64, 64, "), (768, 1024, 1024, "k_gemm_mfma<64, 64, "), (700, 2176, 3072, "k_gemm_mfma<64, 64, "),
    (32, 15360, 28672, "k_gemm_mfma<64, 64, "),
    # one round of 128 x 128: not split while K is short, nor for a single row of tiles (128 x 8704 x 28672: 13 / 16 % slower split)
    (700, 4352, 4096, "k_gemm_mfma<128, 128, "), (128, 8704, 28672, "k_gemm_mfma<128, 128, "),
]


@pytest.mark.parametrize("T,d_e,N,kernel", PLANS)
def test_gemm_plan_takes_the_faster_kernel(T, d_e, N, kernel):
    assert pme.gemm_plan(T, d_e, N).startswith(kernel)
    assert pme.gemm_plan(T, d_e, N, variant=1).startswith(kernel.replace(", 0>", ", 1>"))


# shapes that a tile does not take: half a K step of 256 codes, less than a step for each wave, an id that is none
@pytest.mark.parametrize("tile,T,d_e", [(116, 16, 1152), (116, 8, 1024), (117, 16, 1152), (118, 16, 1152), (118, 300, 1152), (101, 16, 1152),
                                        (115, 16, 2048), (122, 16, 2048), (35, 8, 2176), (36, 16, 1024), (37, 16, 2048)])
def test_a_forced_tile_that_refuses_is_not_replaced(tile, T, d_e):
    variant = 2 if tile >= 100 else 0
    f, buf = pme.lib().pme_gemm_plan, C.create_string_buffer(64)
    try:
        pme.set_gemm_tile(tile)
        assert pme.gemm_plan(T, d_e, 300, variant=variant) == ("k_mxgemm_generic" if variant else "k_gemm_generic")
        pme.set_path(pme.PATH_MFMA)
        assert f(variant, T, d_e, 300, buf, 64) == PATH
    finally:
        pme.set_gemm_tile(0)
        pme.set_path(pme.PATH_AUTO)


def test_pack_int4_argument_errors():
    f = pme.lib().pme_pack_int4
    assert f(None, 4, 8, FAKE, None) == NULL
    assert f(FAKE, 4, 8, None, None) == NULL
    assert f(FAKE, 4, 7, FAKE, None) == SHAPE
    assert f(FAKE, -1, 8, FAKE, None) == SHAPE
    assert f(None, 0, 8, None, None) == OK


def test_static_scratch_layer_argument_errors():
    """pme_expanded_linear_static validates like pme_expanded_linear and refuses, before any HIP call, a shape whose
    quantized activations do not fit its static scratch."""
    f = pme.lib().pme_expanded_linear_static

    def call(x=FAKE, xt=1, T=8, d=8192, ldx=8192, d_e=8448, qw=FAKE, sw=FAKE, N=2048, y=FAKE, ldy=2048):
        return f(x, xt, T, d, ldx, d_e, qw, sw, N, y, ldy, None)

    assert call(x=None) == NULL
    assert call(qw=None) == NULL
    assert call(y=None) == NULL
    assert call(ldy=2047) == SHAPE
    assert call(d_e=8450) == ORDER
    assert call(y=FAKE + 1) == ALIGN
    assert call(T=0, x=None) == OK
    # 4096 tokens of 15360 expanded features need 31.5 MB of codes: beyond the 16 MiB scratch
    assert pme.workspace_bytes(4096, 14336, 15360, 4096) > pme.STATIC_SCRATCH_BYTES
    assert call(T=4096, d=14336, ldx=14336, d_e=15360, N=4096, ldy=4096) == WORKSPACE
    assert pme.workspace_bytes(2048, 14336, 15360, 4096) <= pme.STATIC_SCRATCH_BYTES


def _kernel_metadata():
    """The kernels of the built library and their resources, from the metadata notes of its gfx950 code objects."""
    import struct
    msgpack = pytest.importorskip("msgpack")
    data = open(os.path.join(ROOT, "paper_2503_17513_amd", "libpme.so"), "rb").read()
    kernels, pos = [], 0
    while (pos := data.find(b"\x7fELF", pos + 1)) > 0:
        if struct.unpack_from("<H", data, pos + 18)[0] != 224:                     # EM_AMDGPU
            continue
        table, (entry, count) = struct.unpack_from("<Q", data, pos + 40)[0], struct.unpack_from("<HH", data, pos + 58)
        for header in range(pos + table, pos + table + entry * count, entry):
            if struct.unpack_from("<I", data, header + 4)[0] != 7:                  # SHT_NOTE
                continue
            at, size = struct.unpack_from("<QQ", data, header + 24)
            note, end = pos + at, pos + at + size
            while note < end:
                name, desc, kind = struct.unpack_from("<III", data, note)
                body = note + 12 + (name + 3) // 4 * 4
                if kind == 32:                                                     # NT_AMDGPU_METADATA
                    kernels += msgpack.unpackb(data[body:body + desc])["amdhsa.kernels"]
                note = body + (desc + 3) // 4 * 4
    return kernels


def test_rotation_and_k_split_kernels_use_no_scratch():
    # every instantiation holds its accumulators and what it fetches ahead in registers; spilled ones have cost up to 1.7 x
    kernels = [k for k in _kernel_metadata() if "k_rotate_mfma" in k[".name"] or "k_gemm_kslice" in k[".name"]]
    assert len(kernels) > 100
    assert not [k[".name"] for k in kernels if k[".private_segment_fixed_size"] or k[".vgpr_spill_count"]]


def test_one_token_and_k_split_decode_kernels_use_no_scratch():
    # the token's values, the fetched weights and the accumulators stay in registers
    kernels = []
    # the one-token kernel at two widths and two quantizers; every tile of either K-split kernel
    for args, least in (("9TokenArgs", 4), ("10KSliceArgs", 8 * 3), ("11MxSliceArgs", 6)):
        found = [k for k in _kernel_metadata() if args in k[".symbol"]]
        assert len(found) >= least, args
        kernels += found
    assert not [k[".name"] for k in kernels if k[".private_segment_fixed_size"] or k[".vgpr_spill_count"]]


# (T, d_e, N, variant) on either side of the lines of the choice that the fitted times draw
FITTED_PLANS = [
    # two rounds of 128 x 192: with asymmetric codes the loader tile (141 us shared, 129 so)
    (3000, 8960, 3300, 1, "k_gemm_mfma<128, 192, 2, 2, 128, 3, 1, 1, true>"), (3000, 8960, 3300, 0, "k_gemm_mfma<128, 192, 2, 2, 64, 3, 0, 1, false>"),
    # MXFP4 by 64 x 64 tiles of a shared K loop before: 24.6 us and 18.7 so, 35.1 and 14.1
    (333, 9728, 2048, 2, "k_mxgemm_kslice<64, 64, 4, 128, 2>"), (78, 15360, 704, 2, "k_mxgemm_kslice<16, 32, 4, 128, 3>"),
    (33, 2176, 704, 2, "k_mxgemm_kslice<32, 32, 4, 64, 4>"), (4096, 15360, 4096, 2, "k_mxgemm_mfma<256, 256, 2, 2, "),
    (2048, 8704, 2048, 2, "k_mxgemm_mfma<128, 128, "), (300, 512, 256, 2, "k_mxgemm_mfma<64, 64, 2, 2, 64, 3, true>"),
    (12, 8704, 2048, 2, "k_mxgemm_kslice<16, 32, 4, 128, 3>"), (130, 8704, 300, 2, "k_mxgemm_kslice<16, 32, 4, 128, 3>"),
    # few tokens, MXFP4: streaming where the K-split tiles lose with weights from memory (us from the caches / from memory, streaming and
    # K-split: 8 x 8704 x 1024 7.3 / 7.3 and 5.3 / 8.6, 8 x 11008 x 1024 8.5 / 8.6 and 5.6 / 9.9, 1 x 22016 x 2048 13.0 / 13.1 and 9.6 / 14.7,
    # 17 x 2176 x 1024 3.9 / 3.9 and 3.9 / 5.2, 32 x 4480 x 2048 7.1 / 7.2 and 4.5 / 8.3, 1 x 2176 x 10496 5.0 / 5.1 and 5.7 / 7.5), and the
    # other side of each line (2 x 12288 x 2048 9.5 / 9.5 and 6.7 / 9.6, 9 x 10240 x 2048 10.1 / 10.2 and 6.5 / 9.8, 8 x 4480 x 4160 7.0 / 7.1
    # and 4.7 / 6.4, 16 x 2560 x 6144 6.2 / 6.4 and 4.1 / 5.4, 1 x 8448 x 4160 9.6 / 9.8 and 5.9 / 7.8)
    (8, 8448, 2048, 2, "k_mxgemm_decode"), (8, 8704, 1024, 2, "k_mxgemm_decode"), (10, 8704, 2048, 2, "k_mxgemm_decode"),
    (11, 8704, 2048, 2, "k_mxgemm_kslice<16, 32, "), (12, 5120, 1024, 2, "k_mxgemm_decode"), (11, 6144, 1024, 2, "k_mxgemm_kslice<16, 32, "),
    (16, 4608, 2048, 2, "k_mxgemm_decode"), (17, 4608, 2048, 2, "k_mxgemm_kslice<32, 32, 4, 128, "), (8, 10240, 2048, 2, "k_mxgemm_decode"),
    (9, 10240, 2048, 2, "k_mxgemm_kslice<16, 32, "), (8, 11008, 1024, 2, "k_mxgemm_decode"), (2, 12288, 2048, 2, "k_mxgemm_kslice<8, 32, "),
    (1, 12288, 2048, 2, "k_mxgemm_decode"), (1, 22016, 4096, 2, "k_mxgemm_decode"), (1, 8448, 4160, 2, "k_mxgemm_kslice<16, 32, "),
    (17, 2176, 1024, 2, "k_mxgemm_decode"), (32, 4480, 4096, 2, "k_mxgemm_decode"), (32, 4480, 4160, 2, "k_mxgemm_kslice<32, 32, 4, 64, "),
    (8, 4480, 4160, 2, "k_mxgemm_kslice<32, 32, 4, 64, "), (8, 2176, 4160, 2, "k_mxgemm_decode"), (1, 2176, 10496, 2, "k_mxgemm_decode"),
    (16, 2304, 6144, 2, "k_mxgemm_decode"), (16, 2560, 6144, 2, "k_mxgemm_kslice<16, 32, "), (17, 2176, 6144, 2, "k_mxgemm_kslice<32, 32, 4, 64, "),
]


@pytest.mark.parametrize("T,d_e,N,variant,kernel", FITTED_PLANS)
def test_gemm_plan_by_fitted_times(T, d_e, N, variant, kernel):
    assert pme.gemm_plan(T, d_e, N, variant=variant).startswith(kernel)
