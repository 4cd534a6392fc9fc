"""GPU parity of the MXFP4 path (paper Section 4, second quantization setting) against the CPU oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2503_17513_amd as pme
from parity_util import check_mx_gemm, check_mx_quant, to_device
from workloads import custom_spec, make_workload

pytestmark = pytest.mark.gpu
GENERIC, MFMA = pme.PATH_GENERIC, pme.PATH_MFMA


@pytest.fixture(autouse=True)
def _reset():
    yield
    pme.set_path(pme.PATH_AUTO)
    pme.set_gemm_tile(0)


def _acts(T, d, d_e, in_dtype="bf16", seed=0):
    spec = custom_spec(T, d, d_e, 8, in_dtype=in_dtype, act_dist="student_t3", outlier_frac=0.01, outlier_gain=50.0, seed=seed)
    return make_workload(spec, weights=False).x


QUANT_CASES = [
    ("b12_k3_generic", 9, 80, 96, "f32", (GENERIC,)),
    ("b68_k5", 21, 2048, 2176, "bf16", (GENERIC, MFMA)),
    ("b132_k6", 8, 8192, 8448, "bf16", (GENERIC, MFMA)),
    ("b68_k7", 9, 8192, 8704, "bf16", (GENERIC, MFMA)),
    ("b60_k8", 5, 14336, 15360, "bf16", (GENERIC, MFMA)),
    ("b20_k9", 3, 8192, 10240, "bf16", (GENERIC, MFMA)),
    ("f32_b68_k5", 6, 2048, 2176, "f32", (GENERIC, MFMA)),
    ("many_tokens_k7", 530, 8192, 8704, "bf16", (MFMA,)),
    ("b68_k5_token_per_wave", 1029, 2048, 2176, "bf16", (MFMA,)),
    ("b12_k10_folded", 5, 8192, 12288, "bf16", (GENERIC, MFMA)),
    ("b312_k6", 5, 14336, 19968, "bf16", (GENERIC, MFMA)),
]


@pytest.mark.parametrize("name,T,d,d_e,in_dtype,paths", QUANT_CASES, ids=[c[0] for c in QUANT_CASES])
def test_rotate_and_quantize_mxfp4(name, T, d, d_e, in_dtype, paths):
    x = _acts(T, d, d_e, in_dtype, seed=len(name))
    if T > 2:
        x[1] = 0.0
        x[2] = 0.0
        x[2, d // 3] = 1.0
    xd = to_device(x, in_dtype)
    ref = oracle.rotate_structured(x, d_e)
    for path in paths:
        pme.set_path(path)
        qx, ex = pme.hadamard_expand_quant_mxfp4(xd, d_e)
        torch.cuda.synchronize()
        check_mx_quant(qx, ex, ref)
        if T > 2:
            assert int(ex[1].max()) == 0 and int(qx[1].max()) == 0     # all-zero token: smallest scale, zero codes


def test_mxfp4_rejects_d_e_not_multiple_of_32():
    x = torch.zeros((4, 64), dtype=torch.float32, device="cuda")
    with pytest.raises(pme.PmeError) as e:
        pme.hadamard_expand_quant_mxfp4(x, 80)
    assert e.value.status == 2


GEMM_CASES = [("small_ragged", 50, 70, 96, (GENERIC,)), ("one_k_step", 40, 72, 128, (GENERIC, MFMA)),
              ("ragged_tiles", 300, 200, 2176, (GENERIC, MFMA)), ("wide_rows", 260, 520, 1280, (GENERIC, MFMA)),
              ("c2_shape_rows", 2048, 384, 2176, (MFMA,)), ("big_tile", 1024, 4096, 512, (MFMA,)),
              # at most 32 tokens: the weight-streaming kernel, 1 or 2 groups of 16 tokens; beyond: tiles
              ("decode_shape", 8, 2048, 8448, (GENERIC, MFMA)), ("decode_one_token_one_chunk", 1, 24, 128, (GENERIC, MFMA)),
              ("decode_16_ragged_n", 16, 100, 384, (GENERIC, MFMA)), ("decode_33_odd_chunks", 33, 40, 640, (GENERIC, MFMA)),
              ("decode_48", 48, 72, 1280, (MFMA,)), ("decode_64", 64, 130, 2176, (GENERIC, MFMA)),
              ("sixty_five_tokens_tiled", 65, 72, 256, (MFMA,))]


@pytest.mark.parametrize("name,T,N,d_e,paths", GEMM_CASES, ids=[c[0] for c in GEMM_CASES])
def test_mxfp4_gemm(name, T, N, d_e, paths):
    rng = np.random.default_rng(T + N)
    qx = rng.integers(0, 16, size=(T, d_e), dtype=np.uint8)
    qw = rng.integers(0, 16, size=(N, d_e), dtype=np.uint8)
    ex = rng.integers(118, 132, size=(T, d_e // 32), dtype=np.uint8)
    ew = rng.integers(118, 130, size=(N, d_e // 32), dtype=np.uint8)
    args = [torch.from_numpy(a).cuda() for a in (oracle.pack_fp4(qx), ex, oracle.pack_fp4(qw), ew)]
    for path in paths:
        pme.set_path(path)
        y = pme.mxfp4_gemm(*args).to(torch.float32).cpu().numpy()
        check_mx_gemm(y, qx, ex, qw, ew)


@pytest.mark.parametrize("T", (17, 32))
@pytest.mark.parametrize("d_e", (256, 384, 512, 640, 896, 1152))
def test_mxfp4_gemm_two_groups_of_tokens_on_few_chunks(T, d_e):
    """17 .. 32 tokens where some of a workgroup's waves have one 128-code chunk and others none or two: a wave without a
    second chunk must not run its matrix instruction (outputs were NaN now and then, from registers never written)."""
    rng = np.random.default_rng(d_e + T)
    N = 592
    qx = rng.integers(0, 16, size=(T, d_e), dtype=np.uint8)
    qw = rng.integers(0, 16, size=(N, d_e), dtype=np.uint8)
    ex = rng.integers(118, 132, size=(T, d_e // 32), dtype=np.uint8)
    ew = rng.integers(118, 130, size=(N, d_e // 32), dtype=np.uint8)
    args = [torch.from_numpy(a).cuda() for a in (oracle.pack_fp4(qx), ex, oracle.pack_fp4(qw), ew)]
    pme.set_path(MFMA)
    x = torch.randn((64, 512), device="cuda")
    for _ in range(5):
        pme.hadamard_expand_quant(x, 512)          # leaves values of another kernel in the registers
        y = pme.mxfp4_gemm(*args).to(torch.float32).cpu().numpy()
        check_mx_gemm(y, qx, ex, qw, ew)


@pytest.mark.parametrize("tile", range(1, 15))
def test_mxfp4_gemm_every_tile(tile):
    rng = np.random.default_rng(tile)
    T, N, d_e = 300, 520, 1280
    qx = rng.integers(0, 16, size=(T, d_e), dtype=np.uint8)
    qw = rng.integers(0, 16, size=(N, d_e), dtype=np.uint8)
    ex = rng.integers(120, 130, size=(T, d_e // 32), dtype=np.uint8)
    ew = rng.integers(120, 130, size=(N, d_e // 32), dtype=np.uint8)
    args = [torch.from_numpy(a).cuda() for a in (oracle.pack_fp4(qx), ex, oracle.pack_fp4(qw), ew)]
    pme.set_path(MFMA)
    pme.set_gemm_tile(100 + tile)
    y = pme.mxfp4_gemm(*args).to(torch.float32).cpu().numpy()
    check_mx_gemm(y, qx, ex, qw, ew)


# Outputs that the automatic choice gives to the tiles of 128 x 64, 192 x 128 and 256 x 192: several tiles in both directions, the last of
# either ragged.  Rows are sampled so that each of a tile's waves and every token fragment of a wave has some.
@pytest.mark.parametrize("T,d_e,N,tile", [(267, 12288, 4352, "128, 64"), (2895, 15360, 5457, "192, 128"), (3606, 9728, 3136, "256, 192")])
def test_mxfp4_gemm_automatic_choice(T, d_e, N, tile):
    g = torch.Generator(device="cuda").manual_seed(T)
    qx, qw = (torch.randint(0, 256, (n, d_e // 2), dtype=torch.uint8, device="cuda", generator=g) for n in (T, N))
    ex, ew = (torch.randint(118, 130, (n, d_e // 32), dtype=torch.uint8, device="cuda", generator=g) for n in (T, N))
    assert pme.gemm_plan(T, d_e, N, variant=2).startswith(f"k_mxgemm_mfma<{tile}, ")
    pme.set_path(MFMA)
    y = pme.mxfp4_gemm(qx, ex, qw, ew)
    rows = torch.unique(torch.cat([torch.arange(7, T, max(29, T // 24 // 32 * 32 + 29)), torch.tensor([0, T - 1])])).cuda()
    check_mx_gemm(y[rows].float().cpu().numpy(), oracle.unpack_fp4(qx[rows].cpu().numpy()), ex[rows].cpu().numpy(),
                  oracle.unpack_fp4(qw.cpu().numpy()), ew.cpu().numpy())


# Scale bytes arrive in groups of 512 codes: less than one group, whole ones, a remainder of 128 and of 256 codes, and more
# groups than the two of the ring; the last rows' remainder lies at the end of the scale tensors.
@pytest.mark.parametrize("d_e", (256, 512, 1152, 1792, 2560))
@pytest.mark.parametrize("tile", range(1, 15))
def test_mxfp4_gemm_scale_groups(tile, d_e):
    if d_e % 256 and tile in (1, 3, 6, 8, 9, 12, 13, 14):      # 128-byte rows
        pytest.skip("the tile takes whole steps of 256 codes")
    rng = np.random.default_rng(tile + d_e)
    T, N = 65, 72
    qx = rng.integers(0, 16, size=(T, d_e), dtype=np.uint8)
    qw = rng.integers(0, 16, size=(N, d_e), dtype=np.uint8)
    ex = rng.integers(112, 136, size=(T, d_e // 32), dtype=np.uint8)
    ew = rng.integers(112, 136, size=(N, d_e // 32), dtype=np.uint8)
    args = [torch.from_numpy(a).cuda() for a in (oracle.pack_fp4(qx), ex, oracle.pack_fp4(qw), ew)]
    pme.set_path(MFMA)
    pme.set_gemm_tile(100 + tile)
    y = pme.mxfp4_gemm(*args).to(torch.float32).cpu().numpy()
    check_mx_gemm(y, qx, ex, qw, ew)


# The tiles whose waves split K (16 .. 21: tokens, channels, waves, bytes a row): one token, the tile's edges and beyond, ragged
# channels (16-byte and single stores); K of one step a wave, shares that differ by one step, a last group of scales cut short.
KSPLIT = {16: (8, 32, 8, 128), 17: (16, 32, 4, 128), 18: (32, 32, 4, 128), 19: (64, 32, 4, 128), 20: (64, 64, 4, 128), 21: (32, 32, 4, 64)}


@pytest.mark.parametrize("tile,d_e", [(t, 2 * k[3] * s) for t, k in KSPLIT.items() for s in (k[2], k[2] + 1, 3 * k[2] - 1, 5 * k[2] + 2)])
def test_mxfp4_gemm_k_split_tiles(tile, d_e):
    bm, bn = KSPLIT[tile][:2]
    rng = np.random.default_rng(tile + d_e)
    pme.set_path(MFMA)
    pme.set_gemm_tile(100 + tile)
    for T, N in ((1, 8), (bm, bn), (bm + 1, bn + 8), (2 * bm - 1, 2 * bn + 3)):
        assert pme.gemm_plan(T, d_e, N, variant=2).startswith("k_mxgemm_kslice<%d, %d, %d, %d, " % KSPLIT[tile])
        qx = rng.integers(0, 16, size=(T, d_e), dtype=np.uint8)
        qw = rng.integers(0, 16, size=(N, d_e), dtype=np.uint8)
        ex = rng.integers(112, 136, size=(T, d_e // 32), dtype=np.uint8)
        ew = rng.integers(112, 136, size=(N, d_e // 32), dtype=np.uint8)
        args = [torch.from_numpy(a).cuda() for a in (oracle.pack_fp4(qx), ex, oracle.pack_fp4(qw), ew)]
        guard = torch.full((T + 1, N + 5), 7.0, dtype=torch.bfloat16, device="cuda")
        pme.mxfp4_gemm(*args, y=guard[:T, :N])
        y = guard.to(torch.float32).cpu().numpy()
        check_mx_gemm(y[:T, :N], qx, ex, qw, ew)
        assert (y[T:] == 7.0).all() and (y[:, N:] == 7.0).all()


@pytest.mark.parametrize("T", (5, 20))
def test_mxfp4_gemm_few_tokens_with_unaligned_scales(T):
    """Scale rows that are not 4-byte aligned: the streaming kernel takes them, whatever kernel is estimated fastest."""
    rng = np.random.default_rng(T)
    N, d_e = 640, 8448
    qx = rng.integers(0, 16, size=(T, d_e), dtype=np.uint8)
    qw = rng.integers(0, 16, size=(N, d_e), dtype=np.uint8)
    ex = rng.integers(112, 136, size=(T, d_e // 32), dtype=np.uint8)
    ew = rng.integers(112, 136, size=(N, d_e // 32), dtype=np.uint8)

    def odd(a):
        buf = torch.empty(a.size + 1, dtype=torch.uint8, device="cuda")
        buf[1:] = torch.from_numpy(a).cuda().flatten()
        return buf[1:].view(a.shape)

    pme.set_path(MFMA)
    y = pme.mxfp4_gemm(torch.from_numpy(oracle.pack_fp4(qx)).cuda(), odd(ex), torch.from_numpy(oracle.pack_fp4(qw)).cuda(), odd(ew))
    check_mx_gemm(y.to(torch.float32).cpu().numpy(), qx, ex, qw, ew)


@pytest.mark.parametrize("shape", ((40, 2048, 2176, 200), (130, 8192, 8704, 300)))
def test_mxfp4_layer_end_to_end(shape):
    T, d, d_e, N = shape
    rng = np.random.default_rng(5)
    x = _acts(T, d, d_e, "bf16", seed=2)
    W = (rng.standard_normal((d, N)) / np.sqrt(d)).astype(np.float32)
    xd = to_device(x, "bf16")
    wt = torch.from_numpy(np.ascontiguousarray(W.T)).cuda()
    qw, ew = pme.hadamard_expand_quant_mxfp4(wt, d_e)          # offline weight side: rows of W^T
    check_mx_quant(qw, ew, oracle.expand_weight(W, d_e).T)
    y = pme.expanded_linear_mxfp4(xd, d_e, qw, ew).to(torch.float32).cpu().numpy()
    qx, ex = pme.hadamard_expand_quant_mxfp4(xd, d_e)
    check_mx_quant(qx, ex, oracle.rotate_structured(x, d_e))
    check_mx_gemm(y, oracle.unpack_fp4(qx.cpu().numpy()), ex.cpu().numpy(), oracle.unpack_fp4(qw.cpu().numpy()), ew.cpu().numpy())
    ref = x.astype(np.float64) @ W.astype(np.float64)
    assert np.linalg.norm(y - ref) / np.linalg.norm(ref) < 0.25
