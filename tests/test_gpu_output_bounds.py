"""Output bounds: every GEMM kernel of the library, on shapes with partial tiles, writes C[b][i][j] for i < M, j < N and
nothing else, and the attention kernels write their output and nothing else. C is a window of a larger buffer filled with a bit pattern (a NaN payload no kernel produces): leading
dimension ldc > N, guard words in front of the first row and behind the last one. After the call the window must match
the oracle and every other word must still hold the pattern, bit for bit."""
import numpy as np
import pytest
import torch

from oracle import layer_ref, ref
from paper_2411_09909_amd import binding, synth
from tests import gpu_util as G

pytestmark = pytest.mark.gpu

TOL = 1e-3
CANARY = 0x7FC0DEAD  # a quiet NaN with a payload, as int32
GUARD = 4096  # words in front of and behind the matrix


def canary_window(batch, M, N, pad, dtype=torch.float32):
    """A [batch, M, N] window with leading dimension N + pad inside a pattern-filled buffer. Returns (buffer as
    integers, window, mask of the words the call may write)."""
    ld = N + pad
    words = torch.int32 if dtype == torch.float32 else torch.int16
    pattern = CANARY if dtype == torch.float32 else 0x7FC5
    buf = torch.full((GUARD + batch * M * ld + GUARD,), pattern, dtype=words, device="cuda")
    body = buf[GUARD:GUARD + batch * M * ld].view(batch, M, ld)
    window = body.view(dtype)[:, :, :N]
    allowed = torch.zeros_like(buf, dtype=torch.bool)
    allowed[GUARD:GUARD + batch * M * ld].view(batch, M, ld)[:, :, :N] = True
    return buf, window, allowed, pattern


def assert_padding_untouched(buf, allowed, pattern, what):
    touched = (buf != pattern) & ~allowed
    n = int(touched.sum())
    assert n == 0, "%s: %d words outside C were written (first at flat index %d)" % (
        what, n, int(torch.nonzero(touched)[0]))


def operands(batch, M, N, K, scale, asym, gs=32):
    a = synth.activations(batch * M, K, seed=M + K, n_outlier=2, outlier_gain=60.0)
    b = synth.weights(batch * N, K, seed=N)
    ac, as_ = ref.quantize(a, gs, scale, asym)
    bc, bs = ref.quantize(b, gs, scale, asym)
    shp = lambda t, r: t.reshape((batch, r) + t.shape[1:])  # noqa: E731
    return shp(ac, M), shp(as_, M), shp(bc, N), shp(bs, N)


# (label, scale, asymmetric, group size, per-call options, shapes) — one entry per kernel and store path
KERNELS = [
    ("panel 256x256", ref.FP8_E5M2, 1, 32, dict(tile="256x256", few_rows=-1), [(1, 300, 270, 160), (2, 257, 31, 96)]),
    ("panel 256x128", ref.FP8_E5M2, 1, 32, dict(tile="256x128", few_rows=-1), [(1, 300, 270, 160), (2, 257, 31, 96)]),
    ("panel 64x256", ref.FP8_E5M2, 0, 32, dict(tile="64x256", few_rows=-1), [(1, 300, 270, 160), (2, 65, 257, 96)]),
    ("panel, groups of 16, E4M3", ref.FP8_E4M3, 1, 16, dict(few_rows=-1), [(1, 130, 100, 64)]),
    ("hybrid", ref.FP8_E5M2, 1, 32, dict(e5m2_kernel="hybrid", few_rows=-1), [(1, 300, 270, 384), (2, 257, 31, 128)]),
    ("fused", ref.FP8_E5M2, 1, 32, dict(e5m2_kernel="fused", few_rows=-1), [(1, 300, 270, 384), (2, 257, 31, 128)]),
    ("block-scaled FP4", ref.E8M0_FLOOR, 0, 32, dict(few_rows=-1), [(1, 300, 270, 384), (2, 257, 31, 128)]),
    ("sign-split FP4", ref.E8M0_FLOOR, 1, 32, dict(pot_kernel="split", few_rows=-1), [(1, 300, 270, 384), (2, 257, 31, 128)]),
    ("merged FP8", ref.E8M0_FLOOR, 1, 32, dict(pot_kernel="merged_fp8", few_rows=-1), [(1, 300, 270, 160), (2, 257, 31, 96)]),
    ("merged FP6", ref.E8M0_FLOOR, 1, 32, dict(pot_kernel="merged_fp6", few_rows=-1), [(1, 300, 270, 160), (2, 257, 31, 96)]),
    ("few rows, one K slice", ref.FP8_E5M2, 1, 32, dict(few_rows=1), [(1, 5, 70, 512), (2, 33, 100, 256), (1, 200, 45, 512)]),
    ("few rows, K slices", ref.FP8_E5M2, 1, 32, dict(few_rows=2), [(1, 5, 70, 512), (2, 100, 100, 1024), (1, 250, 33, 512)]),
    ("few rows, power-of-two scales", ref.E8M0_FLOOR, 1, 32, dict(few_rows=3), [(1, 31, 65, 768)]),
]


@pytest.mark.parametrize("label,scale,asym,gs,opts,shapes", KERNELS, ids=[k[0] for k in KERNELS])
def test_gemm_writes_only_its_window(label, scale, asym, gs, opts, shapes):
    for batch, M, N, K in shapes:
        ac, as_, bc, bs = operands(batch, M, N, K, scale, asym, gs)
        buf, window, allowed, pattern = canary_window(batch, M, N, pad=37)
        fmt = binding.make_format(scale, asym, gs)
        out = window if batch > 1 else window[0]
        binding.gemm(fmt, *(G.to_dev_u8(t if batch > 1 else t[0]) for t in (ac, as_, bc, bs)), out=out,
                     options=binding.gemm_options(**opts))
        torch.cuda.synchronize()
        what = "%s %dx%dx%dx%d" % (label, batch, M, N, K)
        assert_padding_untouched(buf, allowed, pattern, what)
        Cr = ref.gemm(ac, as_, bc, bs, gs, scale, asym)
        assert G.rel_fro(window.cpu().numpy(), Cr) <= TOL, what


def test_scaled_gemm_writes_only_its_window():
    """The double-scaling product (tensor-wise scales in the epilogue of the panel kernel)."""
    M, N, K = 130, 100, 64
    a = synth.activations(M, K, seed=1, n_outlier=1, outlier_gain=30.0)
    b = synth.weights(N, K, seed=2)
    fmt = binding.make_format(binding.FP8_E4M3, True, 16)
    ad, bd = G.to_dev_bf16(a), G.to_dev_bf16(b)
    pa, pb = binding.tensor_scale(ad), binding.tensor_scale(bd)
    ac, as_ = binding.quantize(fmt, ad, tensor_pair=pa)
    bc, bs = binding.quantize(fmt, bd, tensor_pair=pb)
    buf, window, allowed, pattern = canary_window(1, M, N, pad=5)
    binding.gemm(fmt, ac, as_, bc, bs, out=window[0], a_pair=pa, b_pair=pb)
    torch.cuda.synchronize()
    assert_padding_untouched(buf, allowed, pattern, "scaled GEMM")
    sa, sb = float(pa[0]), float(pb[0])
    Cr = ref.gemm(ac.cpu().numpy(), as_.cpu().numpy(), bc.cpu().numpy(), bs.cpu().numpy(), 16, ref.FP8_E4M3, 1, sa, sb)
    assert G.rel_fro(window[0].cpu().numpy(), Cr) <= TOL


@pytest.mark.parametrize("scale,asym", [(ref.FP8_E5M2, 1), (ref.E8M0_FLOOR, 0), (ref.E8M0_FLOOR, 1)])
@pytest.mark.parametrize("M,width,K,pad", [(300, 96, 160, 8), (257, 160, 128, 3), (70, 32, 256, 0)])
def test_gated_gemm_writes_only_its_window(M, width, K, pad, scale, asym):
    """The GEMM with the gated activation as its epilogue writes BF16: through LDS with 16-byte stores when the output
    allows it (pad 8: leading dimension a multiple of 8), element by element otherwise (pad 3). Small problems: the kernel
    that reads both operands as packed codes, the merged FP6 kernel and, where K is no multiple of 128, the BF16 panels."""
    gated_window(M, width, K, pad, scale, asym)


@pytest.mark.parametrize("scale,asym,M,width,K,pad", [
    (ref.FP8_E5M2, 1, 800, 96, 160, 8), (ref.FP8_E5M2, 0, 801, 160, 128, 3),        # BF16 panels
    (ref.E8M0_FLOOR, 0, 800, 5504, 1024, 8), (ref.E8M0_FLOOR, 0, 801, 5536, 1024, 3),  # block-scaled FP4
    (ref.E8M0_ROUND, 0, 300, 160, 128, 3), (ref.E8M0_ROUND, 0, 70, 96, 256, 8),     # the same, few rows
    (ref.E8M0_FLOOR, 1, 800, 160, 1024, 8), (ref.E8M0_FLOOR, 1, 801, 96, 160, 3)])  # merged FP6
def test_gated_gemm_on_the_tiled_kernels_writes_only_its_window(M, width, K, pad, scale, asym):
    """The same on the three tiled kernels, partial tiles in both directions; and the oracle's gated activation of the
    oracle's product, on some rows: at most one BF16 step from it, by the FP32 accumulation's difference."""
    from tests.test_gpu_layer import assert_bf16_close
    a, wg, wu, window = gated_window(M, width, K, pad, scale, asym)
    rows = sorted({0, 1, 31, 32, M // 2, M - 2, M - 1} & set(range(M)))
    gu = ref.gemm(*ref.quantize(a[rows], 32, scale, asym), *ref.quantize(np.concatenate([wg, wu], 0), 32, scale, asym), 32,
                  scale, asym)
    assert_bf16_close(window[0][rows].contiguous(), layer_ref.silu_mul(gu.astype(np.float32)), "gated GEMM")


def gated_window(M, width, K, pad, scale, asym):
    import ctypes
    a = synth.activations(M, K, seed=M, n_outlier=1, outlier_gain=30.0)
    wg, wu = synth.weights(width, K, seed=3), synth.weights(width, K, seed=4)
    fmt = binding.make_format(scale, asym)
    ac, as_ = binding.quantize(fmt, G.to_dev_bf16(a))
    inter = binding.interleave_gate_up(G.to_dev_bf16(wg), G.to_dev_bf16(wu)).contiguous()
    ic, is_ = binding.quantize(fmt, inter)
    buf, window, allowed, pattern = canary_window(1, M, width, pad, dtype=torch.bfloat16)
    need = binding.gemm_silu_mul_workspace_bytes(fmt, M, width, K)
    ws = torch.empty(max(need, 1), dtype=torch.uint8, device="cuda")
    binding._check(binding.load().amxfp4_gemm_silu_mul(
        ctypes.byref(fmt), M, width, K, ac.data_ptr(), as_.data_ptr(), ic.data_ptr(), is_.data_ptr(),
        window.data_ptr(), width + pad, ws.data_ptr() if need else None, need, binding._stream()))
    torch.cuda.synchronize()
    assert_padding_untouched(buf, allowed, pattern, "gated GEMM %dx%dx%d" % (M, width, K))
    plain = binding.gemm_silu_mul(fmt, ac, as_, ic, is_)   # contiguous output of its own
    torch.cuda.synchronize()
    assert torch.equal(window[0].contiguous().view(torch.int16), plain.view(torch.int16))
    return a, wg, wu, window


@pytest.mark.parametrize("M,N,K,tile", [(1290, 8001, 384, 4), (300, 16001, 128, 5), (257, 8191, 4096, 6), (700, 11001, 128, 7)])
@pytest.mark.parametrize("pad", [37, 63])
def test_tiles_that_only_the_rule_picks_write_only_their_window(M, N, K, tile, pad):
    from tests.test_gpu_tile_order import operand, tile_of
    assert tile_of(M, N, K, whole_lines=False) == tile
    ac, as_, a = operand(M, K, 0x3C, 1, 3)
    bc, bs, b = operand(N, K, 0x3C, 1, 4)
    buf, window, allowed, pattern = canary_window(1, M, N, pad)
    binding.gemm(binding.make_format(ref.FP8_E5M2, 1, 32), ac, as_, bc, bs, out=window[0], options=binding.gemm_options(few_rows=-1))
    assert_padding_untouched(buf, allowed, pattern, "tile %d" % tile)
    assert torch.equal(window[0].double(), a @ b.T)


@pytest.mark.parametrize("M,N,K,pad", [(1100, 28672, 4096, 32), (1100, 28672, 4096, 5), (1290, 26688, 4096, 32)])
def test_weights_in_pieces_write_only_their_window(M, N, K, pad):
    """A pitch of whole lines, and of five rows of tiles any."""
    from tests.test_gpu_tile_order import operand
    from tests.test_routes import i32, i64, flag, rule
    assert rule("_ZN3amx22bf16_columns_at_a_timeEillllb", i64, i32, i64, i64, i64, i64, flag)(1, M, N, K, 1, pad % 32 == 0) < N
    ac, as_, a = operand(M, K, 0x3C, 1, 5)
    bc, bs, b = operand(N, K, 0x3C, 1, 6)
    buf, window, allowed, pattern = canary_window(1, M, N, pad)
    binding.gemm(binding.make_format(ref.FP8_E5M2, 1, 32), ac, as_, bc, bs, out=window[0], options=binding.gemm_options(few_rows=-1, tile="256x256"))
    assert_padding_untouched(buf, allowed, pattern, "pieces")
    for n0 in range(0, N, 4096):
        assert torch.equal(window[0][:, n0:n0 + 4096].double(), a @ b[n0:n0 + 4096].T)


@pytest.mark.parametrize("fmt_args", [(ref.E8M0_FLOOR, False), (ref.E8M0_FLOOR, True), (ref.FP8_E5M2, True)])
@pytest.mark.parametrize("M,N", [(300, 1057), (1100, 18721)])  # C below and above 80 MB, in either case more than one column of tiles
def test_store_policies_same_bits_and_only_the_window(M, N, fmt_args):
    """Rows of C that are whole lines, half lines and neither (by the pitch, and by the base's alignment) are stored in different ways,
    a large C in another way than a small one. The same product through all of them."""
    K = 256
    fmt = binding.make_format(*fmt_args, 32)
    gen = torch.Generator(device="cuda").manual_seed(M)
    a = binding.quantize(fmt, torch.randn((M, K), generator=gen, device="cuda").to(torch.bfloat16))
    b = binding.quantize(fmt, torch.randn((N, K), generator=gen, device="cuda").to(torch.bfloat16))
    options = binding.gemm_options(few_rows=-1)  # (the tiled kernels)
    base = None
    for pitch, shift in [((N + 31) // 32 * 32, 0), ((N + 15) // 16 * 16 + 16 * (((N + 15) // 16) % 2 == 0), 0), (N, 0), ((N + 31) // 32 * 32, 3)]:
        buf = torch.full((GUARD + shift + M * pitch + GUARD,), CANARY, dtype=torch.int32, device="cuda")
        body = buf[GUARD + shift:GUARD + shift + M * pitch].view(M, pitch)
        binding.gemm(fmt, *a, *b, out=body.view(torch.float32)[:, :N], options=options)
        got = body[:, :N].clone()
        base = got if base is None else base
        assert torch.equal(got, base), (pitch, shift)
        body[:, :N] = CANARY
        assert bool((buf == CANARY).all()), (pitch, shift)
    assert torch.isfinite(base.view(torch.float32)).all()


@pytest.mark.parametrize("M,N,K,batch,scaled,fmt_args", [
    (300, 1057, 4352, 1, False, (ref.E8M0_FLOOR, False, 32)), (300, 1057, 4352, 1, False, (ref.FP8_E5M2, True, 32)),  # a deep K: streaming
    (300, 1057, 4352, 1, False, (ref.E8M0_FLOOR, True, 32)),
    (300, 1057, 256, 3, False, (ref.E8M0_FLOOR, False, 32)), (300, 1057, 256, 3, False, (ref.FP8_E5M2, True, 32)),
    (300, 1057, 256, 3, False, (ref.E8M0_FLOOR, True, 32)),
    (1501, 1057, 256, 1, True, (ref.FP8_E4M3, False, 16)), (1501, 1057, 4352, 1, True, (ref.FP8_E4M3, True, 16))])
def test_store_policies_of_a_deep_k_a_batch_and_tensor_scales(M, N, K, batch, scaled, fmt_args):
    """Whole lines, half lines, neither, and rows at a pitch of 8192 elements (stored column by column): the same bits, only the window."""
    fmt = binding.make_format(*fmt_args)
    gen = torch.Generator(device="cuda").manual_seed(K + batch)
    x, w = (torch.randn((batch, r, K), generator=gen, device="cuda").to(torch.bfloat16) for r in (M, N))
    if scaled:
        pairs = [binding.tensor_scale(t[0]) for t in (x, w)]
        ops = [u for t, p in zip((x, w), pairs) for u in binding.quantize(fmt, t[0], tensor_pair=p)]
        how = {"a_pair": pairs[0], "b_pair": pairs[1]}
    else:
        ops = [u if batch > 1 else u[0] for t in (x, w) for u in binding.quantize_batched(fmt, t)]
        how = {"options": binding.gemm_options(few_rows=-1)}  # (the tiled kernels)
    base = None
    for pitch, shift in [(1088, 0), (1072, 0), (N, 0), (1088, 3), (8192, 0), (8192, 16)]:
        buf = torch.full((GUARD + shift + batch * M * pitch + GUARD,), CANARY, dtype=torch.int32, device="cuda")
        body = buf[GUARD + shift:GUARD + shift + batch * M * pitch].view(batch, M, pitch)
        out = body.view(torch.float32)[:, :, :N]
        binding.gemm(fmt, *ops, out=out if batch > 1 else out[0], **how)
        got = body[:, :, :N].clone()
        base = got if base is None else base
        assert torch.equal(got, base), (pitch, shift)
        body[:, :, :N] = CANARY
        assert bool((buf == CANARY).all()), (pitch, shift)
    assert torch.isfinite(base.view(torch.float32)).all()


@pytest.mark.parametrize("M", [1, 16, 19, 32])
def test_48_columns_to_a_workgroup_write_only_their_window(M):
    """(9001 columns: the last workgroup has 25)"""
    from tests.test_gpu_tile_order import operand
    ac, as_, a = operand(M, 512, 0x3C, 1, 3)
    bc, bs, b = operand(9001, 512, 0x3C, 1, 4)
    buf, window, allowed, pattern = canary_window(1, M, 9001, 37)
    binding.gemm(binding.make_format(ref.FP8_E5M2, 1, 32), ac, as_, bc, bs, out=window[0])
    assert_padding_untouched(buf, allowed, pattern, "48 columns")
    assert torch.equal(window[0].double(), a @ b.T)


@pytest.mark.parametrize("merged", [False, True])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("heads,Sq,Sk", [(3, 1, 64), (4, 33, 96), (8, 130, 320), (3, 161, 352), (720, 70, 160)])
def test_attention_writes_only_its_output(heads, Sq, Sk, D, merged):
    """The last rows of a wave's 32 queries lie past Sq: dropped by the window of the stores (heads of 128) or skipped. Guard words
    in front of the output and behind it; one head at a time gives the same rows, so no head wrote into another's."""
    fmt, gen = binding.make_format(ref.FP8_E5M2, 1, 32), torch.Generator("cuda").manual_seed(Sq)
    q, k, v = (torch.randn((n, s, D), generator=gen, device="cuda").to(torch.bfloat16) for n, s in ((heads, Sq), (heads, Sk), (heads, Sk)))
    ops = [binding.quantize_batched(fmt, q), binding.quantize_batched(fmt, k), binding.quantize_batched(fmt, v, k_axis=1)]
    dtype, pattern = (torch.bfloat16, 0x7FC5) if merged else (torch.float32, CANARY)
    buf = torch.full((2 * GUARD + heads * Sq * D,), pattern, dtype=torch.int16 if merged else torch.int32, device="cuda")
    body = buf[GUARD:GUARD + heads * Sq * D]
    out = body.view(dtype).view((Sq, heads * D) if merged else (heads, Sq, D))
    binding.attention(fmt, *ops[0], *ops[1], *ops[2], D ** -0.5, True, out=out, merged=merged)
    torch.cuda.synchronize()
    assert (buf[:GUARD] == pattern).all() and (buf[GUARD + heads * Sq * D:] == pattern).all() and (body != pattern).all()
    for h in {0, 1, heads // 2, heads - 1}:
        one = binding.attention(fmt, *(t[h:h + 1].contiguous() for pair in ops for t in pair), D ** -0.5, True, merged=merged)
        assert torch.equal(out.view(Sq, heads, D)[:, h] if merged else out[h], one if merged else one[0])
