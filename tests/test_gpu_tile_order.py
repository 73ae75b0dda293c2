"""The order in which the GEMM kernels' tiles are dealt to the XCDs: every tile exactly once, also where the tiles are
dealt as equal runs instead of supertiles (a partial supertile in M or in N would cost a round). Integer operands with unit
scales: the sums stay below 2^24, so every kernel must give the exact product."""
import pytest
import torch

from oracle import ref
from paper_2411_09909_amd import binding

pytestmark = pytest.mark.gpu

VALUES = torch.tensor([0, .5, 1, 1.5, 2, 3, 4, 6, 0, -.5, -1, -1.5, -2, -3, -4, -6], dtype=torch.float64)  # of the codes


def operand(rows, K, unit, asym, seed, gs=32):
    """Codes whose values are whole numbers (0.5 and 1.5 left out), every scale 1, the byte `unit`."""
    gen = torch.Generator("cuda").manual_seed(seed)
    pick = torch.tensor([0, 2, 4, 5, 6, 7, 8, 10, 12, 13, 14, 15], device="cuda", dtype=torch.uint8)
    nib = pick[torch.randint(0, len(pick), (rows, K), generator=gen, device="cuda")]
    codes = nib[:, 0::2] | (nib[:, 1::2] << 4)
    scales = torch.full((rows, K // gs) + ((2,) if asym else ()), unit, dtype=torch.uint8, device="cuda")
    return codes.contiguous(), scales, VALUES.cuda()[nib.long()]


@pytest.mark.parametrize("M,N", [(20, 33 * 256 - 7),    # one row of tiles, 33 columns
                                 (2300, 5100),          # 9 x 20 tiles: bands of 5 and 4 rows
                                 (1290, 28 * 256 + 1),  # 6 x 29
                                 (300, 250),            # fewer tiles than XCDs
                                 (2040, 8190)])         # 8 x 32: whole supertiles
@pytest.mark.parametrize("scale,asym,options", [
    (ref.FP8_E5M2, 1, dict(tile="256x256")), (ref.FP8_E5M2, 1, dict(tile="256x128")), (ref.FP8_E5M2, 1, dict(tile="64x256")),
    (ref.FP8_E5M2, 1, dict(e5m2_kernel="hybrid")), (ref.FP8_E5M2, 0, dict(e5m2_kernel="fused")),
    (ref.E8M0_FLOOR, 0, {}), (ref.E8M0_FLOOR, 1, dict(pot_kernel="merged_fp6")),
    (ref.E8M0_FLOOR, 1, dict(pot_kernel="merged_fp8")), (ref.E8M0_FLOOR, 1, dict(pot_kernel="split"))])
def test_every_tile_once(M, N, scale, asym, options):
    K = 128
    unit = 0x3C if scale == ref.FP8_E5M2 else 127
    ac, as_, a = operand(M, K, unit, asym, 1)
    bc, bs, b = operand(N, K, unit, asym, 2)
    out = torch.full((M, N), float("nan"), device="cuda")
    got = binding.gemm(binding.make_format(scale, asym, 32), ac, as_, bc, bs, out=out,
                       options=binding.gemm_options(few_rows=-1, **options))
    assert torch.equal(got.double(), a @ b.T)


@pytest.mark.parametrize("M,N,K,tile", [
    (1290, 8001, 384, 4), (1500, 7000, 256, 4),     # 192 x 256; 700 and 1290 rows: no multiple of 256
    (300, 16001, 128, 5), (700, 6130, 1024, 5),     # 192 x 128
    (70, 130, 2048, 6), (257, 8191, 4096, 6),       # 128 x 128
    (700, 11001, 128, 7), (1290, 6130, 1024, 7)])   # 192 x 192
def test_tiles_between_the_three_large_ones(M, N, K, tile):
    """The shapes that only the rule picks: remainders in M and N, tiles that reach beyond the 256 rows a panel ends on."""
    from tests.test_routes import i32, i64, flag, rule
    choice = rule("_ZN3amx16bf16_tile_choiceElll", i32, i64, i64, i64)(M, N, 1)
    assert rule("_ZN3amx17bf16_tile_refinedEillllb", i32, i32, i64, i64, i64, i64, flag)(choice, M, N, K, 1, False) == tile
    ac, as_, a = operand(M, K, 0x3C, 1, 3)
    bc, bs, b = operand(N, K, 0x3C, 1, 4)
    out = torch.full((M, N), float("nan"), device="cuda")
    got = binding.gemm(binding.make_format(ref.FP8_E5M2, 1, 32), ac, as_, bc, bs, out=out, options=binding.gemm_options(few_rows=-1))
    assert torch.equal(got.double(), a @ b.T)


def tile_of(M, N, K, gated=False, whole_lines=True):
    from tests.test_routes import i32, i64, flag, rule
    return rule("_ZN3amx9bf16_tileEllllbbb", i32, i64, i64, i64, i64, flag, flag, flag)(M, N, K, 1, gated, False, whole_lines)


@pytest.mark.parametrize("asym", [0, 1])
@pytest.mark.parametrize("M,N,K,tile", [(1290, 8000, 384, 4), (257, 13120, 384, 5), (801, 1024, 2080, 6)])
def test_gated_product_on_the_tiles_between(M, N, K, tile, asym):
    """Their gated epilogue: bit for bit the separate operator on the exact sums (whole numbers)."""
    assert tile_of(M, N, K, gated=True) == tile
    ac, as_, a = operand(M, K, 0x3C, asym, 7)
    bc, bs, b = operand(N, K, 0x3C, asym, 8)
    got = binding.gemm_silu_mul(binding.make_format(ref.FP8_E5M2, asym, 32), ac, as_, bc, bs)
    pairs = (a @ b.T).float().view(M, N // 64, 2, 32)  # blocks of 32 gate and up columns in turn
    want = binding.silu_mul(torch.cat([pairs[:, :, 0].reshape(M, N // 2), pairs[:, :, 1].reshape(M, N // 2)], 1))
    assert torch.equal(got.view(torch.int16), want.view(torch.int16))


@pytest.mark.parametrize("asym", [0, 1])
@pytest.mark.parametrize("M,N,K,tile", [(801, 9985, 384, 4), (257, 13057, 384, 5), (801, 1025, 2080, 6), (700, 11001, 384, 7)])
def test_tensor_scales_on_the_tiles_between(M, N, K, tile, asym):
    """Their epilogue with tensor-wise scales (powers of two here), E4M3 group scales in groups of 16: the exact product."""
    assert tile_of(M, N, K, whole_lines=False) == tile
    ac, as_, a = operand(M, K, 0x38, asym, 9, gs=16)
    bc, bs, b = operand(N, K, 0x38, asym, 10, gs=16)
    pa, pb = torch.tensor([8.0, 0.125], device="cuda"), torch.tensor([0.25, 4.0], device="cuda")
    out = torch.full((M, N), float("nan"), device="cuda")
    got = binding.gemm(binding.make_format(ref.FP8_E4M3, asym, 16), ac, as_, bc, bs, out=out, a_pair=pa, b_pair=pb)
    assert torch.equal(got.double(), 2.0 * (a @ b.T))


@pytest.mark.parametrize("M,N,K", [(1100, 28672, 4096), (1290, 26688, 4096)])
def test_wide_weights_in_pieces(M, N, K):
    """B's panel goes through the workspace in pieces (the last one shorter): the exact product, and bit for bit what prepared
    weights give, whose panel is whole; the gated product likewise."""
    from tests.test_routes import i32, i64, flag, rule
    at_a_time = rule("_ZN3amx22bf16_columns_at_a_timeEillllb", i64, i32, i64, i64, i64, i64, flag)(1, M, N, K, 1, True)
    assert at_a_time < N and N % at_a_time != 0
    ac, as_, a = operand(M, K, 0x3C, 1, 5)
    bc, bs, b = operand(N, K, 0x3C, 1, 6)
    fmt, options = binding.make_format(ref.FP8_E5M2, 1, 32), binding.gemm_options(few_rows=-1, tile="256x256")
    out = torch.full((M, N), float("nan"), device="cuda")
    got = binding.gemm(fmt, ac, as_, bc, bs, out=out, options=options)
    for n0 in range(0, N, 4096):
        assert torch.equal(got[:, n0:n0 + 4096].double(), a @ b[n0:n0 + 4096].T)
    prepared = binding.prepare_weights(fmt, bc, bs)
    assert torch.equal(binding.gemm_prepared(fmt, ac, as_, bc, bs, prepared), binding.gemm(fmt, ac, as_, bc, bs))
    assert torch.equal(binding.gemm_silu_mul(fmt, ac, as_, bc, bs, prepared=prepared), binding.gemm_silu_mul(fmt, ac, as_, bc, bs))


@pytest.mark.parametrize("M,N,K,scale,unit,asym,gs", [
    (1100, 28672, 4096, ref.FP8_E5M2, 0x3C, 0, 32), (1100, 28672, 4096, ref.FP8_E4M3, 0x38, 0, 16),
    (1290, 26688, 4096, ref.FP8_E4M3, 0x38, 1, 16),
    (1100, 14112, 8192, ref.FP8_E5M2, 0x3C, 1, 32)])  # five rows of tiles: the larger limit of a piece (204 MB)
def test_pieces_of_other_formats(M, N, K, scale, unit, asym, gs):
    """The offset of a piece's scale bytes depends on the group size and on whether the signs have scales of their own. Scales of 1 and
    2 by blocks of rows, so that a wrong row's scale shows."""
    from tests.test_routes import i32, i64, flag, rule
    at_a_time = rule("_ZN3amx22bf16_columns_at_a_timeEillllb", i64, i32, i64, i64, i64, i64, flag)(1, M, N, K, 1, True)
    assert at_a_time < N and N % at_a_time != 0
    ac, as_, a = operand(M, K, unit, asym, 11, gs)
    bc, bs, b = operand(N, K, unit, asym, 12, gs)
    twice = torch.arange(N, device="cuda") % 96 >= 48
    bs[twice] = unit + (4 if scale == ref.FP8_E5M2 else 8)
    b[twice] *= 2
    out = torch.full((M, N), float("nan"), device="cuda")
    got = binding.gemm(binding.make_format(scale, asym, gs), ac, as_, bc, bs, out=out, options=binding.gemm_options(few_rows=-1, tile="256x256"))
    for n0 in range(0, N, 4096):
        assert torch.equal(got[:, n0:n0 + 4096].double(), a @ b[n0:n0 + 4096].T)
