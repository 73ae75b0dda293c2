"""The order in which the GEMM kernels' tiles are dealt to the XCDs: every tile exactly once, also where the tiles are
dealt as equal runs instead of supertiles (a partial supertile in M or in N would cost a round). Integer operands with unit
scales: the sums stay below 2^24, so every kernel must give the exact product."""
import pytest
import torch

from oracle import ref
from paper_2411_09909_amd import binding

pytestmark = pytest.mark.gpu

VALUES = torch.tensor([0, .5, 1, 1.5, 2, 3, 4, 6, 0, -.5, -1, -1.5, -2, -3, -4, -6], dtype=torch.float64)  # of the codes


def operand(rows, K, unit, asym, seed):
    """Codes whose values are whole numbers (0.5 and 1.5 left out), every scale 1."""
    gen = torch.Generator("cuda").manual_seed(seed)
    pick = torch.tensor([0, 2, 4, 5, 6, 7, 8, 10, 12, 13, 14, 15], device="cuda", dtype=torch.uint8)
    nib = pick[torch.randint(0, len(pick), (rows, K), generator=gen, device="cuda")]
    codes = nib[:, 0::2] | (nib[:, 1::2] << 4)
    scales = torch.full((rows, K // 32) + ((2,) if asym else ()), unit, dtype=torch.uint8, device="cuda")
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
