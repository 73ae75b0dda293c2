"""Scale bytes that the cast writes rarely or never: every finite byte of a format, subnormal scales among them. Calls that
promise each other's bits must agree on them."""
import pytest
import torch

from oracle import ref
from paper_2411_09909_amd import binding

pytestmark = pytest.mark.gpu


def operand(rows, K, asym, lo, hi, seed, gs=32):
    """Random codes, scale bytes spread over lo .. hi - 1."""
    gen = torch.Generator("cuda").manual_seed(seed)
    codes = torch.randint(0, 256, (rows, K // 2), dtype=torch.uint8, device="cuda", generator=gen)
    shape = (rows, K // gs) + ((2,) if asym else ())
    return codes, torch.randint(lo, hi, shape, dtype=torch.uint8, device="cuda", generator=gen)


def bits(t):
    return t.view(torch.int32)


# 800 x 11008: few rounds of tiles against a wide B, where expanding B takes a good part of the call
@pytest.mark.parametrize("asym", [1, 0])
@pytest.mark.parametrize("M,N,K", [(800, 11008, 128), (833, 11007, 4096)])
def test_wide_e5m2_product_has_the_panels_bits_for_every_scale_byte(M, N, K, asym):
    """Prepared weights read panels and promise the bits of the plain call, whichever kernel that takes."""
    fmt = binding.make_format(ref.FP8_E5M2, asym, 32)
    a, b = operand(M, K, asym, 0, 0x7C, 1), operand(N, K, asym, 0, 0x7C, 2)
    plain = binding.gemm(fmt, *a, *b)
    panel = binding.gemm(fmt, *a, *b, options=binding.gemm_options(tile="256x256", few_rows=-1))
    prepared = binding.gemm_prepared(fmt, *a, *b, binding.prepare_weights(fmt, *b))
    assert torch.isfinite(plain).all()
    assert torch.equal(bits(plain), bits(panel)) and torch.equal(bits(plain), bits(prepared))
