"""Scale bytes that the cast writes rarely or never: every finite byte of a format, subnormal scales among them, and FP8 bytes
with the sign bit set, which the library ignores. Calls that promise each other's bits must agree on them."""
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


SIGN_ROUTES = [("default, large", 800, 11008, 256, None), ("hybrid", 300, 270, 384, dict(e5m2_kernel="hybrid", few_rows=-1)),
               ("fused", 300, 270, 384, dict(e5m2_kernel="fused", few_rows=-1)), ("panel", 300, 270, 384, dict(tile="256x256", few_rows=-1)),
               ("few rows", 100, 270, 512, dict(few_rows=1)), ("both operands packed", 40, 270, 512, None)]


@pytest.mark.parametrize("scale", [ref.FP8_E5M2, ref.FP8_E4M3])
@pytest.mark.parametrize("asym", [1, 0])
@pytest.mark.parametrize("route,M,N,K,options", SIGN_ROUTES, ids=[r[0] for r in SIGN_ROUTES])
def test_sign_bit_of_fp8_scale_bytes_is_ignored(route, M, N, K, options, asym, scale):
    fmt = binding.make_format(scale, asym, 32)
    (ac, as_), (bc, bs) = operand(M, K, asym, 0, 0x7C, 3), operand(N, K, asym, 0, 0x7C, 4)
    opts = binding.gemm_options(**options) if options is not None else None
    clean = binding.gemm(fmt, ac, as_, bc, bs, options=opts)
    signed_b = binding.gemm(fmt, ac, as_, bc, bs | 0x80, options=opts)
    signed_a = binding.gemm(fmt, ac, as_ | 0x80, bc, bs, options=opts)
    assert torch.equal(bits(clean), bits(signed_b)) and torch.equal(bits(clean), bits(signed_a))
