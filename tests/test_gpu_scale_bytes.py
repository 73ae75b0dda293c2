"""Scale bytes that the cast writes rarely or never: every finite byte of a format, subnormal scales among them, and FP8 bytes
with the sign bit set, which the library ignores. Calls that promise each other's bits must agree on them."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_2411_09909_amd import binding, synth
from tests import gpu_util as G

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


@pytest.mark.parametrize("asym", [1, 0])
@pytest.mark.parametrize("M,N,K,gated", [(100, 70, 384, 0), (300, 70, 512, 0), (900, 300, 512, 0), (40, 128, 512, 1), (300, 128, 384, 1)])
def test_rounded_scales_of_the_largest_inputs(M, N, K, gated, asym):
    """The cast rounds the scale of a BF16 maximum above 1.41 * 2^127 up to 2^126 and its largest element to 4: 2^128, which
    has no 16-bit value. The block-scaled kernels multiply it by a small scale of the other operand all the same."""
    a = synth.activations(M, K, seed=M)
    a[:, 3], a[::2, 40] = 0x7F7F, 0xFF60  # the largest BF16 number, and a negative one above 1.41 * 2^127
    b = synth.weights(N, K, seed=N)
    b.reshape(-1)[:] = (b.reshape(-1) & 0x8000) | (0x1800 + (b.reshape(-1) & 0x3FF))  # 2^-79 or so
    fmt = binding.make_format(ref.E8M0_ROUND, asym, 32)
    (ac, as_), (bc, bs) = binding.quantize(fmt, G.to_dev_bf16(a)), binding.quantize(fmt, G.to_dev_bf16(b))
    assert int(as_.max()) == 253
    want = ref.gemm(ac.cpu().numpy(), as_.cpu().numpy(), bc.cpu().numpy(), bs.cpu().numpy(), 32, ref.E8M0_ROUND, asym)
    if gated:  # rows of B: 32 of the gate, 32 of the up half, in turn; silu(g) is g or nearly 0 at such magnitudes
        out = binding.gemm_silu_mul(fmt, ac, as_, bc, bs).float().cpu().numpy()
        g, u = (want.reshape(M, -1, 2, 32)[:, :, i].reshape(M, -1).astype(np.float64) for i in (0, 1))
        with np.errstate(over="ignore"):
            want = g / (1 + np.exp(-g)) * u
        fits = np.abs(want) < 2.0 ** 127
        assert np.isfinite(out[fits]).all() and G.rel_fro(out[fits], want[fits]) <= 2.0 ** -8
    else:
        C = binding.gemm(fmt, ac, as_, bc, bs).cpu().numpy()
        assert np.isfinite(C).all() and G.rel_fro(C, want) <= 1e-5


@pytest.mark.parametrize("asym", [1, 0])
@pytest.mark.parametrize("M,K", [(5, 256), (24, 288), (40, 544), (300, 288)])
def test_both_operands_packed_over_the_whole_range_of_power_of_two_scales(M, K, asym):
    """Bytes 0 .. 252 of E8M0 (the cast's largest, 2^125, for a BF16 maximum below 2^128), the small ones against the large
    ones so that the products stay in range; elements * 2^-127 are subnormal BF16 numbers."""
    N = 70
    fmt = binding.make_format(ref.E8M0_FLOOR, asym, 32)
    rng = np.random.default_rng(M)
    base = rng.integers(4, 249, K // 32)  # per group position; the other operand mirrors it around 126

    def packed(rows, centre):
        codes = rng.integers(0, 256, (rows, K // 2), dtype=np.uint8)
        shape = (rows, K // 32) + ((2,) if asym else ())
        spread = rng.integers(-4, 4, shape)
        return codes, (centre.reshape((1, -1) + (1,) * asym) + spread).astype(np.uint8)

    (ac, as_), (bc, bs) = packed(M, base), packed(N, 252 - base)
    as_[0], bs[0] = np.where(bs[0] > 126, 0, as_[0]), np.where(bs[0] > 126, 252, bs[0])  # 2^-127 against 2^125
    C = binding.gemm(fmt, *(torch.from_numpy(t).cuda() for t in (ac, as_, bc, bs))).cpu().numpy().astype(np.float64)
    ad, bd = (ref.dequantize(c, s, 32, ref.E8M0_FLOOR, asym).astype(np.float64) for c, s in ((ac, as_), (bc, bs)))
    # K exact products in FP32, any order: K roundings of partial sums, none above the sum of the magnitudes (and one
    # factor of two for the accumulation inside a matrix instruction)
    limit = 2.0 * (K + 2) * 2.0 ** -24 * (np.abs(ad) @ np.abs(bd).T) + 1e-30
    assert np.isfinite(C).all() and (np.abs(C - ad @ bd.T) <= limit).all()
