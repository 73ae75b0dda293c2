"""The GEMM for few rows and small problems that reads both operands as packed codes in one launch (gemm_stream.hip),
against the oracle: every workgroup shape of its rule, partial row and column tiles, K tails, groups of 16, batches,
tensor-wise scales, and nothing written outside the product."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_2411_09909_amd import binding, synth
from tests import gpu_util as G

pytestmark = pytest.mark.gpu

FORMATS = [(ref.FP8_E5M2, 1, 32), (ref.FP8_E5M2, 0, 32), (ref.E8M0_FLOOR, 1, 32), (ref.E8M0_ROUND, 0, 32),
           (ref.FP8_E4M3, 1, 32), (ref.FP8_E4M3, 0, 16), (ref.FP8_E4M3, 1, 16), (ref.FP8_E5M2, 1, 16),
           (ref.E8M0_FLOOR, 0, 16)]

# M: both sides of 16, 32, 64, 256, 512 and 768 rows. N: one column, partial tiles, each tile count at which the rule
# changes shape (256 tiles and one more). K: one block, one block per wave and one more, tails of one to seven groups.
SHAPES = [(1, 1, 32), (16, 17, 256), (5, 100, 2304), (13, 33, 2272), (16, 4097, 256), (3, 8193, 288), (2, 16400, 256),
          (17, 31, 512), (32, 65, 2048), (20, 4097, 512), (32, 8193, 256), (25, 16385, 256), (31, 50, 4544),
          (33, 64, 256), (64, 45, 2560), (40, 8193, 256), (64, 33, 96), (50, 70, 4448), (64, 4097, 256),
          (65, 100, 512), (96, 8200, 256), (128, 4129, 288), (250, 4097, 256), (257, 65, 2304), (300, 4100, 256),
          (512, 4160, 288), (513, 130, 2080), (768, 2050, 512)]


def bound(a, b, K):
    """Largest error an FP32 sum of K exact products can have in any order: K roundings of partial sums, none above the
    sum of the products' magnitudes (and one factor of two for the accumulation inside a matrix instruction)."""
    return 2.0 * (K + 2) * 2.0 ** -24 * (np.abs(a) @ np.abs(b).T) + 1e-30


@pytest.mark.parametrize("scale,asym,gs", FORMATS)
@pytest.mark.parametrize("M,N,K", SHAPES)
def test_against_the_oracle(M, N, K, scale, asym, gs):
    a = synth.activations(M, K, seed=M + K, n_outlier=1, outlier_gain=60.0)
    b = synth.weights(N, K, seed=N)
    ac, as_ = ref.quantize(a, gs, scale, asym)
    bc, bs = ref.quantize(b, gs, scale, asym)
    fmt = binding.make_format(scale, asym, gs)
    ops = [G.to_dev_u8(t) for t in (ac, as_, bc, bs)]
    # a window of a larger buffer, pattern around it
    pad = torch.full((M + 2, N + 5), -7.0, device="cuda")
    out = pad[1:M + 1, :N]
    binding.gemm(fmt, *ops, out=out)
    torch.cuda.synchronize()
    C = out.cpu().numpy().astype(np.float64)
    ad, bd = (ref.dequantize(c, s, gs, scale, asym).astype(np.float64) for c, s in ((ac, as_), (bc, bs)))
    assert (np.abs(C - ad @ bd.T) <= bound(ad, bd, K)).all()
    full = pad.cpu().numpy()
    assert (full[0] == -7).all() and (full[M + 1] == -7).all() and (full[:, N:] == -7).all()
    # the tiled kernels on the same operands (options keep them)
    other = binding.gemm(fmt, *ops, options=binding.gemm_options(few_rows=-1)).cpu().numpy().astype(np.float64)
    assert (np.abs(other - ad @ bd.T) <= bound(ad, bd, K)).all()


@pytest.mark.parametrize("scale,gs", [(ref.FP8_E5M2, 32), (ref.FP8_E4M3, 32), (ref.FP8_E4M3, 16), (ref.E8M0_FLOOR, 32)])
@pytest.mark.parametrize("M", [7, 24, 48])
def test_every_scale_byte(M, scale, gs):
    """Operands made of random codes and of every scale byte of the format in turn (subnormal scales, zero, the largest),
    the two signs of a group different ones; batch of two, K with a tail."""
    rng = np.random.default_rng(M)
    N, K, batch = 70, 544, 2
    top = {ref.FP8_E5M2: 0x7C, ref.FP8_E4M3: 0x7F, ref.E8M0_FLOOR: 140}[scale]
    low = 110 if scale == ref.E8M0_FLOOR else 0

    def operand(rows, first):
        codes = rng.integers(0, 256, (batch, rows, K // 2), dtype=np.uint8)
        n = batch * rows * (K // gs) * 2
        scales = (low + (first + 7 * np.arange(n)) % (top - low)).astype(np.uint8).reshape(batch, rows, K // gs, 2)
        return codes, scales

    (ac, as_), (bc, bs) = operand(M, 0), operand(N, 3)
    C = G.gpu_gemm(ac, as_, bc, bs, scale, 1, group_size=gs).astype(np.float64)
    for i in range(batch):
        ad, bd = (ref.dequantize(c[i], s[i], gs, scale, 1).astype(np.float64) for c, s in ((ac, as_), (bc, bs)))
        assert (np.abs(C[i] - ad @ bd.T) <= bound(ad, bd, K)).all()


def test_fp4_kernel_for_few_rows_against_large_weights():
    """Symmetric power-of-two scales, 80 rows against weights so large that the FP4 kernel is the fastest of those that
    could take them: the workspace asked for is good for it, and the product is right with exactly that much."""
    M, N, K = 80, 20000, 8192
    fmt = binding.make_format(ref.E8M0_FLOOR, 0, 32)
    ac, as_ = ref.quantize(synth.activations(M, K, seed=1), 32, ref.E8M0_FLOOR, 0)
    bc, bs = ref.quantize(synth.weights(N, K, seed=2), 32, ref.E8M0_FLOOR, 0)
    C = G.gpu_gemm(ac, as_, bc, bs, ref.E8M0_FLOOR, 0)
    ad, bd = (ref.dequantize(c, s, 32, ref.E8M0_FLOOR, 0).astype(np.float64) for c, s in ((ac, as_), (bc, bs)))
    assert (np.abs(C - ad @ bd.T) <= bound(ad, bd, K)).all()
    few = binding.gemm_options(few_rows=1)
    assert binding.gemm_workspace_bytes(fmt, M, N, K) >= binding.gemm_workspace_bytes(fmt, M, N, K, options=few)


@pytest.mark.parametrize("M,N,K,asym", [(1, 300, 1024, 0), (24, 4100, 512, 1), (64, 130, 4512, 0), (200, 300, 1056, 1), (1000, 1000, 1024, 0),
                                        (1100, 520, 2048, 1), (1400, 1001, 1024, 0)])
def test_tensor_scaled(M, N, K, asym):
    """Double scaling on the few-rows shapes, and of the many rows that come here with it alone: the product of the dequantized operands times the two tensor-wise scales."""
    fmt = binding.make_format(ref.FP8_E4M3, asym, 16)
    x = G.to_dev_bf16(synth.activations(M, K, seed=M, n_outlier=1, outlier_gain=60.0))
    w = G.to_dev_bf16(synth.weights(N, K, seed=N))
    xp, wp = binding.tensor_scale(x), binding.tensor_scale(w)
    xc, xs = binding.quantize(fmt, x, tensor_pair=xp)
    wc, ws = binding.quantize(fmt, w, tensor_pair=wp)
    C = binding.gemm(fmt, xc, xs, wc, ws, a_pair=xp, b_pair=wp).double()
    xd = binding.dequantize(fmt, xc, xs, torch.float32).double()
    wd = binding.dequantize(fmt, wc, ws, torch.float32).double()
    alpha = float(xp[0]) * float(wp[0])
    err = (C - (xd @ wd.T) * alpha).abs()
    # the sum's bound, and two more roundings: the product of the two scales and the product with it
    limit = (2.0 * (K + 4) * 2.0 ** -24) * (xd.abs() @ wd.abs().T) * alpha
    assert bool((err <= limit + 1e-30).all())


@pytest.mark.parametrize("scale,asym,gs", [(ref.FP8_E5M2, 1, 32), (ref.E8M0_FLOOR, 1, 32), (ref.E8M0_FLOOR, 0, 32),
                                           (ref.FP8_E4M3, 0, 16)])
@pytest.mark.parametrize("M,width,K", [(1, 32, 256), (16, 2080, 288), (20, 96, 2304), (32, 8320, 256), (64, 64, 544),
                                       (100, 4128, 256), (256, 160, 2048), (257, 96, 512), (500, 2080, 288)])
def test_gated_product(M, width, K, scale, asym, gs):
    """The gate / up projection with the activation in the epilogue: every workgroup shape, K tails, rows around 16, 32, 64
    and 256, into a window of a larger buffer."""
    fmt = binding.make_format(scale, asym, gs)
    x = synth.activations(M, K, seed=M, n_outlier=1, outlier_gain=30.0)
    wg, wu = (G.to_dev_bf16(synth.weights(width, K, seed=i)) for i in (1, 2))
    xc, xs = binding.quantize(fmt, G.to_dev_bf16(x))
    wc, ws = binding.quantize(fmt, binding.interleave_gate_up(wg, wu).contiguous())
    pad = torch.full((M + 2, width + 8), -7.0, dtype=torch.bfloat16, device="cuda")
    out = pad[1:M + 1, :width]
    binding.gemm_silu_mul(fmt, xc, xs, wc, ws, out=out)
    torch.cuda.synchronize()
    xd = binding.dequantize(fmt, xc, xs, torch.float32).double()
    gd, ud = (binding.dequantize(fmt, *binding.quantize(fmt, w), torch.float32).double() for w in (wg, wu))
    g, u = xd @ gd.T, xd @ ud.T
    # one BF16 rounding, a few FP32 ones, and what the sums' own errors do to silu(g) * u (|silu'| <= 1.1, |silu| <= |g|)
    sums = 2.0 * (K + 2) * 2.0 ** -24
    eg, eu = sums * (xd.abs() @ gd.abs().T), sums * (xd.abs() @ ud.abs().T)
    want = torch.nn.functional.silu(g) * u
    limit = (2.0 ** -8 + 2.0 ** -20) * want.abs() + 1.1 * eg * (u.abs() + eu) + g.abs() * eu + 1e-30
    assert bool(((out.double() - want).abs() <= limit).all())
    full = pad.float()
    assert bool((full[0] == -7).all() and (full[M + 1] == -7).all() and (full[:, width:] == -7).all())


@pytest.mark.parametrize("scale,asym,gs", [(ref.FP8_E5M2, 1, 32), (ref.E8M0_FLOOR, 1, 32), (ref.E8M0_FLOOR, 0, 32), (ref.FP8_E4M3, 0, 16)])
@pytest.mark.parametrize("M,N,K", [(1, 9001, 256), (16, 12288, 768), (17, 8203, 2304), (32, 16397, 256)])
def test_48_columns_to_a_workgroup(M, N, K, scale, asym, gs):
    """Up to 32 rows against columns that fill the compute units better in workgroups of 48 (stream_48_columns() in
    gemm_stream.h): one and two row tiles, remainders in M and N, fewer K blocks than waves and more."""
    test_against_the_oracle(M, N, K, scale, asym, gs)


@pytest.mark.parametrize("scale,asym,gs", FORMATS)
@pytest.mark.parametrize("N,K", [(17, 32), (300, 544), (4100, 2304), (8200, 256), (8193, 2272), (11008, 512), (16400, 288), (320, 544), (64, 2272)])
def test_one_to_four_rows_same_bits_as_more(N, K, scale, asym, gs):
    """Up to four rows the lanes share out A's rows; from five rows on each dequantizes its own. The same values in the same order: the
    rows of a product of nine rows, bit for bit, for random codes and scale bytes (the sign bit of an FP8 one among them, which is
    ignored)."""
    gen = torch.Generator(device="cuda").manual_seed(N + K)
    bytes_ = lambda *s, lo=0, hi=256: torch.randint(lo, hi, s, generator=gen, device="cuda", dtype=torch.uint8)  # noqa: E731
    # scale bytes whose products stay finite: E5M2 and E4M3 below NaN / infinity, E8M0 around 2^0
    lo, hi = {ref.FP8_E5M2: (0, 0x7C), ref.FP8_E4M3: (0, 0x7F), ref.E8M0_FLOOR: (100, 150), ref.E8M0_ROUND: (100, 150)}[scale]
    pair = (2,) if asym else ()
    fmt = binding.make_format(scale, asym, gs)
    ac, as_, bc, bs = bytes_(9, K // 2), bytes_(9, K // gs, *pair, lo=lo, hi=hi), bytes_(N, K // 2), bytes_(N, K // gs, *pair, lo=lo, hi=hi)
    if scale in (ref.FP8_E5M2, ref.FP8_E4M3):
        as_ |= bytes_(*as_.shape) & 0x80
    more = binding.gemm(fmt, ac, as_, bc, bs)
    assert torch.isfinite(more).all()
    for m in (1, 2, 3, 4):
        few = binding.gemm(fmt, ac[:m].contiguous(), as_[:m].contiguous(), bc, bs)
        assert torch.equal(few.view(torch.int32), more[:m].view(torch.int32)), m
    if N % 64 == 0:
        glu = [binding.gemm_silu_mul(fmt, ac[:m].contiguous(), as_[:m].contiguous(), bc, bs) for m in (1, 4, 9)]
        for g in glu:
            assert torch.equal(g.view(torch.int16), glu[2][:g.shape[0]].view(torch.int16))


@pytest.mark.parametrize("scale,asym,gs", [(ref.FP8_E5M2, 1, 32), (ref.E8M0_FLOOR, 0, 32), (ref.FP8_E4M3, 0, 16)])
@pytest.mark.parametrize("M", [1, 4, 5])
@pytest.mark.parametrize("N,K", [(300, 544), (4100, 512)])
def test_a_batch_of_few_rows_same_bits_as_single_products(M, N, K, scale, asym, gs):
    fmt, gen = binding.make_format(scale, asym, gs), torch.Generator(device="cuda").manual_seed(M + N)
    a, b = (binding.quantize_batched(fmt, torch.randn((3, r, K), generator=gen, device="cuda").to(torch.bfloat16)) for r in (M, N))
    C = binding.gemm(fmt, *a, *b)
    for i in range(3):
        one = binding.gemm(fmt, *(t[i].clone() for t in a + b))  # (a slice of its own alignment would be refused)
        assert torch.equal(C[i].view(torch.int32), one.view(torch.int32))
