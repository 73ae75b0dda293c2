// The stream GEMM (gemm_stream.h): when it takes a product, and its plain form. The gated form is a file of its own, so that
// the two compile side by side.
#include "gemm_stream.h"

namespace amx {

static bool pot_scales(int scale_kind) { return scale_kind == kScaleE8M0Floor || scale_kind == kScaleE8M0Round; }

// The rounded power-of-two scale of a BF16 maximum above 1.41 * 2^127 is 2^126, and its largest element 4: a value of 2^128,
// which no 16-bit float holds. The block-scaled kernels, which never form it, keep what they took of that format; this one
// takes it only where the few-rows kernel, with the same limit, did.
static bool rounded_pot(int scale_kind, int64_t group_size) { return scale_kind == kScaleE8M0Round && group_size == 32; }

// Time of this kernel for more than 64 rows, us, in the shape <2, 2, 4> below: workgroups of 64 x 64 outputs, 256 at a
// time. Fitted to K 1024 .. 13824, N 1024 .. 28672, 80 .. 2048 rows, where it is within 10 %.
static double stream_us(int scale_kind, bool asym, int64_t M, int64_t N, int64_t K) {
  const double rounds = (double)(((M + 63) / 64 * ((N + 63) / 64) + 255) / 256), k = (double)K / 4096.0;
  return asym ? 4.0 + k * (2.0 + 11.5 * rounds) : 4.0 + k * (1.5 + 9.3 * rounds);
}

// Symmetric power-of-two scales of 32-groups, more than 64 rows: whether the FP4 kernel is the fastest of the three that
// could take them. Besides the output it takes 11 us + 5 ns K, from K 2048 on 12.8 + 4.2 ns K, while its 256 x 256 tiles fit the
// compute units once (512 x 11008 x 1024 20 us, 1024 x 4096 x 2048 23, x 4096 31.6, output included); this kernel 3 us and per round of 256
// workgroups 1.25 us + 1.1 ns K, or 1.7 ns K if that is more (512 x 4096 x 4096, two rounds, 19; 1024 x 4096 x 2048, four, 20; 2048
// x 4096 x 128, eight, 20, the FP4 kernel 12.6). Up to 16384 rows; beyond, the FP4 kernel (32768 x 128 x 128 10.3 against 12.2,
// 100000 x 512 x 128 47 against 104). The few-rows kernel never is the fastest there (28672 x 8192: 80 rows 69 us, 256 rows 137,
// the FP4 kernel 66-69).
bool fp4_beats_stream(int64_t M, int64_t N, int64_t K, double c_bytes) {
  if (M <= 64) return false;
  const double k = (double)K, c = c_bytes * (double)M * (double)N, rounds = (double)(((M + 63) / 64 * ((N + 63) / 64) + 255) / 256);
  const double fp4 = (K < 2048 ? 11.0 + 0.005 * k : 12.8 + 0.0042 * k) + c / 6.5e6;
  const double short_k = 1.25 + 0.00107 * k, long_k = 0.00171 * k;
  return M > 16384 || fp4 <= 3.0 + rounds * (short_k > long_k ? short_k : long_k) + c / 5.1e6;
}

// Whether this kernel takes a product, single problems and batches alike unless said otherwise. us for the whole call,
// AMXFP4-E5M2, here / the kernel that took it otherwise:
//   up to 64 rows: always (1 x 4096 x 4096: 4.8 / 12.7;  64 x 1024 x 1024: 4.0 / 11.2;  32 x 11008 x 4096: 12.5 / 16.9;
//     32 x 28672 x 8192: 41 / 47;  64 x 28672 x 8192: 56 / 60;  groups of 16, whose weights were expanded to BF16 first,
//     24 x 11008 x 4096: 10 / 84)
//   single problems from there on, symmetric power-of-two scales: where the estimates above say so
//   the other formats: up to 256 rows, against weights below 2^27 elements (256 x 4096 x 4096: 17 / 50;  256 x 11008 x
//     4096: 40 / 79;  but 256 x 28672 x 8192: 177 / 151 on the few-rows kernel, which shares the dequantized A);
//     asymmetric power-of-two scales end here (prepared weights beyond 256 rows are their FP6 panel alone);
//   up to 512 rows likewise (512 x 4096 x 4096: 28 / 46;  512 x 4096 x 11008: 67 / 128;  512 x 14336 x 4096: 91 / 143);
//   up to 768 rows where the BF16 panels' tiles leave compute units idle: a long K or few columns (768 x 4096 x 11008:
//     97 / 134;  768 x 1024 x 1024: 7.7 / 17;  but 768 x 14336 x 4096: 135 / 129).
bool stream_path_preferred(int scale_kind, bool asym, int64_t group_size, int64_t M, int64_t N, int64_t K, int64_t batch) {
  if ((group_size != 32 && group_size != 16) || K % 32 != 0) return false;
  if (rounded_pot(scale_kind, group_size) && !skinny_path_supported(M, N, K, batch)) return false;
  if (M <= 64) return true;
  if (batch != 1) return false;
  if (group_size == 32 && pot_scales(scale_kind)) {
    if (!asym) return !fp4_path_supported(M, N, K) ? M <= 256 : !fp4_beats_stream(M, N, K, 4.0);
    return M <= 256 && N * K < (int64_t(1) << 27);
  }
  if (M > 768 || (N * K >= (int64_t(1) << 27) && (group_size == 32 || M > 256))) return false;
  return M <= 512 || K >= 8192 || (M + 63) / 64 * ((N + 63) / 64) <= 512;
}

// The same for the gated product, B [2 width][K] = [N][K]. Beyond 256 rows exactly where the plain product comes here (the
// two give the same bits); up to 256 rows the alternative is a tiled kernel, never the few-rows one, so large weights come
// here too (AMXFP4-E5M2, 28672 x 8192, 256 rows: 177 us against 350), and asymmetric power-of-two scales while the FP6
// kernel's merge of the weights and its one round of tiles, 20 us + 4.7 ns K + 0.37 ps N K, takes longer.
bool stream_glu_preferred(int scale_kind, bool asym, int64_t group_size, int64_t M, int64_t N, int64_t K) {
  if (rounded_pot(scale_kind, group_size)) return false;
  if (M > 64 && group_size == 32 && scale_kind == kScaleE8M0Floor && !asym)
    return !fp4_path_supported(M, N, K) ? M <= 256 : !fp4_beats_stream(M, N, K, 1.0);
  if (M > 256 || M <= 64) return stream_path_preferred(scale_kind, asym, group_size, M, N, K, 1);
  if ((group_size != 32 && group_size != 16) || K % 32 != 0) return false;
  if (group_size == 32 && pot_scales(scale_kind)) {
    return stream_us(scale_kind, asym, M, N, K) < 20.0 + 0.0047 * (double)K + 3.7e-7 * (double)N * (double)K;
  }
  return true;
}

hipError_t launch_gemm_stream(int scale_kind, bool asym, int64_t group_size, int64_t M, int64_t N, int64_t K,
                              const uint8_t* A_codes, const uint8_t* A_scales, const uint8_t* B_codes,
                              const uint8_t* B_scales, const float* A_tensor_pair, const float* B_tensor_pair, float* C,
                              int64_t ldc, int64_t batch, hipStream_t s, const KernelTimer& timer) {
  return stream_launch<false>(scale_kind, asym, group_size, M, N, K, A_codes, A_scales, B_codes, B_scales, A_tensor_pair,
                              B_tensor_pair, C, ldc, batch, s, timer);
}

}  // namespace amx
