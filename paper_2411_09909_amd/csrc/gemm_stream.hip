// The stream GEMM (gemm_stream.h): when it takes a product, and its plain form. The gated form is a file of its own, so that
// the two compile side by side.
#include "gemm_stream.h"

namespace amx {

static bool pot_scales(int scale_kind) { return scale_kind == kScaleE8M0Floor || scale_kind == kScaleE8M0Round; }

// The rounded power-of-two scale of a BF16 maximum above 1.41 * 2^127 is 2^126, and its largest element 4: a value of 2^128,
// which no 16-bit float holds. The block-scaled kernels, which never form it, keep what they took of that format; this one
// takes it only where the few-rows kernel, with the same limit, did.
static bool rounded_pot(int scale_kind, int64_t group_size) { return scale_kind == kScaleE8M0Round && group_size == 32; }

// Time of this kernel for more than 64 rows, us: 64 x 64 outputs per workgroup, counted in rounds of 256 (two share a
// compute unit and its vector unit, which is the bound), or the smaller shapes that still give each compute unit one;
// writing C counts (c_bytes per element of M x N), and so does loading scale bytes one by one where K is no multiple of
// 256. Within some 10 % at 96 .. 768 rows, N 1024 .. 32001, K 1024 .. 14336.
static double stream_us(bool asym, int64_t group_size, int64_t M, int64_t N, int64_t K, double c_bytes) {
  const int64_t rows32 = (M + 31) / 32, t32 = (N + 31) / 32, t64 = (N + 63) / 64;
  const double rounds = (double)(((M + 63) / 64 * t64 + 255) / 256);
  const double per_4096 = rows32 * t32 <= 256   ? (asym ? 4.4 : 3.0)
                          : rows32 * t64 <= 256 ? (asym ? 7.5 : 5.0)
                          : rounds == 1.0       ? (asym ? 11.0 : 9.0)
                                                : (asym ? 10.4 : 7.8) * rounds;
  const double tail = K % kStreamBlockK == 0 ? 1.0 : group_size == 16 ? (asym ? 2.0 : 1.65) : asym ? 1.5 : 1.25;
  return tail * (3.5 + per_4096 * (double)K / 4096.0) + c_bytes * (double)M * (double)N / 5.1e6;
}

// More than 256 rows of FP8-scaled operands on this kernel although the estimates above, made for weights that stay in the
// caches, say the panels: the panels' tiles then wait for memory (a 4096 x 14336 product takes 155 us at 320 as at 768 rows,
// and 30 more for the expansion), this kernel reads a quarter of the bytes. Measured on three sets of buffers in turn, 2945
// sizes of 257 to 1700 rows, N 1000 to 33000, K 1024 to 28672; us on the panels / here / the panels with prepared weights:
// E5M2 symmetric 768 x 8192 x 8192 149 / 99 / 106; asymmetric 149 / 135 / 105, which therefore stays on the panels; NVFP4 320 x 8192 x 28672 466 / 167, 640 x
// 28672 x 8192 461 / 311, 1024 x 8192 x 8192 178 / 136.
// Up to 768 rows: a product on prepared weights goes where the plain one goes, and beyond 768 rows it reads nothing but the
// prepared form. For the same reason the estimate here has to be 8 % below that of the panels without the expansion, 12 % up
// to a K of 4096 (547 x 8960 x 3072, symmetric, prepared, 32 / 36), 15 % for a K below 2048 (757 x 6496 x 1536 26 / 28;
// below 1024 none: 550 x 13952 x 512 20 / 26), 25 % for one that is no multiple of 256.
// Tensor-wise scales have no prepared form: their line is against the whole call, they come here up to 1500 rows, by 18 %
// from 1025 on (at 8 %: 1343 x 6144 x 4096 71 / 81), and alone against 2^27 weight elements or more, there up to 1024 rows
// (1500 x 28672 x 8192 645 / 770). Beyond 1500 rows the panels (1683 x 9184 x 28672 793 / 881).
// Nor may weights that stay in the caches lose (3400 calls whose route these lines had moved, the same buffers again and again, us
// before / here): no product without tensor-wise scales comes here whose estimate is above that of its prepared form on the tile that
// it runs (symmetric, prepared, 548 x 11008 x 4096 51 / 61, 576 x 11296 x 6400 71 / 94, 525 x 17792 x 6144 94 / 131; of 56 such sizes the least 1.12
// times, although the plain call gains a tenth there; of 154 that stay the slowest 1.03 times, 0.74 on average), and beyond 768 rows
// the estimate has to be 7 % below that of the panels as they are in the caches (NVFP4 1344 x 4096 x 14336 163 / 176, 973 x 8192 x 8192
// 139 / 148, 1138 x 5120 x 13824 167 / 178; from memory those gained 2 to 5 %). What is left, of 4530: single sizes
// (NVFP4 953 x 8544 x 5888 102 / 117), and below 257 rows, where this rule has no say, symmetric, prepared, 200 rows and more of a K
// that is no multiple of 256 (206 x 24128 x 9888 158 / 169; the plain call takes half the time there).
static bool beats_panels(bool asym, int64_t group_size, bool scaled, int64_t M, int64_t N, int64_t K) {
  if (M <= 256 || M > (scaled ? 1500 : 768) || K < 1024) return false;
  if (N * K >= (int64_t(1) << 27) && (!scaled || M > 1024)) return false;
  const int64_t rows32 = (M + 31) / 32, t32 = (N + 31) / 32, t64 = (N + 63) / 64, groups = (M + 63) / 64 * t64;
  const double k = (double)K, rounds = (double)((groups + 255) / 256);
  double here = 1.03 * stream_us(asym, group_size, M, N, K, 4.0);
  if (K % kStreamBlockK == 0 && rounds > 1.0 && rows32 * t32 > 256 && rows32 * t64 > 256) {
    const double small_groups = group_size == 16 ? (asym ? 1.13 : 1.05) : 1.0, many = rounds > 8.0 ? 1.05 : 1.0;
    here = 3.5 + (asym ? 10.9 : 7.9) * rounds * small_groups * many * k / 4096.0 + 4.0 * (double)(M * N) / 5.1e6;
  }
  // (the estimate of the panels is of weights in the caches too; from K 4608 on it falls short, by a quarter from 13824 on)
  const double cold = K <= 4608 ? 1.0 : K >= 13824 ? 1.25 : 1.0 + 0.25 * (k - 4608.0) / 9216.0;
  const double expansion = scaled ? 0.0 : 0.51e-6 * (double)(N * K), panels = bf16_path_us(M, N, K, 4.0) - expansion;
  const double margin = K % kStreamBlockK != 0 ? 0.75 : M > 1024 ? 0.82 : K < 2048 ? 0.85 : K <= 4096 ? 0.88 : 0.92;
  return here <= margin * cold * panels && (scaled ? M <= 768 || here <= 0.93 * panels : here <= bf16_prepared_us(M, N, K));
}

// Symmetric power-of-two scales of 32-groups, more than 64 rows: whether the FP4 kernel is the fastest of the three that
// could take them. Besides the output it takes 11 us + 5 ns K, from K 2048 on 12.8 + 4.2 ns K, while its 256 x 256 tiles
// fit the compute units once (512 x 11008 x 1024 20 us, 1024 x 4096 x 2048 23, x 4096 31.6, output included); this kernel
// 3 us and per round of 256 workgroups 1.25 us + 1.1 ns K, or 1.7 ns K if that is more (512 x 4096 x 4096, two rounds,
// 19; 1024 x 4096 x 2048, four, 20; 2048 x 4096 x 128, eight, 20, the FP4 kernel 12.6). Up to 16384 rows; beyond, the FP4
// kernel (32768 x 128 x 128 10.3 against 12.2, 100000 x 512 x 128 47 against 104). The few-rows kernel never is the
// fastest there (28672 x 8192: 80 rows 69 us, 256 rows 137, the FP4 kernel 66-69).
bool fp4_beats_stream(int64_t M, int64_t N, int64_t K, double c_bytes) {
  if (M <= 64) return false;
  const double k = (double)K, c = c_bytes * (double)M * (double)N, rounds = (double)(((M + 63) / 64 * ((N + 63) / 64) + 255) / 256);
  const double fp4 = (K < 2048 ? 11.0 + 0.005 * k : 12.8 + 0.0042 * k) + c / 6.5e6;
  const double short_k = 1.25 + 0.00107 * k, long_k = 0.00171 * k;
  return M > 16384 || fp4 <= 3.0 + rounds * (short_k > long_k ? short_k : long_k) + c / 5.1e6;
}

// Up to 64 rows against K so long that the few-rows kernel, which cuts K into slices for workgroups of their own, is the
// faster one: here a workgroup's eight waves share all of K, a block of 256 each in turn (the more rows, the longer), and
// few columns are few workgroups. AMXFP4-E5M2, us here / there: 32 x 1024 x 28672 27 / 22, x 16384 16.6 / 17.5; 32 x 4096
// x 28672 27.4 / 25.2; 64 x 128 x 24576 29.5 / 26.2, 64 x 8192 x 28672 59.6 / 53.9, x 20480 the same; 1 x 512 x 40960 25
// / 23, x 28672 19 / 21; 32 x 32 x 16384 16.4 / 14.1. Symmetric scales, whose dequantization is half the work: 32 x 512 x
// 65536 1.25 times, x 40960 1.08 and 17 rows of it 0.85.
static bool long_k_few_rows(int scale_kind, bool asym, int64_t M, int64_t N, int64_t K) {
  if (N <= 64) K += K * 3 / 10;  // one or two workgroups: the lines lie lower
  if (!asym) return M > 16 && (M <= 32 ? K > 49152 && N <= 2048 : K > 57344 && N <= 64);
  const bool e4m3 = scale_kind == kScaleE4M3;  // (its few-rows kernel dequantizes through FP32: slower)
  if (M <= 16) return K > (e4m3 ? 49152 : 32768) && N <= 2048;
  if (M <= 32) return K > 24576 && !e4m3 ? N <= 4096 : K > (e4m3 ? 20480 : 16384) && N <= 2048;
  if (e4m3) return K > 32768 && N <= 8192;
  return K > 20480 ? N <= 8192 : K > 16384 && N <= 512;
}

// A batch of more than 32 rows each and more than two rounds of workgroups: the few-rows kernel, which dequantizes A
// once, where its 256 columns per workgroup are filled, and where K is a single block, which one wave here takes alone
// (us here / there: 32 x 64 x 4096 x 1024 38.4 / 34.5;  512 x 64 x 512 x 256 51 / 33;  but 32 x 64 x 2048 x 1024 21 / 23,
// 512 x 64 x 128 x 4096 66 / 170), or with very many workgroups two blocks (64 x 48 x 2048 x 512 29.6 / 24.3, symmetric 24.2
// / 22.6;  but 24 x 48 x 2048 x 512 14.5 / 14.7, symmetric 11.9 / 13.8).
static bool batch_few_rows(int64_t M, int64_t N, int64_t K, int64_t batch) {
  const int64_t groups = batch * ((N + 63) / 64);
  return M > 32 && groups > 512 && (N >= 4096 || (N >= 512 && K <= (groups >= 2048 ? 2 : 1) * kStreamBlockK));
}

// Whether this kernel takes a product. scaled: with tensor-wise scales (then the panels are the only other kernel). us for
// the whole call, AMXFP4-E5M2, here / the kernel that took it otherwise:
//   up to 64 rows, except for a long K and for some batches (above): 1 x 4096 x 4096 4.8 / 12.7;  64 x 1024 x 1024 4.0 / 11.2;
//     32 x 11008 x 4096 12.5 / 16.9;  32 x 28672 x 8192 41 / 47;  64 x 28672 x 8192 56 / 60;  groups of 16, whose weights were
//     expanded to BF16 first, 24 x 11008 x 4096 10 / 84;
//   single problems from there on, symmetric power-of-two scales: where the estimates above say so
//   the other formats up to 256 rows, against weights below 2^27 elements: where the estimates of this and of the few-rows
//     kernel, which shares the dequantized A, say so (256 x 4096 x 4096 17 / 50;  256 x 11008 x 4096 40 / 79;  but 96 x 10240
//     x 8192 45 / 35;  256 x 5120 x 13824 74 / 70;  256 x 32001 x 4096 99 / 83), always with symmetric scales, from 128 rows
//     on whatever the weights (256 x 32001 x 4096 73 / 78;  256 x 8192 x 28672 114 / 142, 160 x 28672 x 8192 102 / 110;  but
//     90 x 8960 x 28672 94 / 72). Asymmetric power-of-two scales end here (prepared weights beyond 256 rows are their FP6
//     panel alone);
//   up to 512 rows, and to 768 rows with a long K or few columns: where the estimate is below that of the panels, B's
//     expansion included (512 x 4096 x 4096 27 / 42;  512 x 4096 x 11008 64 / 101;  448 x 11008 x 4096 61 / 64, but 512 rows
//     73 / 65;  448 x 4544 x 4544 43 / 48, but 512 rows 58 / 48;  with the same buffers again and again 640 x 8192 x 8192 113 /
//     109, 768 rows 138 / 113, 512 x 13824 x 5120 102 / 92, and on three sets of them in turn, whose weights come from memory,
//     115 / 148, 137 / 150, 103 / 127: the line lies between the two).
//     A product on prepared weights comes here with the plain one, whose bits it promises, although it would save the
//     expansion: that costs it 4 to 6 us at 384-512 x 6144 x 4096 and 320-448 x 4544 x 4544 (37-39 / 31-34 and 42-43 / 37-39, the
//     plain calls 37-39 / 42-45 and 42-43 / 47-48), and where several rounds are taken (384 x 11008 x 4096: 60 / 39-57, plain 60 /
//     58-62) more.
// c_bytes: of the output per element of M x N.
static bool stream_preferred(int scale_kind, bool asym, int64_t group_size, bool scaled, int64_t M, int64_t N, int64_t K,
                             int64_t batch, double c_bytes) {
  if ((group_size != 32 && group_size != 16) || K % 32 != 0) return false;
  const bool few_rows = group_size == 32 && !scaled && skinny_path_supported(M, N, K, batch);  // the kernel of that name
  if (!scaled && rounded_pot(scale_kind, group_size) && !few_rows) return false;
  if (M <= 64)
    return !few_rows || (batch > 1 ? !batch_few_rows(M, N, K, batch) : !long_k_few_rows(scale_kind, asym, M, N, K));
  if (batch != 1) return false;
  const bool pot = group_size == 32 && pot_scales(scale_kind);
  if (pot && !asym) return !fp4_path_supported(M, N, K) ? M <= 256 : !fp4_beats_stream(M, N, K, c_bytes);
  if (!pot && beats_panels(asym, group_size, scaled, M, N, K)) return true;
  if (N * K >= (int64_t(1) << 27) && (M > 256 || (group_size == 32 && (asym || M < 128)))) return false;
  if (M <= 256 && few_rows) return !asym || stream_us(asym, group_size, M, N, K, c_bytes) <= skinny_path_us(M, N, K);
  if (pot) return M <= 256;
  if (M > 768 || (M > 512 && K < 8192 && (M + 63) / 64 * ((N + 63) / 64) > 512)) return false;
  return stream_us(asym, group_size, M, N, K, c_bytes) <= bf16_path_us(M, N, K, c_bytes);
}

bool stream_path_preferred(int scale_kind, bool asym, int64_t group_size, bool scaled, int64_t M, int64_t N, int64_t K,
                           int64_t batch) {
  return stream_preferred(scale_kind, asym, group_size, scaled, M, N, K, batch, 4.0);
}

// The same for the gated product, B [2 width][K] = [N][K], whose output is BF16 and half as wide. Beyond 256 rows exactly where
// the plain product comes here: the two give the same bits. Up to 256 rows symmetric power-of-two scales by the same
// estimates, and otherwise the alternative is a tiled kernel, never the few-rows one, so large weights come here too
// (AMXFP4-E5M2, 28672 x 8192, 256 rows: 177 us against 350), and asymmetric power-of-two scales while this kernel's 4 us + (0.5
// + 2.8 per round) ns K is less than the FP6 kernel's merge of the weights and its one round of tiles, 20 us + 4.7 ns K + 0.37
// ps N K (256 x 22016 x 4096: 70 against 63, on prepared weights 48).
bool stream_glu_preferred(int scale_kind, bool asym, int64_t group_size, int64_t M, int64_t N, int64_t K) {
  if ((group_size != 32 && group_size != 16) || K % 32 != 0 || rounded_pot(scale_kind, group_size)) return false;
  if (M > 256) return stream_path_preferred(scale_kind, asym, group_size, false, M, N, K, 1);
  if (M <= 64) return true;
  const bool pot = group_size == 32 && pot_scales(scale_kind);
  if (pot && !asym) return stream_preferred(scale_kind, asym, group_size, false, M, N, K, 1, 1.0);
  const double k = (double)K, rounds = (double)(((M + 63) / 64 * ((N + 63) / 64) + 255) / 256);
  return !pot || 4.0 + k / 4096.0 * (2.0 + 11.5 * rounds) < 20.0 + 0.0047 * k + 3.7e-7 * (double)N * k;
}

hipError_t launch_gemm_stream(int scale_kind, bool asym, int64_t group_size, int64_t M, int64_t N, int64_t K,
                              const uint8_t* A_codes, const uint8_t* A_scales, const uint8_t* B_codes,
                              const uint8_t* B_scales, const float* A_tensor_pair, const float* B_tensor_pair, float* C,
                              int64_t ldc, int64_t batch, hipStream_t s, const KernelTimer& timer) {
  return stream_launch<false>(scale_kind, asym, group_size, M, N, K, A_codes, A_scales, B_codes, B_scales, A_tensor_pair,
                              B_tensor_pair, C, ldc, batch, s, timer);
}

}  // namespace amx
