// Fully quantized GEMM (Sec. 4.3) for at most 64 rows on the A side: one launch, both operands read as packed codes.
//
// What bounds such a product is reading the weights (B) once, or, for small weights, the chain of launches and memory
// latencies. So nothing is prepared in memory and nothing is shared between waves while they run: a wave owns NT column
// tiles of C and every WAVES-th block of 256 along K, streams its rows' codes and scales into registers one block ahead
// (buffer loads; no LDS, no barrier, no expansion pass), dequantizes both operands to exact 16-bit floats and
// multiplies them on the 16-bit MFMA. The waves of a workgroup share the columns and split K between them; their sums
// meet in LDS at the end, in a fixed order, so there are no partial tiles in memory and no reduction launch.
//
// MFMA shape R x R (R = 32: v_mfma_f32_32x32x16, R = 16: v_mfma_f32_16x16x32, for up to 16 rows: half the work on rows
// that do not exist). Of a block of 256 elements of its row, a lane owns the contiguous piece lane / R (R / 2 words of
// eight codes); k-step s multiplies word s of every lane. Both operands follow that order, so their sums match, and a
// sum over k does not care which order it is.
//
// Dequantization (dequant_regs.h), packed 16-bit arithmetic: FP8 scales as FP16 (E5M2: the scale byte is the upper byte
// of an FP16, values biased by 2^-3 per operand, taken out at the end; E4M3: the byte's bits are an FP16 times 2^-8, the
// elements are converted times 2^8, no bias left), power-of-two scales through the conversion's own scale operand to
// BF16. A value has at most 6 significant bits: exact in all of them.
//
// Groups of 32 and 16, any K the formats take (a last block shorter than 256 is read chunk by chunk), an optional factor
// alpha (the product of two tensor-wise scales).

#include "dequant_regs.h"
#include "device_formats.h"
#include "gemm_common.h"

namespace amx {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int kStreamBlockK = 256;  // 128 bytes of codes per row: one cache line
constexpr int64_t kStreamMaxM = 64;

// One lane's share of one row of one K block: W words of codes and their scale bytes.
template <bool ASYM, int GS_LOG2, int R>
struct StreamPiece {
  static constexpr int kWords = R / 2;                           // 8 codes each
  static constexpr int kEntries = (kWords * 8) >> GS_LOG2;       // scale entries
  static constexpr int kScaleBytes = kEntries * (ASYM ? 2 : 1);  // 2, 4, 8 or 16
  static constexpr int kWordsPerEntry = kWords / kEntries;
  u32x4 w[kWords / 4];
  uint32_t s[kScaleBytes < 4 ? 1 : kScaleBytes / 4];
};

// Entry e's scale pair in the form the dequantization takes (see dequant_regs.h).
template <int SCALE_KIND, bool ASYM>
__device__ __forceinline__ void stream_scales(const uint32_t* s, int e, uint32_t& s_pos, uint32_t& s_neg) {
  const int bp = ASYM ? 2 * e : e;
  const uint32_t reg = s[bp >> 2];
  const uint32_t b0 = bp & 3, b1 = b0 + 1;
  if constexpr (SCALE_KIND == kScaleE8M0Floor) {
    s_pos = ((reg >> (8 * b0)) & 255u) << 23;
    s_neg = ASYM ? ((reg >> (8 * b1)) & 255u) << 23 : s_pos;
  } else {
    // byte -> (byte << 8) in both halves; the cast never sets a scale's sign bit and it is ignored
    s_pos = __builtin_amdgcn_perm(0u, reg, (b0 << 24) | (0x0Cu << 16) | (b0 << 8) | 0x0Cu);
    s_neg = ASYM ? __builtin_amdgcn_perm(0u, reg, (b1 << 24) | (0x0Cu << 16) | (b1 << 8) | 0x0Cu) : s_pos;
    if constexpr (SCALE_KIND == kScaleE5M2) {
      s_pos &= 0x7F007F00u, s_neg &= 0x7F007F00u;
    } else {  // 0eeeemmm << 7 is an FP16: 2^-8 times the scale
      s_pos = (s_pos >> 1) & 0x3F803F80u, s_neg = (s_neg >> 1) & 0x3F803F80u;
    }
  }
}

template <int SCALE_KIND, bool ASYM>
__device__ __forceinline__ u32x4 stream_dequant(uint32_t word, uint32_t s_pos, uint32_t s_neg) {
  if constexpr (SCALE_KIND == kScaleE4M3)
    return u32x4{dequant2_f16<ASYM, 0>(word, s_pos, s_neg, 256.0f), dequant2_f16<ASYM, 1>(word, s_pos, s_neg, 256.0f),
                 dequant2_f16<ASYM, 2>(word, s_pos, s_neg, 256.0f), dequant2_f16<ASYM, 3>(word, s_pos, s_neg, 256.0f)};
  else
    return dequant_word<SCALE_KIND, ASYM>(word, s_pos, s_neg);
}

// grid: (ceil(N / (NT R)), 1, batch); block: WAVES waves. M <= MT R. WHOLE: K is a multiple of 256 (so every row's scale
// bytes start on a multiple of four, as their vector loads need); otherwise scale entries are loaded byte by byte.
template <int SCALE_KIND, bool ASYM, int GS_LOG2, int R, int MT, int NT, int WAVES, bool WHOLE>
__global__ __launch_bounds__(64 * WAVES) void gemm_stream_kernel(
    const uint8_t* A_codes, const uint8_t* A_scales, const uint8_t* B_codes, const uint8_t* B_scales, float* C,
    int M, int64_t N, int64_t K, int64_t ldc, const float* alpha_a, const float* alpha_b) {
  using Piece = StreamPiece<ASYM, GS_LOG2, R>;
  constexpr int kAcc = R * R / 64;  // accumulator registers per tile: 16 or 4
  constexpr bool kF16 = SCALE_KIND == kScaleE5M2 || SCALE_KIND == kScaleE4M3;
  typedef float acc_t __attribute__((ext_vector_type(kAcc)));
  __shared__ float sums[WAVES * MT * NT * kAcc * 64];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r = lane % R, piece = lane / R;
  const int64_t b = blockIdx.z, n0 = (int64_t)blockIdx.x * (NT * R);
  const int rows_b = N - n0 < NT * R ? (int)(N - n0) : NT * R;
  const int row_codes = (int)(K >> 1), row_scales = (int)((K >> GS_LOG2) * (ASYM ? 2 : 1));

  // Raw buffers over this workgroup's rows of either operand: rows past the end read as zero (codes 0: value 0).
  auto buffer = [](const uint8_t* p, int bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(p), 0, bytes, 0x00020000);
  };
  const uint8_t* ac = A_codes + b * M * row_codes;
  const uint8_t* as = A_scales + b * M * row_scales;
  const uint8_t* bc = B_codes + (b * N + n0) * row_codes;
  const uint8_t* bs = B_scales + (b * N + n0) * row_scales;

  constexpr int kNowhere = INT32_MIN;                // an offset past the end of any of these buffers
  int oc[MT > NT ? MT : NT], os[MT > NT ? MT : NT];  // byte offsets of the lane's piece of block 0 in row t R + r
#pragma unroll
  for (int t = 0; t < (MT > NT ? MT : NT); ++t) {
    oc[t] = (t * R + r) * row_codes + piece * (Piece::kWords * 4);
    os[t] = (t * R + r) * row_scales + piece * Piece::kScaleBytes;
  }

  acc_t acc[MT][NT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int v = 0; v < kAcc; ++v) acc[i][j][v] = 0.f;

  // the scale entries of the lane's piece, byte by byte; entries of elements from `left` on read as zero
  auto load_scale_bytes = [&](Piece& p, __amdgpu_buffer_rsrc_t rs, int t, int so, int left) {
    const int k0 = piece * (Piece::kWords * 8);
#pragma unroll
    for (int i = 0; i < (Piece::kScaleBytes < 4 ? 1 : Piece::kScaleBytes / 4); ++i) p.s[i] = 0;
#pragma unroll
    for (int i = 0; i < Piece::kScaleBytes; ++i) {
      const int e = ASYM ? i >> 1 : i;
      const uint32_t v = (uint8_t)__builtin_amdgcn_raw_buffer_load_b8(rs, k0 + (e << GS_LOG2) < left ? os[t] : kNowhere, so + i, 0);
      p.s[i >> 2] |= v << (8 * (i & 3));
    }
  };
  // block `blk` of row tile t; `on` false (uniform): the buffer is empty, every load returns zero without a request
  auto load_tile = [&](Piece& p, const uint8_t* codes, const uint8_t* scales, int rows, int t, int blk, bool on) {
    const __amdgpu_buffer_rsrc_t rc = buffer(codes, on ? rows * row_codes : 0), rs = buffer(scales, on ? rows * row_scales : 0);
#pragma unroll
    for (int c = 0; c < Piece::kWords / 4; ++c)
      p.w[c] = __builtin_amdgcn_raw_buffer_load_b128(rc, oc[t], blk * (kStreamBlockK / 2) + c * 16, 0);
    const int so = blk * ((kStreamBlockK >> GS_LOG2) * (ASYM ? 2 : 1));
    if constexpr (!WHOLE) {
      load_scale_bytes(p, rs, t, so, kStreamBlockK);
    } else if constexpr (Piece::kScaleBytes == 16) {
      const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rs, os[t], so, 0);
      p.s[0] = v[0], p.s[1] = v[1], p.s[2] = v[2], p.s[3] = v[3];
    } else if constexpr (Piece::kScaleBytes == 8) {
      const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(rs, os[t], so, 0);
      p.s[0] = v[0], p.s[1] = v[1];
    } else if constexpr (Piece::kScaleBytes == 4) {
      p.s[0] = __builtin_amdgcn_raw_buffer_load_b32(rs, os[t], so, 0);
    } else {
      p.s[0] = __builtin_amdgcn_raw_buffer_load_b16(rs, os[t], so, 0);
    }
  };
  // the last, shorter block: chunks of 32 elements past K read as zero
  auto load_tail = [&](Piece& p, const uint8_t* codes, const uint8_t* scales, int rows, int t, int blk, int left) {
    const __amdgpu_buffer_rsrc_t rc = buffer(codes, rows * row_codes), rs = buffer(scales, rows * row_scales);
#pragma unroll
    for (int c = 0; c < Piece::kWords / 4; ++c)
      p.w[c] = __builtin_amdgcn_raw_buffer_load_b128(rc, piece * (Piece::kWords * 8) + 32 * c < left ? oc[t] : kNowhere,
                                                     blk * (kStreamBlockK / 2) + c * 16, 0);
    load_scale_bytes(p, rs, t, blk * ((kStreamBlockK >> GS_LOG2) * (ASYM ? 2 : 1)), left);
  };

  auto multiply = [&](const Piece (&pa)[MT], const Piece (&pb)[NT]) {
#pragma unroll
    for (int e = 0; e < Piece::kEntries; ++e) {
      uint32_t ap[MT], an[MT], bp[NT], bn[NT];
#pragma unroll
      for (int i = 0; i < MT; ++i) stream_scales<SCALE_KIND, ASYM>(pa[i].s, e, ap[i], an[i]);
#pragma unroll
      for (int j = 0; j < NT; ++j) stream_scales<SCALE_KIND, ASYM>(pb[j].s, e, bp[j], bn[j]);
#pragma unroll
      for (int x = 0; x < Piece::kWordsPerEntry; ++x) {
        const int s = e * Piece::kWordsPerEntry + x;
        u32x4 av[MT];
#pragma unroll
        for (int i = 0; i < MT; ++i) av[i] = stream_dequant<SCALE_KIND, ASYM>(pa[i].w[s >> 2][s & 3], ap[i], an[i]);
#pragma unroll
        for (int j = 0; j < NT; ++j) {
          const u32x4 bv = stream_dequant<SCALE_KIND, ASYM>(pb[j].w[s >> 2][s & 3], bp[j], bn[j]);
#pragma unroll
          for (int i = 0; i < MT; ++i) {
            if constexpr (R == 32 && kF16)
              acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, av[i]), __builtin_bit_cast(f16x8, bv),
                                                                 acc[i][j], 0, 0, 0);
            else if constexpr (R == 32)
              acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, av[i]), __builtin_bit_cast(bf16x8, bv),
                                                                  acc[i][j], 0, 0, 0);
            else if constexpr (kF16)
              acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, av[i]), __builtin_bit_cast(f16x8, bv),
                                                                 acc[i][j], 0, 0, 0);
            else
              acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, av[i]), __builtin_bit_cast(bf16x8, bv),
                                                                  acc[i][j], 0, 0, 0);
          }
        }
      }
    }
  };

  // This wave's full blocks are wave, wave + WAVES, ..: nb of them. Two register sets; a set is refilled as soon as it
  // has been multiplied, two blocks ahead, so a block's loads travel while another one is multiplied. Loads past the
  // last block go to an empty buffer instead of being skipped: the number of loads in flight is then the same on every
  // path, and waiting for one set never means waiting for the other.
  const int full = (int)(K / kStreamBlockK);
  [[maybe_unused]] const int left = (int)(K % kStreamBlockK);
  const int nb = full > wave ? (full - wave + WAVES - 1) / WAVES : 0;
  auto load = [&](Piece (&pa)[MT], Piece (&pb)[NT], int i) {
    const bool on = i < nb;
    const int blk = wave + i * WAVES;
#pragma unroll
    for (int j = 0; j < NT; ++j) load_tile(pb[j], bc, bs, rows_b, j, blk, on);
#pragma unroll
    for (int t = 0; t < MT; ++t) load_tile(pa[t], ac, as, M, t, blk, on);
  };
  if (nb > 0) {
    Piece a0[MT], b0[NT], a1[MT], b1[NT];
    load(a0, b0, 0);
    load(a1, b1, 1);
    for (int i = 0;; i += 2) {
      multiply(a0, b0);
      if (i + 1 >= nb) break;
      load(a0, b0, i + 2);
      multiply(a1, b1);
      if (i + 2 >= nb) break;
      load(a1, b1, i + 3);
    }
  }
  if constexpr (!WHOLE) {
    if (left != 0 && wave == full % WAVES) {
      Piece a0[MT], b0[NT];
#pragma unroll
      for (int j = 0; j < NT; ++j) load_tail(b0[j], bc, bs, rows_b, j, full, left);
#pragma unroll
      for (int t = 0; t < MT; ++t) load_tail(a0[t], ac, as, M, t, full, left);
      multiply(a0, b0);
    }
  }

  // the waves' sums, added in ascending wave order
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int v = 0; v < kAcc; ++v) sums[(((wave * MT + i) * NT + j) * kAcc + v) * 64 + lane] = acc[i][j][v];
  __syncthreads();
  const float alpha = alpha_a ? alpha_a[0] * alpha_b[0] : 1.0f;
  constexpr int kTile = MT * NT * kAcc * 64;
  float* Cb = C + b * M * ldc + n0;
#pragma unroll
  for (int e = 0; e < (kTile + 64 * WAVES - 1) / (64 * WAVES); ++e) {
    const int idx = e * 64 * WAVES + (int)threadIdx.x;
    if (kTile % (64 * WAVES) == 0 || idx < kTile) {
      float s = sums[idx];
#pragma unroll
      for (int w = 1; w < WAVES; ++w) s += sums[w * kTile + idx];
      // register v of lane l: 32 x 32 tiles: row 8 (v / 4) + 4 (l / 32) + v % 4; 16 x 16: row 4 (l / 16) + v
      const int l = idx & 63, v = (idx >> 6) % kAcc, j = (idx / (64 * kAcc)) % NT, i = idx / (64 * kAcc * NT);
      const int row = i * R + (R == 32 ? 8 * (v >> 2) + 4 * (l >> 5) + (v & 3) : 4 * (l >> 4) + v);
      const int col = j * R + l % R;
      if constexpr (SCALE_KIND == kScaleE5M2) s *= 64.0f;  // undo the two biases
      if (alpha_a) s *= alpha;
      if (row < M && col < rows_b) Cb[row * ldc + col] = s;
    }
  }
}

bool stream_path_supported(int64_t group_size, int64_t M, int64_t K) {
  return (group_size == 32 || group_size == 16) && M >= 1 && M <= kStreamMaxM && K % 32 == 0;
}

// Where the few-rows kernel of gemm_skinny.hip, which shares A through LDS and can cut K over workgroups, takes the same
// operands (groups of 32, K a multiple of 256), it stays the faster one in two corners; us for the whole call, here / there:
//   more than 16 rows, a long K and few columns, where K over the waves of one workgroup leaves each of them a long chain:
//     32 x 4096 x 14336: 20.6 / 18.9;  32 x 8192 x 28672: 50 / 47;  64 x 4096 x 14336: 35 / 25;  (16 rows: 12.8 / 18.5)
//   more than 32 rows against large weights, where dequantizing A in every wave is what counts:
//     64 x 10240 x 8192: 34 / 30;  48 x 28672 x 8192: 69 / 57;  (64 x 8192 x 8192: 20.9 / 24.6;  40 x 14336 x 4096: 20 / 23)
// Elsewhere this kernel: 1 x 4096 x 4096: 4.8 / 12.7;  64 x 1024 x 1024: 5.8 / 11.2;  32 x 11008 x 4096: 12.8 / 16.9;
// 16 x 28672 x 8192: 39 / 46. The other formats would expand B to BF16 first (24 x 11008 x 4096 in groups of 16: 84 us).
bool stream_path_preferred(int64_t group_size, int64_t M, int64_t N, int64_t K) {
  if (!stream_path_supported(group_size, M, K)) return false;
  if (group_size != 32 || K % kStreamBlockK != 0 || M <= 16) return true;
  if (K >= 12288 && N <= 8192) return false;
  return M <= 32 ? N * K < (int64_t(1) << 27) : N * K <= (int64_t(1) << 26);
}

hipError_t launch_gemm_stream(int scale_kind, bool asym, int64_t group_size, int64_t M, int64_t N, int64_t K,
                              const uint8_t* A_codes, const uint8_t* A_scales, const uint8_t* B_codes,
                              const uint8_t* B_scales, const float* A_tensor_pair, const float* B_tensor_pair, float* C,
                              int64_t ldc, int64_t batch, hipStream_t s, const KernelTimer& timer) {
  if (!stream_path_supported(group_size, M, K)) return hipErrorInvalidValue;
  hipError_t e = hipSuccess;
  if (timer.start && (e = hipEventRecord(timer.start, s)) != hipSuccess) return e;
  auto run = [&]<int SK, bool ASYM, int GSL, int R, int MT, int NT, int WAVES, bool WHOLE>() {
    hipLaunchKernelGGL((gemm_stream_kernel<SK, ASYM, GSL, R, MT, NT, WAVES, WHOLE>),
                       dim3((unsigned)((N + NT * R - 1) / (NT * R)), 1, (unsigned)batch), dim3(64 * WAVES), 0, s, A_codes,
                       A_scales, B_codes, B_scales, C, (int)M, N, K, ldc, A_tensor_pair, B_tensor_pair);
    return hipGetLastError();
  };
  // Columns per workgroup: as few as still give the 256 compute units one workgroup of eight waves each; beyond 1024
  // tiles wider ones of four waves, several to a compute unit. (us by columns, AMXFP4-E5M2 16 rows: N 8192, K 8192:
  // 16 columns 14.9, 32: 12.1, 64: 17.9;  N 6144, K 4096: 8.4, 7.5, 11.5;  N 4096: 5.4, 7.3, 11.4;  N 28672, K 8192: 64
  // columns in eight waves 42.7, in four 39.0. 32 rows: N 14336, K 4096: 32 columns 14.8, 64: 13.4;  N 6144: 9.5, 12.8;
  // N 4096: two tiles of 16 rows and 16 columns 7.4, one of 32 rows and columns 9.3.)
  const int64_t t16 = (N + 15) / 16 * batch, t32 = (N + 31) / 32 * batch;
  auto shape = [&]<int SK, bool ASYM, int GSL>() {
    if (K % kStreamBlockK != 0) {
      if (M <= 16) return run.template operator()<SK, ASYM, GSL, 16, 1, 2, 8, false>();
      if (M <= 32) return run.template operator()<SK, ASYM, GSL, 32, 1, 1, 8, false>();
      return run.template operator()<SK, ASYM, GSL, 32, 2, 1, 8, false>();
    }
    if (M <= 16) {
      if (t16 <= 256) return run.template operator()<SK, ASYM, GSL, 16, 1, 1, 8, true>();
      if (t16 <= 512) return run.template operator()<SK, ASYM, GSL, 16, 1, 2, 8, true>();
      if (t16 <= 1024) return run.template operator()<SK, ASYM, GSL, 16, 1, 4, 8, true>();
      return run.template operator()<SK, ASYM, GSL, 16, 1, 4, 4, true>();
    }
    if (M <= 32) {
      if (t32 <= 128) return run.template operator()<SK, ASYM, GSL, 16, 2, 1, 8, true>();
      if (t32 <= 256) return run.template operator()<SK, ASYM, GSL, 32, 1, 1, 8, true>();
      if (t32 <= 512) return run.template operator()<SK, ASYM, GSL, 32, 1, 2, 8, true>();
      return run.template operator()<SK, ASYM, GSL, 32, 1, 2, 4, true>();
    }
    if (t32 <= 256) return run.template operator()<SK, ASYM, GSL, 32, 2, 1, 8, true>();
    return run.template operator()<SK, ASYM, GSL, 32, 2, 2, 4, true>();
  };
  auto group = [&]<int SK, bool ASYM>() {
    return group_size == 16 ? shape.template operator()<SK, ASYM, 4>() : shape.template operator()<SK, ASYM, 5>();
  };
  // E8M0 floor and round share the byte encoding
  if (scale_kind == kScaleE5M2)
    e = asym ? group.template operator()<kScaleE5M2, true>() : group.template operator()<kScaleE5M2, false>();
  else if (scale_kind == kScaleE4M3)
    e = asym ? group.template operator()<kScaleE4M3, true>() : group.template operator()<kScaleE4M3, false>();
  else
    e = asym ? group.template operator()<kScaleE8M0Floor, true>() : group.template operator()<kScaleE8M0Floor, false>();
  if (e != hipSuccess) return e;
  if (timer.stop) e = hipEventRecord(timer.stop, s);
  return e;
}

}  // namespace amx
