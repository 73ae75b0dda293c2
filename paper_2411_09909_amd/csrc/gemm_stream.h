// Kernel and launch rule of the fully quantized GEMM (Sec. 4.3) for few rows on the A side and for small problems: one
// launch, both operands read as packed codes.
//
// What bounds a product with few rows is reading the weights (B) once, or, for small weights, the chain of launches and
// memory latencies. So nothing is prepared in memory and nothing is shared between waves while they run: a wave owns MT x
// NT tiles of C and every WAVES-th block of 256 along K, dequantizes both operands to exact 16-bit floats in registers and
// multiplies them on the 16-bit MFMA. The waves of a workgroup share the tiles and split K between them; their sums meet in
// LDS at the end, in a fixed order, so there are no barriers while K is walked, no partial tiles in memory and no reduction
// launch. With more rows the vector arithmetic of the dequantization is the bound (MT + NT dequantized fragments of 16 + 3
// instructions for MT NT MFMAs), until, from about 512 rows on, expanding the weights once pays.
//
// Access: a vector cache has a limited number of line requests in flight, so a block's codes are fetched in whole cache
// lines, 8 lanes to the 128 bytes of a row, straight into LDS of the wave's own, and read back from there in the MFMA's
// row-per-lane order. (Loading the fragments' 16-byte pieces straight into registers asks for every line four to eight
// times: 16 x 28672 x 8192 39 us, 512 x 4096 x 4096 40 us; as it is 35 us = 3.8 TB/s and 28 us.)
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
// Groups of 32 and 16, any K the formats take (chunks of 32 past K in the last block read as zero), an optional factor
// alpha (the product of two tensor-wise scales).

#pragma once
#include "dequant_regs.h"
#include "device_formats.h"
#include "gemm_common.h"

namespace amx {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int kStreamBlockK = 256;  // 128 bytes of codes per row: one cache line

// One lane's share of one row of one K block: W words of codes and their scale bytes.
template <bool ASYM, int GS_LOG2, int R>
struct StreamPiece {
  static constexpr int kWords = R / 2;                           // 8 codes each
  static constexpr int kEntries = (kWords * 8) >> GS_LOG2;       // scale entries
  static constexpr int kScaleBytes = kEntries * (ASYM ? 2 : 1);  // 2, 4, 8 or 16
  static constexpr int kScaleWords = kScaleBytes < 4 ? 1 : kScaleBytes / 4;
  static constexpr int kWordsPerEntry = kWords / kEntries;
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

// grid: (ceil(N / (NT R)), ceil(M / (MT R)), batch); block: WAVES waves. WHOLE: K is a multiple of 256 (so every row's scale
// bytes start on a multiple of four, as their vector loads need); otherwise scale entries are loaded byte by byte.
// FEW (R = 16, one row tile; 0: not): at most so many rows of A. A lane's share of a fragment is then a padding row's in most lanes, so
// the wave's lanes share out the rows there are instead (a word of eight codes each, FEW / 2 times), dequantize them into LDS and read
// the fragments from there, every lane row l % FEW; the rows of C beyond are not stored. Of a block's 272 vector instructions (16 x 16
// tiles, asymmetric FP8-E5M2) 136 + 36 are left. Us, one row, all lanes on their own fragments / shared out: 4096 x 14336 10.5 / 8.5,
// 4096 x 11008 8.9 / 7.4, 11008 x 4096 8.9 / 8.2, 28672 x 8192 33.8 / 31.5, 8192 x 28672 31.5 / 27.1; symmetric 4096 x 14336 7.3 / 6.8;
// NVFP4 4544 x 4544 7.6 / 6.9. (As well for eight rows: 4 % of 5 to 8 rows' time, and beyond three column tiles one workgroup instead of two
// to a compute unit. Rows 16 bytes apart instead of swizzled: the same, 28672 x 8192 5 % slower.)
// GLU: B's rows are the gate and up rows interleaved in blocks of 32; C is then the BF16 output [M][ldc] of N / 2 columns,
// bf16(silu(gate) * up). Its sums are the plain product's in the same order wherever both come here in the same shape, which
// is everywhere but at 17 to 32 rows with N <= 4096 or 48 columns to a workgroup (there the plain form has R = 16, the gated
// one always R = 32).
template <int SCALE_KIND, bool ASYM, int GS_LOG2, int R, int MT, int NT, int WAVES, int FEW, bool WHOLE, bool GLU>
__global__ __launch_bounds__(64 * WAVES) void gemm_stream_kernel(
    const uint8_t* A_codes, const uint8_t* A_scales, const uint8_t* B_codes, const uint8_t* B_scales, float* C,
    int64_t M, int64_t N, int64_t K, int64_t ldc, const float* alpha_a, const float* alpha_b) {
  using Piece = StreamPiece<ASYM, GS_LOG2, R>;
  constexpr int kAcc = R * R / 64;  // accumulator registers per tile: 16 or 4
  constexpr int kTiles = MT + NT;   // row tiles of A, then column tiles (rows of B)
  constexpr bool kF16 = SCALE_KIND == kScaleE5M2 || SCALE_KIND == kScaleE4M3;
  static_assert(FEW == 0 || (R == 16 && MT == 1 && FEW == 4));
  constexpr int kCodeTiles = FEW ? NT : kTiles;  // tiles whose codes go through LDS as they are
  // A row of A dequantized: 32 chunks of eight elements. Chunk c of row q lies in slot c ^ ((q & 3) + 4 (c / 16)), so that the reads of
  // a k-step, chunk 8 piece + s of four rows, fall on banks of their own.
  constexpr int kFewRowBytes = 2 * kStreamBlockK;
  constexpr int kRowBytes = kStreamBlockK / 2, kFewBytes = FEW * kFewRowBytes;
  constexpr int kWaveBytes = kCodeTiles * R * kRowBytes + kFewBytes;  // one block of a wave's codes, its rows of A
  constexpr int kSumBytes = WAVES * MT * NT * kAcc * 64 * 4;
  typedef float acc_t __attribute__((ext_vector_type(kAcc)));
  // the waves' blocks of codes; their sums at the end
  __shared__ __attribute__((aligned(1024))) uint8_t lds[WAVES * kWaveBytes > kSumBytes ? WAVES * kWaveBytes : kSumBytes];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r = lane % R, piece = lane / R;
  const int64_t b = blockIdx.z, n0 = (int64_t)blockIdx.x * (NT * R), m0 = (int64_t)blockIdx.y * (MT * R);
  const int rows_a = M - m0 < MT * R ? (int)(M - m0) : MT * R;
  const int rows_b = N - n0 < NT * R ? (int)(N - n0) : NT * R;
  const int row_codes = (int)(K >> 1), row_scales = (int)((K >> GS_LOG2) * (ASYM ? 2 : 1));

  // Raw buffers over this workgroup's rows of either operand: rows past the end read as zero (codes 0: value 0).
  auto buffer = [](const uint8_t* p, int bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(p), 0, bytes, 0x00020000);
  };
  const __amdgpu_buffer_rsrc_t ac = buffer(A_codes + (b * M + m0) * row_codes, rows_a * row_codes);
  const __amdgpu_buffer_rsrc_t as = buffer(A_scales + (b * M + m0) * row_scales, rows_a * row_scales);
  const __amdgpu_buffer_rsrc_t bc = buffer(B_codes + (b * N + n0) * row_codes, rows_b * row_codes);
  const __amdgpu_buffer_rsrc_t bs = buffer(B_scales + (b * N + n0) * row_scales, rows_b * row_scales);
  constexpr int kNowhere = INT32_MIN;  // an offset past the end of any of these buffers

  // A direct-to-LDS load brings 8 rows x 128 bytes, whole cache lines: lane l fetches for row l / 8 the 16-byte chunk
  // whose slot in LDS is l % 8. Chunk c of row q lies in slot c ^ ((q >> 1) & 7), so that the 64 lanes of a fragment read
  // (16 bytes from each of R rows) spread over all banks.
  const int chunk_even = (lane & 7) ^ (lane >> 4);  // of rows 16 i .. 16 i + 7; rows 16 i + 8 ..: ^ 4
  const int gather = (lane >> 3) * row_codes;
  uint8_t* const mine = lds + wave * kWaveBytes;
  int read_off[Piece::kWords / 4];
#pragma unroll
  for (int c = 0; c < Piece::kWords / 4; ++c)
    read_off[c] = r * kRowBytes + (((piece * (Piece::kWords / 4) + c) ^ ((r >> 1) & 7)) << 4);
  const int scale_off = r * row_scales + piece * Piece::kScaleBytes;

  acc_t acc[MT][NT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int v = 0; v < kAcc; ++v) acc[i][j][v] = 0.f;

  uint32_t s_next[kTiles][Piece::kScaleWords];  // scale bytes of the block whose codes are on their way
  uint8_t* const few_lds = mine + kCodeTiles * R * kRowBytes;
  uint32_t few_word[FEW ? FEW / 2 : 1], few_scales[FEW ? FEW / 2 : 1];  // word lane % 32 of rows lane / 32, lane / 32 + 2, ..
  // Requests block `blk` of all tiles: codes to LDS, scale bytes to s_next. left: elements of the block that exist (256
  // but for a last, shorter block, whose chunks of 32 elements past K read as zero).
  auto request = [&](int blk, [[maybe_unused]] int left) {
    if constexpr (FEW != 0) {
      const int word = lane & 31, row = lane >> 5;
      const bool there = WHOLE || word * 8 < left;
      const int code_off = there ? row * row_codes + word * 4 : kNowhere;
      const int scale_at = there ? row * row_scales + ((word * 8) >> GS_LOG2) * (ASYM ? 2 : 1) : kNowhere;
#pragma unroll
      for (int i = 0; i < FEW / 2; ++i) {
        few_word[i] = __builtin_amdgcn_raw_buffer_load_b32(ac, code_off, 2 * i * row_codes + blk * kRowBytes, 0);
        const int so = 2 * i * row_scales + blk * ((kStreamBlockK >> GS_LOG2) * (ASYM ? 2 : 1));
        if constexpr (ASYM)
          few_scales[i] = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(as, scale_at, so, 0);
        else
          few_scales[i] = (uint8_t)__builtin_amdgcn_raw_buffer_load_b8(as, scale_at, so, 0);
      }
    }
#pragma unroll
    for (int t = FEW ? MT : 0; t < kTiles; ++t) {
      const bool is_a = t < MT;
      const int row0 = (is_a ? t : t - MT) * R;
#pragma unroll
      for (int l = 0; l < R / 8; ++l) {
        const int chunk = (l & 1) ? chunk_even ^ 4 : chunk_even;
        int off = gather + chunk * 16;
        if constexpr (!WHOLE) off = chunk * 32 < left ? off : kNowhere;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(is_a ? ac : bc, (lds_ptr_t)(mine + ((FEW ? t - MT : t) * R + 8 * l) * kRowBytes), 16, off,
                                                 (row0 + 8 * l) * row_codes + blk * kRowBytes, 0, 0);
      }
      const int so = row0 * row_scales + blk * ((kStreamBlockK >> GS_LOG2) * (ASYM ? 2 : 1));
      if constexpr (!WHOLE) {
#pragma unroll
        for (int i = 0; i < Piece::kScaleWords; ++i) s_next[t][i] = 0;
#pragma unroll
        for (int i = 0; i < Piece::kScaleBytes; ++i) {
          const int k = piece * (Piece::kWords * 8) + ((ASYM ? i >> 1 : i) << GS_LOG2);
          const uint32_t v = (uint8_t)__builtin_amdgcn_raw_buffer_load_b8(is_a ? as : bs, k < left ? scale_off : kNowhere, so + i, 0);
          s_next[t][i >> 2] |= v << (8 * (i & 3));
        }
      } else if constexpr (Piece::kScaleBytes == 16) {
        const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(is_a ? as : bs, scale_off, so, 0);
        s_next[t][0] = v[0], s_next[t][1] = v[1], s_next[t][2] = v[2], s_next[t][3] = v[3];
      } else if constexpr (Piece::kScaleBytes == 8) {
        const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(is_a ? as : bs, scale_off, so, 0);
        s_next[t][0] = v[0], s_next[t][1] = v[1];
      } else if constexpr (Piece::kScaleBytes == 4) {
        s_next[t][0] = __builtin_amdgcn_raw_buffer_load_b32(is_a ? as : bs, scale_off, so, 0);
      } else {
        s_next[t][0] = __builtin_amdgcn_raw_buffer_load_b16(is_a ? as : bs, scale_off, so, 0);
      }
    }
  };

  // This wave's blocks are wave, wave + WAVES, .. A block's codes pass through the wave's own LDS into registers as soon as
  // they have arrived; the next block's are then requested into the same LDS and travel while this one is multiplied. No
  // other wave touches that LDS, so waiting for the wave's own loads is all the synchronisation there is.
  const int blocks = (int)((K + kStreamBlockK - 1) / kStreamBlockK);
  if (wave < blocks) request(wave, (int)K - wave * kStreamBlockK);
  for (int blk = wave; blk < blocks; blk += WAVES) {
    AMX_WAIT_VMCNT(0);
    asm volatile("" ::: "memory");
    u32x4 w[kTiles][Piece::kWords / 4];
    uint32_t sc[kTiles][Piece::kScaleWords];
    if constexpr (FEW != 0) {
#pragma unroll
      for (int i = 0; i < FEW / 2; ++i) {
        uint32_t s_pos, s_neg;
        stream_scales<SCALE_KIND, ASYM>(&few_scales[i], 0, s_pos, s_neg);
        *reinterpret_cast<u32x4*>(few_lds + (2 * i + (lane >> 5)) * kFewRowBytes + (((lane & 31) ^ (((2 * i + (lane >> 5)) & 3) + 4 * ((lane >> 4) & 1))) << 4)) =
            stream_dequant<SCALE_KIND, ASYM>(few_word[i], s_pos, s_neg);
      }
    }
#pragma unroll
    for (int t = FEW ? MT : 0; t < kTiles; ++t) {
#pragma unroll
      for (int c = 0; c < Piece::kWords / 4; ++c)
        w[t][c] = *reinterpret_cast<const u32x4*>(mine + (FEW ? t - MT : t) * R * kRowBytes + read_off[c]);
#pragma unroll
      for (int i = 0; i < Piece::kScaleWords; ++i) sc[t][i] = s_next[t][i];
    }
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): the codes are in registers, their LDS may be refilled
    asm volatile("" ::: "memory");
    if (blk + WAVES < blocks) request(blk + WAVES, (int)K - (blk + WAVES) * kStreamBlockK);
#pragma unroll
    for (int e = 0; e < Piece::kEntries; ++e) {
      uint32_t s_pos[kTiles], s_neg[kTiles];
#pragma unroll
      for (int t = FEW ? MT : 0; t < kTiles; ++t) stream_scales<SCALE_KIND, ASYM>(sc[t], e, s_pos[t], s_neg[t]);
#pragma unroll
      for (int x = 0; x < Piece::kWordsPerEntry; ++x) {
        const int s = e * Piece::kWordsPerEntry + x;
        u32x4 av[MT];
#pragma unroll
        for (int i = 0; i < MT; ++i) {
          if constexpr (FEW != 0)
            av[i] = *reinterpret_cast<const u32x4*>(few_lds + (r % FEW) * kFewRowBytes + ((8 * piece + (s ^ ((r & 3) + 4 * (piece >> 1)))) << 4));
          else
            av[i] = stream_dequant<SCALE_KIND, ASYM>(w[i][s >> 2][s & 3], s_pos[i], s_neg[i]);
        }
#pragma unroll
        for (int j = 0; j < NT; ++j) {
          const u32x4 bv = stream_dequant<SCALE_KIND, ASYM>(w[MT + j][s >> 2][s & 3], s_pos[MT + j], s_neg[MT + j]);
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
  }

  // the waves' sums, added in ascending wave order (other waves' codes may still be on their way into the LDS that the
  // sums take)
  float* sums = reinterpret_cast<float*>(lds);
  __syncthreads();
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int v = 0; v < kAcc; ++v) sums[(((wave * MT + i) * NT + j) * kAcc + v) * 64 + lane] = acc[i][j][v];
  __syncthreads();
  constexpr int kTile = MT * NT * kAcc * 64;
  auto total = [&](int idx) {
    float s = sums[idx];
#pragma unroll
    for (int w = 1; w < WAVES; ++w) s += sums[w * kTile + idx];
    if constexpr (SCALE_KIND == kScaleE5M2) s *= 64.0f;  // undo the two biases
    return s;
  };
  // register v of lane l: 32 x 32 tiles: row 8 (v / 4) + 4 (l / 32) + v % 4; 16 x 16: row 4 (l / 16) + v
  auto row_of = [](int i, int v, int l) { return i * R + (R == 32 ? 8 * (v >> 2) + 4 * (l >> 5) + (v & 3) : 4 * (l >> 4) + v); };
  if constexpr (GLU) {
    static_assert(NT * R == 64, "one block of gate rows and one of up rows per workgroup");
    uint16_t* out = reinterpret_cast<uint16_t*>(C) + m0 * ldc + (n0 >> 1);
    constexpr int kHalf = NT / 2;  // column tiles of the gate; the up columns follow
#pragma unroll
    for (int e = 0; e < (kTile / 2 + 64 * WAVES - 1) / (64 * WAVES); ++e) {
      const int p = e * 64 * WAVES + (int)threadIdx.x;
      const int l = p & 63, v = (p >> 6) % kAcc, j = (p / (64 * kAcc)) % kHalf, i = p / (64 * kAcc * kHalf);
      if ((kTile / 2) % (64 * WAVES) == 0 || p < kTile / 2) {
        const int gate = ((i * NT + j) * kAcc + v) * 64 + l, row = row_of(i, v, l);
        const float value = silu_mul_value(total(gate), total(gate + kHalf * kAcc * 64));
        if (row < rows_a && 64 <= rows_b) out[row * ldc + j * R + l % R] = (uint16_t)bf16_rne(value);
      }
    }
    return;
  }
  const float alpha = alpha_a ? alpha_a[0] * alpha_b[0] : 1.0f;
  float* Cb = C + (b * M + m0) * ldc + n0;
#pragma unroll
  for (int e = 0; e < (kTile + 64 * WAVES - 1) / (64 * WAVES); ++e) {
    const int idx = e * 64 * WAVES + (int)threadIdx.x;
    if (kTile % (64 * WAVES) == 0 || idx < kTile) {
      const int l = idx & 63, v = (idx >> 6) % kAcc, j = (idx / (64 * kAcc)) % NT, i = idx / (64 * kAcc * NT);
      const int row = row_of(i, v, l), col = j * R + l % R;
      float s = total(idx);
      if (alpha_a) s *= alpha;
      if (row < rows_a && col < rows_b) Cb[row * ldc + col] = s;
    }
  }
}

// Whether workgroups of 48 columns fill their rounds of 256 compute units at least a tenth better than those of 64.
inline bool stream_48_columns(int64_t N, int64_t batch) {
  if (batch != 1 || N <= 8192) return false;
  auto fill = [](int64_t groups) { return (double)groups / (double)((groups + 255) / 256); };
  return fill((N + 47) / 48) >= 1.1 * fill((N + 63) / 64);
}

template <bool GLU>
static hipError_t stream_launch(int scale_kind, bool asym, int64_t group_size, int64_t M, int64_t N, int64_t K,
                              const uint8_t* A_codes, const uint8_t* A_scales, const uint8_t* B_codes,
                              const uint8_t* B_scales, const float* A_tensor_pair, const float* B_tensor_pair, float* C,
                              int64_t ldc, int64_t batch, hipStream_t s, const KernelTimer& timer) {
  if ((group_size != 32 && group_size != 16) || K % 32 != 0) return hipErrorInvalidValue;
  hipError_t e = hipSuccess;
  if (timer.start && (e = hipEventRecord(timer.start, s)) != hipSuccess) return e;
  auto run_few = [&]<int SK, bool ASYM, int GSL, int R, int MT, int NT, int WAVES, bool WHOLE, int FEW>() {
    hipLaunchKernelGGL((gemm_stream_kernel<SK, ASYM, GSL, R, MT, NT, WAVES, FEW, WHOLE, GLU>),
                       dim3((unsigned)((N + NT * R - 1) / (NT * R)), (unsigned)((M + MT * R - 1) / (MT * R)), (unsigned)batch),
                       dim3(64 * WAVES), 0, s, A_codes, A_scales, B_codes, B_scales, C, M, N, K, ldc, A_tensor_pair, B_tensor_pair);
    return hipGetLastError();
  };
  auto run = [&]<int SK, bool ASYM, int GSL, int R, int MT, int NT, int WAVES, bool WHOLE>() {
    if constexpr (R == 16 && MT == 1 && (ASYM || SK != kScaleE8M0Floor))  // (symmetric power-of-two scales: nothing gained)
      if (M <= 4) return run_few.template operator()<SK, ASYM, GSL, R, MT, NT, WAVES, WHOLE, 4>();
    return run_few.template operator()<SK, ASYM, GSL, R, MT, NT, WAVES, WHOLE, 0>();
  };
  // The smallest tiles that still give the 256 compute units one workgroup of eight waves each; beyond that tiles of 64 x
  // 64 in workgroups of four waves, two to a compute unit. (AMXFP4-E5M2, us by tile: 16 rows, N 4096, K 4096: 16 x 16 4.8,
  // 16 x 32 6.1;  N 6144: 7.6, 6.8;  N 28672, K 8192: 39, 36, 16 x 64 35. 32 rows, N 4096: two 16-row tiles x 16 columns
  // 6.8, 32 x 32 8.0;  N 11008: 32 x 32 13.0, 32 x 64 12.5;  N 28672, K 8192: 44.8, 45.7, the latter in four waves 40.6.
  // 128 rows, N 4096: 32 x 32 13.2, 32 x 64 11.8;  256 rows: 22, 22, 64 x 64 in eight waves 16.7, in four 17.7;  512 rows:
  // 43, 41, 31.6, 27.7, 64 x 128 27.9.)
  // Up to 32 rows, beyond 8192 columns: workgroups of 48 columns (16-row tiles, three column tiles) where they fill the rounds
  // of compute units at least a tenth better than those of 64 (stream_48_columns(); K in whole blocks, plain form). Us, 64 / 48
  // columns: 24 x 11008 x 4096 11.8 / 11.0 (172 workgroups, 230), 20 x 10240 x 8192 18.7 / 16.8, 32 x 22016 x 4096 19.7 / 17.2
  // (344, 459), 1 x 11008 x 4096 10.3 / 9.0, 16 x 10240 x 8192 16.4 / 14.1, 1 x 22016 x 4096 16.7 / 13.8; NVFP4, 24 x 11008 x
  // 4096 9.4 / 8.9; but 32 x 28672 x 8192 (448, 598) 39.9 / 45.4, 32 x 13824 x 5120 (216, 288) 14.4 / 20.6. (One workgroup of 112
  // columns to each unit for 28672: 43.5, too few lines in flight.)
  const int64_t t16 = (N + 15) / 16 * batch, t32 = (N + 31) / 32 * batch, rows32 = (M + 31) / 32;
  auto shape = [&]<int SK, bool ASYM, int GSL>() {
    auto pick = [&]<bool WHOLE>() {
      if constexpr (!GLU && WHOLE) {
        if (M <= 16 && stream_48_columns(N, batch)) return run.template operator()<SK, ASYM, GSL, 16, 1, 3, 8, WHOLE>();
        if (M <= 32 && stream_48_columns(N, batch)) return run.template operator()<SK, ASYM, GSL, 16, 2, 3, 8, WHOLE>();
      }
      if (M <= 16) {
        if constexpr (!GLU) {
          if (t16 <= 256) return run.template operator()<SK, ASYM, GSL, 16, 1, 1, 8, WHOLE>();
          if (t16 <= 512) return run.template operator()<SK, ASYM, GSL, 16, 1, 2, 8, WHOLE>();
        }
        return run.template operator()<SK, ASYM, GSL, 16, 1, 4, 8, WHOLE>();
      }
      if constexpr (!GLU) {  // (the gated form needs 64 columns to a workgroup)
        if (M <= 32 && t32 <= 128) return run.template operator()<SK, ASYM, GSL, 16, 2, 1, 8, WHOLE>();
        if (rows32 * t32 <= 256) return run.template operator()<SK, ASYM, GSL, 32, 1, 1, 8, WHOLE>();
      }
      if (rows32 * ((t32 + 1) / 2) <= 256) return run.template operator()<SK, ASYM, GSL, 32, 1, 2, 8, WHOLE>();
      if (M <= 32) return run.template operator()<SK, ASYM, GSL, 32, 1, 2, 4, WHOLE>();
      if ((rows32 + 1) / 2 * ((t32 + 1) / 2) <= 256) return run.template operator()<SK, ASYM, GSL, 32, 2, 2, 8, WHOLE>();
      return run.template operator()<SK, ASYM, GSL, 32, 2, 2, 4, WHOLE>();
    };
    return K % kStreamBlockK == 0 ? pick.template operator()<true>() : pick.template operator()<false>();
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
