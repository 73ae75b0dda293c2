// The fused attention for few queries (attention_decode.hip has the definition and the other kernel) where the queries of a key /
// value head fill at most 16 columns: (q_heads / kv_heads) * Sq <= 16, which is a new token of most models.
//
// Per-tile arithmetic, the ranges of keys and their combination are attention_decode.hip's. What bounds that kernel is one chain per
// range: a wave walks its key tiles one by one (dequantize K, product, maximum, exponentials, cast, dequantize V, product: 2 us a
// tile), on matrix tiles of 32 columns of which 1 to 8 hold a query, and four sequences give a SIMD one wave. Here
//   - a range is a workgroup of four waves. A round takes four key tiles (or eight, below), one to a wave: dequantization and first
//     product need nothing of the other tiles; then the waves exchange the tiles' maxima through LDS, and each knows the running
//     maximum that its tile's probabilities are cast against. Each wave accumulates its tiles' share of the output against its own last
//     maximum; the shares are added at the end, times 2^(m_wave - m_range), as ranges are;
//   - products are 16 x 16 x 32: half the scores, exponentials and casts per tile, half the accumulators (32 with heads of 128), so four
//     waves per SIMD (121 to 128 registers with heads of 128, 85 to 89 with heads of 64; as four waves with 32 columns, or with two rounds'
//     requests in flight, they spill or gain nothing);
//   - V of a round goes through registers into LDS (two buffers, one barrier a round); V and K of the next round are requested before
//     this round's second product;
//   - neighbouring ranges run on one XCD.
// The whole call (this kernel and the combination), us, before this kernel and the combination by four waves / now, cache in codes, 32 / 8
// heads of 128, three caches in turn: AMXFP4 4 sequences x 8192 keys 23.1 / 15.8, 1 x 8192 16.3 / 8.5, 16 x 8192
// 61 / 45 (3.3 TB/s), 1 x 16384 22.3 / 11.8; OCP MXFP4 16 x 8192 47 / 38; 32 / 32 heads of 64, 9 x 2048 25.8 / 20.6. Of these, with the
// combination by one wave: 16.5, 11.3, 46, 14.5, 38, 21.0; and so with two waves to a range: 24.3, 14.0, 81; with eight: 18.1, 12.4, 52;
// ranges dealt to the XCDs in turn: 19.4, 12.8, 48 (an eighth of each line of V's scale bytes used per fetch).
//
// Layouts in registers. First product, S^T[key, query] = K_tile . Q^T: lane l of the A operand holds row l % 16 and 8 head dimensions
// of quarter l / 16; k-step s multiplies word s of the quarter's D / 4 contiguous dimensions, for K and Q alike. Row i of block kb
// (two blocks of 16) is key 8 (i / 4) + 4 kb + i % 4 of the tile, so that the accumulator registers of lane quarter q (rows 4 q ..
// 4 q + 3 of both blocks) are keys 8 q .. 8 q + 7: as the B operand of the one k-step of the second product, O^T[d, query] += V^T .
// P^T, they meet word q of the 16 bytes that a row of V^T has for the tile.
#include "../../include/amxfp4.h"
#include "attention_decode.h"
#include "gemm_common.h"
#include "kernels.h"

namespace amx {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

template <int SCALE_KIND>
__device__ __forceinline__ f32x4 decode_mfma_16(u32x4 a, u32x4 b, f32x4 acc) {
  if constexpr (kDecodeF16<SCALE_KIND>)
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), acc, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc, 0, 0, 0);
}

// over the four lanes l % 16 of a column
__device__ __forceinline__ float column_max(float v) {
  const auto a = __builtin_amdgcn_permlane16_swap(f2u(v), f2u(v), false, false);
  v = fmaxf(u2f(a[0]), u2f(a[1]));
  const auto b = __builtin_amdgcn_permlane32_swap(f2u(v), f2u(v), false, false);
  return fmaxf(u2f(b[0]), u2f(b[1]));
}
__device__ __forceinline__ float column_sum(float v) {
  const auto a = __builtin_amdgcn_permlane16_swap(f2u(v), f2u(v), false, false);
  v = u2f(a[0]) + u2f(a[1]);
  const auto b = __builtin_amdgcn_permlane32_swap(f2u(v), f2u(v), false, false);
  return u2f(b[0]) + u2f(b[1]);
}

// A lane's share of a row of K or Q: the words of codes of its quarter's D / 4 dimensions and the scale bytes of their group, as they
// were loaded.
template <int D>
struct QuarterPiece {
  uint32_t word[D / 32];
  uint32_t scales;
};

constexpr int kNowhere16 = (int)0x80000000;      // an offset beyond every buffer: such a load returns zeros

// codes_off, scales_off: of the lane; row: more rows, alike in all lanes
template <int D, bool ASYM>
__device__ __forceinline__ void load_quarter(__amdgpu_buffer_rsrc_t codes, __amdgpu_buffer_rsrc_t scales, int codes_off, int scales_off,
                                             int row, QuarterPiece<D>& p) {
  if constexpr (D == 128) {
    const u32x4 c = __builtin_amdgcn_raw_buffer_load_b128(codes, codes_off, row * (D / 2), 0);
#pragma unroll
    for (int i = 0; i < 4; ++i) p.word[i] = c[i];
  } else {
    const u32x2 c = __builtin_amdgcn_raw_buffer_load_b64(codes, codes_off, row * (D / 2), 0);
    p.word[0] = c[0], p.word[1] = c[1];
  }
  if constexpr (ASYM)
    p.scales = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(scales, scales_off, row * (D / 32) * 2, 0);
  else
    p.scales = (uint8_t)__builtin_amdgcn_raw_buffer_load_b8(scales, scales_off, row * (D / 32), 0);
}

template <int SCALE_KIND, bool ASYM, int D>
__device__ __forceinline__ u32x4 decode_quarter(const QuarterPiece<D>& p, int s) {
  return decode_word_of_pair<SCALE_KIND, ASYM>(p.word[s], kDecodeF16<SCALE_KIND> ? p.scales & 0x7F7Fu : p.scales);
}

// grid: (key_splits, kv_heads); block: W waves, each with T tiles of a round. part: as attention_decode_kernel writes it. WIDE: the
// scale bytes of V that a lane fetches, those of kPieces neighbouring key tiles of a row, are one aligned piece.
template <int SCALE_KIND, bool ASYM, int D, int W, int T, bool WIDE>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(4, 4))) void attention_decode_16_kernel(
    const uint8_t* __restrict__ Qc, const uint8_t* __restrict__ Qs, const uint8_t* __restrict__ Kc,
    const uint8_t* __restrict__ Ks, const uint8_t* __restrict__ Vc, const uint8_t* __restrict__ Vs,
    float* __restrict__ part, int Sq, int Sk, int per, int tiles_per_split, float scale_log2, int causal) {
  constexpr int kSteps = D / 32, kRowBlocks = D / 16;
  constexpr int kRound = W * T;            // key tiles
  constexpr int kPair = ASYM ? 2 : 1;      // scale bytes of a group
  constexpr int kPieces = D * T / 64;      // 16-byte pieces of V's codes, and scales of V, that a lane fetches per round
  constexpr int kLine = kRound * 16;       // codes of a round's tiles in a row of V^T
  constexpr int kBuffer = D * kLine, kScaleBuffer = D * kRound * kPair;
  constexpr int kScaleLoads = WIDE ? 1 : kPieces, kScaleBytes = kPieces / kScaleLoads * kPair;
  constexpr int kSwizzleRows = 16 / kRound;  // rows after which a line's banks come round
  // V codes of two rounds, then their scale bytes, row by row; at the end the waves' shares of the output (W x D x 16 floats)
  constexpr int kShares = W * kRowBlocks * 1024, kV = 2 * (kBuffer + kScaleBuffer);
  __shared__ __attribute__((aligned(1024))) uint8_t lds[kShares > kV ? kShares : kV];
  __shared__ __attribute__((aligned(16))) float tile_max[2 * 16 * kRound];  // [column][tile of the round]
  __shared__ float wave_sum[W * 16];
  uint8_t* const v_lines = lds;
  uint8_t* const v_scales = lds + 2 * kBuffer;

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), col = lane & 15, quarter = lane >> 4;
  // Neighbouring ranges share the lines of V's scale bytes (16 of 128 bytes are a range of eight tiles'), so each XCD, which gets every
  // eighth workgroup, takes one run of them: L2 then fetches such a line once.
  const int nsplits = (int)gridDim.x, wg = (int)(blockIdx.y * gridDim.x + blockIdx.x), wgs = nsplits * (int)gridDim.y;
  const int xcd = wg & 7, run = wgs >> 3, more = wgs & 7, range = xcd * run + (xcd < more ? xcd : more) + (wg >> 3);
  const int g = range / nsplits, split = range - g * nsplits;
  const int off = Sk - Sq;
  const bool col_valid = col < per * Sq;
  const int qi = col_valid ? col % Sq : 0;
  // a padding column multiplies zeros and sees every key: its numbers stay finite and are never read
  const int limit = col_valid && causal ? qi + off : Sk - 1;
  constexpr bool kF16 = kDecodeF16<SCALE_KIND>;
  const float score_scale = kF16 ? scale_log2 * 64.0f : scale_log2;  // (the biases: attention_decode.hip)

  const int tiles_all = Sk >> 5;
  const int t0 = split * tiles_per_split;
  const int t1 = t0 + tiles_per_split < tiles_all ? t0 + tiles_per_split : tiles_all;

  // (the addresses are the same in every lane; said explicitly, or the descriptors end up in vector registers and every load in a loop
  // over their distinct values; bytes: below 2^30, Sk is at most 2^20)
  auto buffer_of = [](const uint8_t* p, int64_t bytes) {
    const uint64_t a = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)a), hi = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32));
    return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<uint8_t*>(((uint64_t)hi << 32) | lo), 0,
                                             __builtin_amdgcn_readfirstlane((int)bytes), 0x00020000);
  };
  const int v_row_bytes = Sk >> 1, vs_row_bytes = tiles_all * kPair;
  const __amdgpu_buffer_rsrc_t k_rsrc = buffer_of(Kc + (int64_t)g * Sk * (D / 2), (int64_t)Sk * (D / 2));
  const __amdgpu_buffer_rsrc_t ks_rsrc = buffer_of(Ks + (int64_t)g * Sk * (D / 32) * kPair, (int64_t)Sk * (D / 32) * kPair);
  const __amdgpu_buffer_rsrc_t v_rsrc = buffer_of(Vc + (int64_t)g * D * v_row_bytes, (int64_t)D * v_row_bytes);
  const __amdgpu_buffer_rsrc_t vs_rsrc = buffer_of(Vs + (int64_t)g * D * vs_row_bytes, (int64_t)D * vs_row_bytes);
  const __amdgpu_buffer_rsrc_t q_rsrc = buffer_of(Qc + (int64_t)g * per * Sq * (D / 2), (int64_t)per * Sq * (D / 2));
  const __amdgpu_buffer_rsrc_t qs_rsrc = buffer_of(Qs + (int64_t)g * per * Sq * (D / 32) * kPair, (int64_t)per * Sq * (D / 32) * kPair);

  // What a wave requests of the round that starts at key tile t: its tiles' K rows, its share of V.
  const int key_in_tile = 8 * (col >> 2) + (col & 3);  // of row l % 16 in block 0; 4 more in block 1
  const int k_lane = key_in_tile * (D / 2) + quarter * (D / 8), ks_lane = (key_in_tile * (D / 32) + quarter * D / 128) * kPair;
  const int v_tile = tid % kRound, v_row = tid / kRound;  // of piece u: row v_row + 64 / T u
  const int s_row = tid / (64 * W / D), s_tile = tid % (64 * W / D) * kPieces;
  const int v_lane = v_row * v_row_bytes + v_tile * 16, vs_lane = s_row * vs_row_bytes + s_tile * kPair;
  QuarterPiece<D> kp[T][2];
  u32x4 vl[kPieces];
  uint32_t vsc[kScaleBytes == 8 ? 2 : kScaleLoads];
  auto request = [&](int t_lanes) {
    const int t = __builtin_amdgcn_readfirstlane(t_lanes);  // (alike in all lanes; the compiler loses that over the loop)
#pragma unroll
    for (int j = 0; j < T; ++j) {
      const int kt = t + wave + W * j;
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
        load_quarter<D, ASYM>(k_rsrc, ks_rsrc, kt < t1 ? k_lane : kNowhere16, kt < t1 ? ks_lane : kNowhere16, kt * 32 + 4 * kb, kp[j][kb]);
    }
#pragma unroll
    for (int u = 0; u < kPieces; ++u)
      vl[u] = __builtin_amdgcn_raw_buffer_load_b128(v_rsrc, t + v_tile < t1 ? v_lane : kNowhere16, 64 / T * u * v_row_bytes + t * 16, 0);
#pragma unroll
    for (int k = 0; k < kScaleLoads; ++k) {  // (past the row's end: the next row's, or zeros; of tiles that nobody multiplies)
      const int so = t * kPair + k * kScaleBytes;
      if constexpr (kScaleBytes == 8) {
        const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(vs_rsrc, vs_lane, so, 0);
        vsc[0] = v[0], vsc[1] = v[1];
      } else if constexpr (kScaleBytes == 4) {
        vsc[k] = __builtin_amdgcn_raw_buffer_load_b32(vs_rsrc, vs_lane, so, 0);
      } else if constexpr (kScaleBytes == 2) {
        vsc[k] = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(vs_rsrc, vs_lane, so, 0);
      } else {
        vsc[k] = (uint8_t)__builtin_amdgcn_raw_buffer_load_b8(vs_rsrc, vs_lane, so, 0);
      }
    }
  };
  // tile j of row r in LDS: slot j ^ (r / kSwizzleRows) % kRound of the row's line, so that the 16 rows of a read spread over the banks
  const int v_store = v_row * kLine + ((v_tile ^ ((v_row / kSwizzleRows) % kRound)) << 4);
  const int v_word = col * kLine + ((wave ^ ((col / kSwizzleRows) % kRound)) << 4) + 4 * quarter;  // (its second tile: slot ^ W)
  auto store_v = [&](int buf) {
#pragma unroll
    for (int u = 0; u < kPieces; ++u) *reinterpret_cast<u32x4*>(v_lines + buf * kBuffer + v_store + u * (64 / T) * kLine) = vl[u];
    constexpr uint32_t kClear = kF16 ? 0x7F7F7F7Fu : 0xFFFFFFFFu;  // (the sign bit of an FP8 scale byte is ignored)
    uint8_t* dst = v_scales + buf * kScaleBuffer + (s_row * kRound + s_tile) * kPair;
#pragma unroll
    for (int k = 0; k < kScaleLoads; ++k) {
      if constexpr (kScaleBytes == 8)
        *reinterpret_cast<u32x2*>(dst) = u32x2{vsc[0] & kClear, vsc[1] & kClear};
      else if constexpr (kScaleBytes == 4)
        *reinterpret_cast<uint32_t*>(dst + 4 * k) = vsc[k] & kClear;
      else if constexpr (kScaleBytes == 2)
        *reinterpret_cast<uint16_t*>(dst + 2 * k) = (uint16_t)(vsc[k] & kClear);
      else
        dst[k] = (uint8_t)(vsc[k] & kClear);
    }
  };

  QuarterPiece<D> query;
  load_quarter<D, ASYM>(q_rsrc, qs_rsrc, col_valid ? col * (D / 2) + quarter * (D / 8) : kNowhere16,
                        col_valid ? (col * (D / 32) + quarter * D / 128) * kPair : kNowhere16, 0, query);  // (head col / Sq, query col % Sq)
  request(t0);
  u32x4 qf[kSteps];
#pragma unroll
  for (int s = 0; s < kSteps; ++s) qf[s] = decode_quarter<SCALE_KIND, ASYM, D>(query, s);  // (zeros in a padding column: codes 0)

  f32x4 o[kRowBlocks];
#pragma unroll
  for (int db = 0; db < kRowBlocks; ++db) o[db] = f32x4{0.f, 0.f, 0.f, 0.f};
  // m: the running maximum of the range (log2 units), alike in all waves; m_wave, l: what this wave's o and sum (this lane's eight
  // of each tile's keys) stand against
  float m = -__builtin_inff(), m_wave = -__builtin_inff(), l = 0.f;

  int buf = 0;
  for (int t = t0; t < t1; t += kRound, buf ^= 1) {
    float x[T][8], mx[T];
#pragma unroll
    for (int j = 0; j < T; ++j) {
      const int kt = t + wave + W * j;
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) {
        if constexpr (T > 1) __builtin_amdgcn_sched_barrier(0);  // (one block's operands at a time in registers)
        f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < kSteps; ++ks) s = decode_mfma_16<SCALE_KIND>(decode_quarter<SCALE_KIND, ASYM, D>(kp[j][kb], ks), qf[ks], s);
#pragma unroll
        for (int v = 0; v < 4; ++v) x[j][4 * kb + v] = s[v] * score_scale;
      }
      if (causal && kt * 32 + 31 > off) {  // some key of the tile is masked for the first query (uniform)
#pragma unroll
        for (int v = 0; v < 8; ++v)
          if (kt * 32 + 8 * quarter + v > limit) x[j][v] = -__builtin_inff();
      }
      mx[j] = -__builtin_inff();
      if (kt < t1) {
#pragma unroll
        for (int v = 0; v < 8; ++v) mx[j] = fmaxf(mx[j], x[j][v]);
        mx[j] = column_max(mx[j]);
      }
      if (quarter == 0) tile_max[(buf * 16 + col) * kRound + W * j + wave] = mx[j];
    }
    store_v(buf);
    if constexpr (T == 1)
      if (t + kRound < t1) request(t + kRound);
    // Every wave has read what it needed of this buffer before it came to the last round's barrier. Only LDS is waited for: the
    // requests stay in flight.
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    float m_tile[T];
#pragma unroll
    for (int j = 0; j < T; ++j) {
      float tm[W];
#pragma unroll
      for (int w = 0; w < W; ++w) tm[w] = tile_max[(buf * 16 + col) * kRound + W * j + w];
      m_tile[j] = m;
#pragma unroll
      for (int w = 0; w < W; ++w) {
        if (w <= wave) m_tile[j] = fmaxf(m_tile[j], tm[w]);
        m = fmaxf(m, tm[w]);
      }
    }
#pragma unroll
    for (int j = 0; j < T; ++j) {
      if (t + wave + W * j >= t1) continue;  // uniform
      if constexpr (T > 1) __builtin_amdgcn_sched_barrier(0);  // (one tile's words at a time in registers)
      uint32_t word[kRowBlocks], sc[kRowBlocks];
#pragma unroll
      for (int db = 0; db < kRowBlocks; ++db) {
        const uint8_t* sb = v_scales + buf * kScaleBuffer + (col * kRound + W * j + wave) * kPair + db * 16 * kRound * kPair;
        sc[db] = ASYM ? *reinterpret_cast<const uint16_t*>(sb) : *sb;
        word[db] = *reinterpret_cast<const uint32_t*>(v_lines + buf * kBuffer + (v_word ^ (16 * W * j)) + db * 16 * kLine);
      }
      // (a query that has seen no key yet keeps probabilities 0 and factor 0 of nothing, not the NaN of -inf - -inf)
      const float m_new = m_tile[j] == -__builtin_inff() ? 0.f : m_tile[j];
      const float alpha = __builtin_amdgcn_exp2f(m_wave - m_new);
      m_wave = m_tile[j];
      const float pmax = __builtin_amdgcn_exp2f(mx[j] - m_new);
      float psum = 0.f;
#pragma unroll
      for (int v = 0; v < 8; ++v) {
        x[j][v] = __builtin_amdgcn_exp2f(x[j][v] - m_new);
        psum += x[j][v];
      }
      l = l * alpha + psum;
      uint32_t pb[4];
      AMX_ATTENTION_TILE_CAST(x[j], pmax, pb, kF16)
      if (__builtin_amdgcn_ballot_w64(alpha != 1.0f) != 0) {
#pragma unroll
        for (int db = 0; db < kRowBlocks; ++db) o[db] *= alpha;
      }
      const u32x4 b = {pb[0], pb[1], pb[2], pb[3]};
#pragma unroll
      for (int db = 0; db < kRowBlocks; ++db)
        o[db] = decode_mfma_16<SCALE_KIND>(decode_word_of_pair<SCALE_KIND, ASYM>(word[db], sc[db]), b, o[db]);
    }
    if constexpr (T > 1)
      if (t + kRound < t1) request(t + kRound);
  }

  // The waves' shares, each against its own maximum, become shares against the range's and are added, some row blocks to a wave,
  // always in the order of the waves. 2^-5 undoes the FP16 biases, exactly.
  const float factor = m_wave == -__builtin_inff() ? 0.f : __builtin_amdgcn_exp2f(m_wave - m);
  const float sum = column_sum(l) * factor, unbias = kF16 ? 0.03125f * factor : factor;
  if (quarter == 0) wave_sum[wave * 16 + col] = sum;
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");  // V has been read
  f32x4* shares = reinterpret_cast<f32x4*>(lds);
#pragma unroll
  for (int db = 0; db < kRowBlocks; ++db) shares[(wave * kRowBlocks + db) * 64 + lane] = o[db] * unbias;
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  float* dst = part + (((int64_t)g * kDecodeCols + col) * nsplits + split) * (D + 2);
#pragma unroll
  for (int i = 0; i < (kRowBlocks + W - 1) / W; ++i) {
    const int db = wave + W * i;
    if (db >= kRowBlocks) break;
    f32x4 v = shares[db * 64 + lane];
#pragma unroll
    for (int w = 1; w < W; ++w) v += shares[(w * kRowBlocks + db) * 64 + lane];
    // register r of row block db is d = 16 db + 4 quarter + r
    if (col_valid) {
      float2* d2 = reinterpret_cast<float2*>(dst + db * 16 + 4 * quarter);  // (rows of D + 2 floats: 8-byte aligned)
      d2[0] = make_float2(v[0], v[1]), d2[1] = make_float2(v[2], v[3]);
    }
  }
  if (wave == 0 && quarter == 0 && col_valid) {
    float all = wave_sum[col];
#pragma unroll
    for (int w = 1; w < W; ++w) all += wave_sum[w * 16 + col];
    dst[D] = m, dst[D + 1] = all;
  }
}

template <int SK, bool ASYM, int D>
static hipError_t launch_16(int per, int64_t Hkv, int64_t Sq, int64_t Sk, const uint8_t* Qc, const uint8_t* Qs, const uint8_t* Kc,
                            const uint8_t* Ks, const uint8_t* Vc, const uint8_t* Vs, float scale, int causal, int splits, float* part,
                            hipStream_t s) {
  const int tiles = (int)(Sk / 32), tiles_per_split = (tiles + splits - 1) / splits;
  auto go = [&]<int W, int T, bool WIDE>() {
    hipLaunchKernelGGL((attention_decode_16_kernel<SK, ASYM, D, W, T, WIDE>), dim3((unsigned)splits, (unsigned)Hkv), dim3(64 * W), 0, s, Qc,
                       Qs, Kc, Ks, Vc, Vs, part, (int)Sq, (int)Sk, per, tiles_per_split, scale * 1.4426950408889634f, causal);
    return hipGetLastError();
  };
  auto wide_or_not = [&]<int W, int T>() {
    constexpr int kPieces = D * T / 64;
    if constexpr (kPieces > 1)
      if (tiles % kPieces != 0 || tiles_per_split % kPieces != 0 || reinterpret_cast<uintptr_t>(Vs) % (kPieces * (ASYM ? 2 : 1)) != 0)
        return go.template operator()<W, T, false>();
    return go.template operator()<W, T, true>();
  };
  // Two tiles to a wave and round (whole lines of V, but no request in flight during the second product): heads of 128 from 2^20 keys of all
  // heads on (136 to 144 MB), in ranges of 16 tiles and more, for keys and values that come from memory. Two tiles / one, 2163 sizes, three
  // caches in turn, symmetric scales: 1.07 to 1.09 at 2^19 keys, 1.00 at 2^19.5, 0.97 at 2^20, 0.95 from 2^21 on (OCP MXFP4 16 x 8192 keys, 8
  // heads, 38.2 / 42.1 us); asymmetric ones, whose dequantization takes longer: 1.07, 1.04, 1.03 (but 16 x 8192 45.4 / 47.4),
  // 1.00. The same cache again and again, which up to 256 MB need not come from memory, 1.06 to 1.09 at 2^20, 1.00 beyond 2^21. Shorter ranges
  // 1.05 to 1.00 up to 2^20. Heads of 64, 5 x 16352 keys, one tile 21.8, two 23.9 us.
  if constexpr (D == 128)
    if (tiles_per_split >= 16 && Hkv * Sk >= (int64_t(1) << 20)) return wide_or_not.template operator()<4, 2>();
  return wide_or_not.template operator()<4, 1>();
}

// Ranges of a single tile leave three of the four waves idle, those of two or three some; the more ranges, the more that costs, most with
// heads of 64, whose tiles are half the work. Ratios of the whole call, this kernel / the other, over 5900 sizes:
//   one tile: 1.03 to 1.18 on average from one range to 65536, heads of 64 to 1.45 (8192 heads, 1024 groups x 32 keys, heads of 64, 15.7 /
//     9.8 us; 288 heads and groups x 96, heads of 128, three ranges, OCP MXFP4 8.4 / 5.7 with the new combination). Some are below 1, to 0.82: heads of 128, 1024 to 8192 ranges of whole chunks of eight
//     tiles (128 heads, 16 x 2048 keys, 64 ranges, two queries 13.3 / 15.8)
//   two tiles: heads of 64 0.92 below 512 ranges, 1.03 to 1.19 from there on (4096 heads, 1024 x 1024, 16 ranges 56.8 / 46.1); of 128 0.84 to 0.97
//   three: heads of 64 beyond 16384 ranges 1.02 to 1.06 up to four columns (816 heads, 408 x 7424, 78 ranges 122 / 110), 0.84 beyond; else 0.70 to 0.95
//   four and more: 0.3 to 0.93
bool attention_decode_16_preferred(int64_t Hq, int64_t Hkv, int64_t Sq, int64_t head_dim, int tiles_per_split, int key_splits) {
  const int64_t columns = (Hq / Hkv) * Sq, ranges = Hkv * key_splits;
  if (columns > 16 || tiles_per_split == 1) return false;
  if (head_dim == 128 || tiles_per_split > 3) return true;
  return tiles_per_split == 2 ? ranges < 512 : ranges < 16384 || columns > 4;
}

hipError_t launch_attention_decode_16(int scale_kind, bool asym, int64_t Hq, int64_t Hkv, int64_t Sq, int64_t Sk, int64_t head_dim,
                                      const uint8_t* Q_codes, const uint8_t* Q_scales, const uint8_t* K_codes, const uint8_t* K_scales,
                                      const uint8_t* V_codes, const uint8_t* V_scales, float scale, int causal, int key_splits,
                                      float* part, hipStream_t s) {
  const int per = (int)(Hq / Hkv);
  auto go = [&]<int SK, bool ASYM>() {
    if (head_dim == 128)
      return launch_16<SK, ASYM, 128>(per, Hkv, Sq, Sk, Q_codes, Q_scales, K_codes, K_scales, V_codes, V_scales, scale, causal, key_splits,
                                      part, s);
    return launch_16<SK, ASYM, 64>(per, Hkv, Sq, Sk, Q_codes, Q_scales, K_codes, K_scales, V_codes, V_scales, scale, causal, key_splits,
                                   part, s);
  };
  switch (scale_kind) {
    case kScaleE5M2: return asym ? go.template operator()<kScaleE5M2, true>() : go.template operator()<kScaleE5M2, false>();
    case kScaleE4M3: return asym ? go.template operator()<kScaleE4M3, true>() : go.template operator()<kScaleE4M3, false>();
    case kScaleE8M0Floor: return asym ? go.template operator()<kScaleE8M0Floor, true>() : go.template operator()<kScaleE8M0Floor, false>();
    case kScaleE8M0Round: return asym ? go.template operator()<kScaleE8M0Round, true>() : go.template operator()<kScaleE8M0Round, false>();
    default: return hipErrorInvalidValue;
  }
}

}  // namespace amx
