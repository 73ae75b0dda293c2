// Fused quantized attention for FEW queries against many keys (decoding: one or a handful of new tokens against a long
// key / value cache). Same per-tile arithmetic as attention.hip (Sec. 5.1 quantizes Q.K^T and the attention map times V;
// online softmax over key tiles of 32, each tile of probabilities cast as one group per query), but organised for the
// shape: the work is reading K and V once, so
//   - K and V are read as they are stored, packed codes and scale bytes, and dequantized in registers to exact 16-bit
//     floats (no BF16 panels in a workspace: a quarter of the bytes, and no expansion pass in front);
//   - the query heads that share a key / value head, and their few queries, are the 32 columns of ONE wave
//     (q_heads / kv_heads * Sq <= 32), so every K and V byte is read by one wave only. Up to 16 columns
//     attention_decode_16.hip takes the call (the rule and its times are there), with the same combination;
//   - the keys are the parallelism: the key tiles are cut into `key_splits` contiguous ranges, one wave per (key / value
//     head, range), no barriers (LDS only as a wave's own staging space for V); each wave leaves its un-normalised
//     result, running maximum and sum in the workspace and a second kernel combines the ranges exactly:
//       m* = max_c m_c,   out = sum_c O_c 2^(m_c - m*) / sum_c l_c 2^(m_c - m*).
//     The probabilities of a range are cast against that range's own running maximum, so the result depends on
//     key_splits (with one range it is the other kernel's result up to summation order).
//
// Layouts in registers. First product, S^T[key, query] = K_tile . Q^T on v_mfma_f32_32x32x16_bf16: lane l of the A
// operand holds key l % 32 and 8 head dimensions, of the B operand query column l % 32 and the same 8 dimensions. Which
// 8 does not matter as long as both agree (a sum over the head dimension): lane half h = l / 32 reads the D / 4
// contiguous bytes of codes of dimensions (D / 2) h .. of its row, and k-step s multiplies word s of them, i.e.
// dimensions (D / 2) h + 8 s .. + 7, for K and Q alike. Second product, O^T[d, query] += V^T . P^T: the probabilities
// leave attention_tile.h as the B operand of two k-steps with the tile's keys in accumulator order
// (16 j + 4 h + {0,1,2,3,8,9,10,11}); lane (d, h) picks exactly those eight codes out of the 16 bytes its V^T row has
// for the tile: two 16-bit pieces of two words, one byte permute.
#include "../../include/amxfp4.h"
#include "attention_decode.h"
#include "gemm_common.h"
#include "kernels.h"

namespace amx {

template <int SCALE_KIND>
__device__ __forceinline__ f32x16 decode_mfma(u32x4 a, u32x4 b, f32x16 acc) {
  if constexpr (kDecodeF16<SCALE_KIND>)
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), acc, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc, 0, 0, 0);
}

// One row's share of a lane for the first product: the D / 4 bytes of codes of dimensions (D / 2) h .. and the scale
// bytes of their D / 64 groups, as they were loaded: taking the bytes apart is left to where they are used, since
// anything done to them here would wait for the load (it did, once per key tile, for most of the tile's time).
typedef uint32_t u32_a2 __attribute__((aligned(2)));  // scale arrays are 2-byte aligned by contract
template <int D>
struct RowPiece {
  uint32_t word[D / 16];
  uint32_t scales;
};

template <int D, bool ASYM>
__device__ __forceinline__ void load_row_piece(const uint8_t* __restrict__ codes, const uint8_t* __restrict__ scales,
                                               int64_t row, int h, RowPiece<D>& p) {
  const uint4* src = reinterpret_cast<const uint4*>(codes + row * (D / 2) + h * (D / 4));
#pragma unroll
  for (int i = 0; i < D / 64; ++i) {
    const uint4 c = src[i];
    p.word[4 * i] = c.x, p.word[4 * i + 1] = c.y, p.word[4 * i + 2] = c.z, p.word[4 * i + 3] = c.w;
  }
  constexpr int kBytes = (D / 64) * (ASYM ? 2 : 1);
  const uint8_t* sb = scales + (row * (D / 32) + h * (D / 64)) * (ASYM ? 2 : 1);
  if constexpr (kBytes == 4)
    p.scales = *reinterpret_cast<const u32_a2*>(sb);
  else if constexpr (kBytes == 2)
    p.scales = *reinterpret_cast<const uint16_t*>(sb);
  else
    p.scales = *sb;
}

// k-step s of a row piece as 16-bit floats (group s / 4 of the piece)
template <int SCALE_KIND, bool ASYM, int D>
__device__ __forceinline__ u32x4 decode_step(const RowPiece<D>& p, int s) {
  const int i = s >> 2;
  const uint32_t pos = (p.scales >> (ASYM ? 16 * i : 8 * i)) & 255u, neg = ASYM ? (p.scales >> (16 * i + 8)) & 255u : pos;
  return decode_word<SCALE_KIND, ASYM>(p.word[s], pos, neg);
}

// A V^T row's share of a lane for one key tile: the 16 bytes of codes of the tile's 32 keys and the group's scale bytes.
struct VPiece {
  uint4 codes;
  uint32_t scales;
};

template <bool ASYM>
__device__ __forceinline__ void load_v_piece(const uint8_t* __restrict__ codes, const uint8_t* __restrict__ scales,
                                             int64_t row, int64_t Sk, int t, VPiece& p) {
  p.codes = *reinterpret_cast<const uint4*>(codes + row * (Sk >> 1) + (int64_t)t * 16);
  const int64_t g = row * (Sk >> 5) + t;
  if constexpr (ASYM)
    p.scales = *reinterpret_cast<const uint16_t*>(scales + g * 2);
  else
    p.scales = scales[g];
}

// grid: (key_splits, kv_heads); block: one wave. part: [kv_heads][32 columns][key_splits][D + 2] floats: the
// un-normalised O of the column in that range, then its running maximum (log2 units) and its sum; only the columns
// that hold a query are written.
//
// CHUNKED (Sk % 256 == 0): V^T rows are contiguous along the keys, so a key tile is 16 bytes of each of the D rows, one
// eighth of a cache line per row, and a wave that fetched them tile by tile would request every line of V eight times
// (and every line of V's scale bytes as often). The wave instead brings V in chunks of 8 key tiles: whole 128-byte
// lines of all D rows by direct-to-LDS loads (8 rows x 128 bytes per load; the 16-byte piece of tile j of row r goes to
// slot j ^ ((r >> 1) & 7) of the row's line in LDS, so that the 32 rows a tile read touches spread over the banks), and
// the chunk's scale bytes as D rows of 4-byte words. One chunk of LDS per wave, refilled when the wave has finished
// the previous chunk (its other wave on the SIMD works meanwhile); no barrier: a wave reads only what it loaded.
template <int SCALE_KIND, bool ASYM, int D, bool CHUNKED>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2, 2))) void attention_decode_kernel(
    const uint8_t* __restrict__ Qc, const uint8_t* __restrict__ Qs, const uint8_t* __restrict__ Kc,
    const uint8_t* __restrict__ Ks, const uint8_t* __restrict__ Vc, const uint8_t* __restrict__ Vs,
    float* __restrict__ part, int Sq, int Sk, int per, int tiles_per_split, float scale_log2, int causal) {
  constexpr int kSteps = D / 16, kRowBlocks = D / 32;
  constexpr int kScaleParts = ASYM ? 4 : 2;  // 4-byte words of scale bytes a row has per chunk of 8 tiles
  __shared__ __attribute__((aligned(1024))) uint8_t v_lines[CHUNKED ? D * 128 : 16];
  __shared__ __attribute__((aligned(256))) uint8_t v_scale_words[CHUNKED ? kScaleParts * D * 4 : 16];
  const int lane = threadIdx.x & 63, col = lane & 31, h = lane >> 5;
  const int split = (int)blockIdx.x, nsplits = (int)gridDim.x, g = (int)blockIdx.y;
  const int off = Sk - Sq;
  const bool col_valid = col < per * Sq;
  const int qi = col_valid ? col % Sq : 0;
  // a padding column multiplies zeros and sees every key: its numbers stay finite and are never read
  const int limit = col_valid && causal ? qi + off : Sk - 1;

  // FP16 operands carry 2^-3 each: the scores come out divided by 2^6, the second product (probabilities times 2^8, so
  // that the smallest of them, 2^-17, is a normal FP16 number, times V / 8) multiplied by 2^5
  constexpr bool kF16 = kDecodeF16<SCALE_KIND>;
  const float score_scale = kF16 ? scale_log2 * 64.0f : scale_log2;

  f32x16 o[kRowBlocks];
#pragma unroll
  for (int db = 0; db < kRowBlocks; ++db)
#pragma unroll
    for (int v = 0; v < 16; ++v) o[db][v] = 0.f;
  float m = -__builtin_inff(), l = 0.f;
  const int row_in_tile = 4 * h;  // key of accumulator register v: 8 (v / 4) + row_in_tile + v % 4

  const int tiles_all = Sk >> 5;
  const int t0 = split * tiles_per_split;
  const int t1 = t0 + tiles_per_split < tiles_all ? t0 + tiles_per_split : tiles_all;
  const int64_t krow0 = (int64_t)g * Sk + col;                      // K row of this lane in tile 0 (key = lane % 32)
  const int64_t vrow0 = (int64_t)g * D + col;                       // V^T row of this lane in row block 0
  // lane half h takes the low (h = 0) or high (h = 1) 16-bit pieces of two neighbouring words: keys 4 h .. 4 h + 3 and
  // 4 h + 8 .. 4 h + 11 of each 16
  const uint32_t pick = h ? 0x07060302u : 0x05040100u;

  // CHUNKED: this head's V^T codes and scale bytes as raw buffers (reads past the end return zeros), and the lane's
  // share of a load of 8 rows x 128 bytes: row L / 8 of the eight, the piece that belongs in slot L % 8
  const int v_row_bytes = Sk >> 1, vs_row_bytes = (Sk >> 5) * (ASYM ? 2 : 1);
  // (the addresses are the same in every lane; said explicitly, or the descriptors end up in vector registers and
  // every load in a loop over their distinct values)
  auto uniform_ptr = [](const uint8_t* p) {
    const uint64_t a = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)a), hi = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32));
    return reinterpret_cast<uint8_t*>(((uint64_t)hi << 32) | lo);
  };
  const __amdgpu_buffer_rsrc_t v_rsrc = __builtin_amdgcn_make_buffer_rsrc(
      uniform_ptr(Vc + (int64_t)g * D * v_row_bytes), 0, __builtin_amdgcn_readfirstlane(D * v_row_bytes), 0x00020000);
  const __amdgpu_buffer_rsrc_t vs_rsrc = __builtin_amdgcn_make_buffer_rsrc(
      uniform_ptr(Vs + (int64_t)g * D * vs_row_bytes), 0, __builtin_amdgcn_readfirstlane(D * vs_row_bytes), 0x00020000);
  const int v_gather0 = (lane >> 3) * v_row_bytes + (((lane & 7) ^ (lane >> 4)) << 4);        // even load units
  const int v_gather1 = (lane >> 3) * v_row_bytes + (((lane & 7) ^ (4 + (lane >> 4))) << 4);  // odd load units
  const int v_read_swz = (col >> 1) & 7;  // rows 32 db + col: (row >> 1) & 7 does not depend on db

  // the chunk of key tile t (CHUNKED): lines and scale words of all D rows
  auto fetch_chunk = [&](int t) {
    const int chunk = t >> 3;
#pragma unroll
    for (int u = 0; u < D / 8; ++u)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(v_rsrc, (lds_ptr_t)(v_lines + u * 1024), 16, (u & 1) ? v_gather1 : v_gather0,
                                               u * 8 * v_row_bytes + chunk * 128, 0, 0);
#pragma unroll
    for (int q = 0; q < kScaleParts; ++q)
#pragma unroll
      for (int k = 0; k < D / 64; ++k)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(vs_rsrc, (lds_ptr_t)(v_scale_words + (q * D + 64 * k) * 4), 4,
                                                 lane * vs_row_bytes,
                                                 64 * k * vs_row_bytes + chunk * (kScaleParts * 4) + q * 4, 0, 0);
  };

  // Everything the first tile needs is requested at once: the query, the K rows, V.
  RowPiece<D> kp, query;
  VPiece vp[CHUNKED ? 1 : kRowBlocks];
  load_row_piece<D, ASYM>(Qc, Qs, ((int64_t)g * per + (col_valid ? col / Sq : 0)) * Sq + qi, h, query);
  if (t0 < t1) {
    load_row_piece<D, ASYM>(Kc, Ks, krow0 + (int64_t)t0 * 32, h, kp);
    if constexpr (CHUNKED) {
      fetch_chunk(t0);
    } else {
#pragma unroll
      for (int db = 0; db < kRowBlocks; ++db) load_v_piece<ASYM>(Vc, Vs, vrow0 + db * 32, Sk, t0, vp[db]);
    }
  }
  // this column's query as the B operand of the first product, resident in registers (zeros in a padding column)
  u32x4 qf[kSteps];
#pragma unroll
  for (int s = 0; s < kSteps; ++s) {
    qf[s] = decode_step<SCALE_KIND, ASYM, D>(query, s);
    if (!col_valid) qf[s] = u32x4{0, 0, 0, 0};
  }
  for (int t = t0; t < t1; ++t) {
    if constexpr (CHUNKED) {
      if (t != t0 && (t & 7) == 0) {
        // the wave is done with the previous chunk (its reads have returned): fetch the chunk of tile t
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        fetch_chunk(t);
      }
      if (t == t0 || (t & 7) == 0) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    // CHUNKED: the tile's 16 bytes of V^T rows 32 db + col and the rows' scale bytes for it. They are taken out of LDS here,
    // before the next K rows are requested: the compiler waits for everything in flight before it reads LDS that
    // direct-to-LDS loads write, and further down that would be the K rows (4 sequences x 8192 keys: 24.1 -> 23.6 us).
    uint4 v_codes[CHUNKED ? kRowBlocks : 1];
    uint32_t v_scales[CHUNKED ? kRowBlocks : 1];
    if constexpr (CHUNKED) {
      const int tj = t & 7;
#pragma unroll
      for (int db = 0; db < kRowBlocks; ++db) {
        const int row = db * 32 + col;
        v_codes[db] = *reinterpret_cast<const uint4*>(v_lines + row * 128 + ((tj ^ v_read_swz) << 4));
        if constexpr (ASYM)
          v_scales[db] = *reinterpret_cast<const uint16_t*>(v_scale_words + ((tj >> 1) * D + row) * 4 + (tj & 1) * 2);
        else
          v_scales[db] = v_scale_words[((tj >> 2) * D + row) * 4 + (tj & 3)];
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    // the next tile's bytes are requested before this tile's arithmetic
    RowPiece<D> kn = kp;
    VPiece vn[CHUNKED ? 1 : kRowBlocks];
    if constexpr (!CHUNKED) {
#pragma unroll
      for (int db = 0; db < kRowBlocks; ++db) vn[db] = vp[db];
    }
    if (t + 1 < t1) {
      load_row_piece<D, ASYM>(Kc, Ks, krow0 + (int64_t)(t + 1) * 32, h, kn);
      if constexpr (!CHUNKED) {
#pragma unroll
        for (int db = 0; db < kRowBlocks; ++db) load_v_piece<ASYM>(Vc, Vs, vrow0 + db * 32, Sk, t + 1, vn[db]);
      }
    }

    f32x16 s;
#pragma unroll
    for (int v = 0; v < 16; ++v) s[v] = 0.f;
#pragma unroll
    for (int ks = 0; ks < kSteps; ++ks) {
      const u32x4 a = decode_step<SCALE_KIND, ASYM, D>(kp, ks);
      s = decode_mfma<SCALE_KIND>(a, qf[ks], s);
    }
    const bool masked = causal && t * 32 + 31 > off;  // some key of the tile is masked for the first query (uniform)
    AMX_ATTENTION_TILE_PROBS(true, s, score_scale, masked, t * 32 + row_in_tile, limit, m, l, pb, alpha, kF16)
    if (__builtin_amdgcn_ballot_w64(alpha != 1.0f) != 0) {  // the maximum moved for some query: rescale
#pragma unroll
      for (int db = 0; db < kRowBlocks; ++db)
#pragma unroll
        for (int v = 0; v < 16; ++v) o[db][v] *= alpha;
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const u32x4 b = {pb[4 * j], pb[4 * j + 1], pb[4 * j + 2], pb[4 * j + 3]};
#pragma unroll
      for (int db = 0; db < kRowBlocks; ++db) {
        const uint4 c = CHUNKED ? v_codes[CHUNKED ? db : 0] : vp[CHUNKED ? 0 : db].codes;
        const uint32_t sc = CHUNKED ? v_scales[CHUNKED ? db : 0] : vp[CHUNKED ? 0 : db].scales;
        const uint32_t w0 = j ? c.z : c.x, w1 = j ? c.w : c.y, vsp = sc & 255u, vsn = ASYM ? sc >> 8 : vsp;
        const u32x4 a = decode_word<SCALE_KIND, ASYM>(__builtin_amdgcn_perm(w1, w0, pick), vsp, vsn);
        o[db] = decode_mfma<SCALE_KIND>(a, b, o[db]);
      }
    }
    kp = kn;
    if constexpr (!CHUNKED) {
#pragma unroll
      for (int db = 0; db < kRowBlocks; ++db) vp[db] = vn[db];
    }
  }

  // register 4c + r of row block db is d = 32 db + 8 c + 4 h + r of column col
  if (!col_valid) return;
  float* dst = part + (((int64_t)g * kDecodeCols + col) * nsplits + split) * (D + 2);
  const float unbias = kF16 ? 0.03125f : 1.0f;  // 2^-5, exact
#pragma unroll
  for (int db = 0; db < kRowBlocks; ++db)
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      float* d4 = dst + db * 32 + c * 8 + 4 * h;
      d4[0] = o[db][4 * c] * unbias, d4[1] = o[db][4 * c + 1] * unbias, d4[2] = o[db][4 * c + 2] * unbias,
      d4[3] = o[db][4 * c + 3] * unbias;
    }
  if (h == 0) dst[D] = m, dst[D + 1] = l;
}

// Over all lanes of a wave: rotations within rows of 16 lanes, then the rows (lane exchanges through LDS took as long as the loads).
template <typename Op>
__device__ __forceinline__ float over_wave(float v, Op op) {
  v = op(v, u2f((uint32_t)__builtin_amdgcn_update_dpp(0, (int)f2u(v), 0x128, 0xF, 0xF, false)));  // row_ror:8
  v = op(v, u2f((uint32_t)__builtin_amdgcn_update_dpp(0, (int)f2u(v), 0x124, 0xF, 0xF, false)));
  v = op(v, u2f((uint32_t)__builtin_amdgcn_update_dpp(0, (int)f2u(v), 0x122, 0xF, 0xF, false)));
  v = op(v, u2f((uint32_t)__builtin_amdgcn_update_dpp(0, (int)f2u(v), 0x121, 0xF, 0xF, false)));
  const auto a = __builtin_amdgcn_permlane16_swap(f2u(v), f2u(v), false, false);
  v = op(u2f(a[0]), u2f(a[1]));
  const auto b = __builtin_amdgcn_permlane32_swap(f2u(v), f2u(v), false, false);
  return op(u2f(b[0]), u2f(b[1]));
}

// W waves per (kv head, column that holds a query): the exact combination of the ranges, in FP32. Each wave works out the
// maximum and the ranges' weights 2^(m_c - m*), a range to a lane (0 for a range in which the query saw no key), and adds up every
// W-th range's row, a weight read from its lane. It is a chain of memory latencies, so the first W F ranges' rows (F to a wave,
// D / 64 floats a lane of each) are requested before anything is known about their weights, and with four waves further ones 64 at a time.
// Four waves of 16, as one wave with 32 rows in flight and lane exchanges through LDS / this: 64 ranges, 32 columns 5.3 -> 2.9 us; the
// whole call of one sequence x 8192 keys 11.3 -> 9.9, of four (32 ranges) 16.5 -> 15.6, 256 ranges 31.5 -> 19.0. Up to 16 ranges one
// wave has them all: with thousands of columns four are waves for nothing (the whole call, us, one wave and exchanges / four waves / this:
// 256 heads of 32 columns, 4 ranges 26.1 / 31.8 / 19.2; 192 of 16, 16 ranges 31.2 / 26.8 / 24.7; 8 of 4, 4 ranges 11.3 / 6.5 / 6.2).
template <int D, int W, int F>
__global__ __launch_bounds__(64 * W) void attention_decode_combine_kernel(const float* __restrict__ part, float* __restrict__ out, int per,
                                                                          int Sq, int nsplits) {
  typedef float row_t __attribute__((ext_vector_type(D / 64)));
  static_assert(W * F <= 64);  // (nsplits <= F unless W F = 64)
  __shared__ float sums[W * D];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), col = (int)blockIdx.x, g = (int)blockIdx.y;
  const float* base = part + ((int64_t)g * kDecodeCols + col) * nsplits * (D + 2);
  row_t rows[F];
  auto request = [&](int c0) {  // (past the last range: the last one again, not used)
#pragma unroll
    for (int i = 0; i < F; ++i)
      rows[i] = *reinterpret_cast<const row_t*>(base + (int64_t)min(c0 + wave + W * i, nsplits - 1) * (D + 2) + lane * (D / 64));
  };
  // maximum and sum of range c0 + lane (none: a range without a key)
  auto range_of = [&](int c0) {
    const float2 ml = *reinterpret_cast<const float2*>(base + (int64_t)min(c0 + lane, nsplits - 1) * (D + 2) + D);
    return c0 + lane < nsplits ? ml : make_float2(0.f, 0.f);
  };
  float2 ml = range_of(0);
  request(0);
  float mx = ml.y > 0.f ? ml.x : -__builtin_inff();
  for (int c0 = 64; c0 < nsplits; c0 += 64) {
    const float2 more = range_of(c0);
    if (more.y > 0.f) mx = fmaxf(mx, more.x);
  }
  mx = over_wave(mx, [](float a, float b) { return fmaxf(a, b); });
  float den = 0.f;
  row_t num;
#pragma unroll
  for (int e = 0; e < D / 64; ++e) num[e] = 0.f;
  for (int c0 = 0; c0 < nsplits; c0 += 64) {
    if (c0 != 0) {
      ml = range_of(c0);
      request(c0);
    }
    const float w = ml.y > 0.f ? __builtin_amdgcn_exp2f(ml.x - mx) : 0.f;
    den += w * ml.y;
#pragma unroll
    for (int i = 0; i < F; ++i) {
      const float weight = u2f((uint32_t)__builtin_amdgcn_readlane((int)f2u(w), wave + W * i));
      const bool there = c0 + wave + W * i < nsplits;  // (a weight of 0 would make NaN of an infinity in the last range's row)
#pragma unroll
      for (int e = 0; e < D / 64; ++e) num[e] += weight * (there ? rows[i][e] : 0.f);
    }
  }
  const float inv = 1.0f / over_wave(den, [](float a, float b) { return a + b; });
  float* dst = out + (((int64_t)g * per + col / Sq) * Sq + col % Sq) * D;
  if constexpr (W == 1) {
    *reinterpret_cast<row_t*>(dst + lane * (D / 64)) = num * inv;
  } else {
    *reinterpret_cast<row_t*>(sums + wave * D + lane * (D / 64)) = num;
    __syncthreads();
    if (tid < D) dst[tid] = ((sums[tid] + sums[D + tid]) + (sums[2 * D + tid] + sums[3 * D + tid])) * inv;
  }
}

bool attention_decode_supported(int64_t Hq, int64_t Hkv, int64_t Sq, int64_t head_dim) {
  return Hkv > 0 && Hq % Hkv == 0 && (Hq / Hkv) * Sq <= kDecodeCols && (head_dim == 128 || head_dim == 64);
}

size_t attention_decode_workspace_bytes(int64_t Hkv, int64_t head_dim, int64_t key_splits) {
  return (size_t)(Hkv * key_splits * kDecodeCols * (head_dim + 2) * 4);
}

template <int SK, bool ASYM, int D>
static hipError_t launch_decode(int64_t Hq, int64_t Hkv, int64_t Sq, int64_t Sk, const uint8_t* Qc, const uint8_t* Qs,
                                const uint8_t* Kc, const uint8_t* Ks, const uint8_t* Vc, const uint8_t* Vs, float scale,
                                int causal, int splits, float* out, float* part, hipStream_t s) {
  const int per = (int)(Hq / Hkv), tiles = (int)(Sk / 32), tiles_per_split = (tiles + splits - 1) / splits;
  hipError_t e;
  if (attention_decode_16_preferred(Hq, Hkv, Sq, D, tiles_per_split, splits)) {
    e = launch_attention_decode_16(SK, ASYM, Hq, Hkv, Sq, Sk, D, Qc, Qs, Kc, Ks, Vc, Vs, scale, causal, splits, part, s);
  } else {
    // whole chunks of 8 key tiles, and V^T of one head within the 32-bit offsets of a buffer: V through LDS by chunks
    if (Sk % 256 == 0 && Sk <= (1 << 24))
      hipLaunchKernelGGL((attention_decode_kernel<SK, ASYM, D, true>), dim3((unsigned)splits, (unsigned)Hkv), dim3(64), 0, s,
                         Qc, Qs, Kc, Ks, Vc, Vs, part, (int)Sq, (int)Sk, per, tiles_per_split,
                         scale * 1.4426950408889634f, causal);
    else
      hipLaunchKernelGGL((attention_decode_kernel<SK, ASYM, D, false>), dim3((unsigned)splits, (unsigned)Hkv), dim3(64), 0, s,
                         Qc, Qs, Kc, Ks, Vc, Vs, part, (int)Sq, (int)Sk, per, tiles_per_split,
                         scale * 1.4426950408889634f, causal);
    e = hipGetLastError();
  }
  if (e != hipSuccess) return e;
  auto combine = [&]<int W, int F>() {
    hipLaunchKernelGGL((attention_decode_combine_kernel<D, W, F>), dim3((unsigned)(per * Sq), (unsigned)Hkv), dim3(64 * W), 0, s, part, out,
                       per, (int)Sq, splits);
  };
  if (splits <= 4)
    combine.template operator()<1, 4>();
  else if (splits <= 16)
    combine.template operator()<1, 16>();
  else
    combine.template operator()<4, 16>();
  return hipGetLastError();
}

hipError_t launch_attention_decode(int scale_kind, bool asym, int64_t Hq, int64_t Hkv, int64_t Sq, int64_t Sk,
                                   int64_t head_dim, const uint8_t* Q_codes, const uint8_t* Q_scales,
                                   const uint8_t* K_codes, const uint8_t* K_scales, const uint8_t* V_codes,
                                   const uint8_t* V_scales, float scale, int causal, int key_splits, float* out,
                                   void* workspace, hipStream_t s) {
  float* part = reinterpret_cast<float*>(workspace);
  auto go = [&]<int SK, bool ASYM>() {
    if (head_dim == 128)
      return launch_decode<SK, ASYM, 128>(Hq, Hkv, Sq, Sk, Q_codes, Q_scales, K_codes, K_scales, V_codes, V_scales, scale,
                                          causal, key_splits, out, part, s);
    return launch_decode<SK, ASYM, 64>(Hq, Hkv, Sq, Sk, Q_codes, Q_scales, K_codes, K_scales, V_codes, V_scales, scale,
                                       causal, key_splits, out, part, s);
  };
  switch (scale_kind) {
    case kScaleE5M2: return asym ? go.template operator()<kScaleE5M2, true>() : go.template operator()<kScaleE5M2, false>();
    case kScaleE4M3: return asym ? go.template operator()<kScaleE4M3, true>() : go.template operator()<kScaleE4M3, false>();
    case kScaleE8M0Floor:
      return asym ? go.template operator()<kScaleE8M0Floor, true>() : go.template operator()<kScaleE8M0Floor, false>();
    case kScaleE8M0Round:
      return asym ? go.template operator()<kScaleE8M0Round, true>() : go.template operator()<kScaleE8M0Round, false>();
    default: return hipErrorInvalidValue;
  }
}

}  // namespace amx
