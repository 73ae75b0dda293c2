// Fused quantized attention: out = softmax(scale * Q_hat . K_hat^T) . V_hat with both products on quantized operands
// (Sec. 5.1 quantizes Q.K^T and the attention map times V) and the attention map never written to memory, for heads of 128
// dimensions (the kernel of heads of 64 is in attention_64.hip; the launch of both is here): the scores
// of one tile of 32 keys become un-normalised probabilities against the running row maximum (online softmax), the
// tile of probabilities is cast as ONE group per query along the keys (the same element and scale format as the
// operands; FP32 values go into the cast), multiplied with the V tile, and the row sum divides at the end.
//
// The scores are computed transposed so that no data has to change lanes between the two products:
//   S^T[key, query] = K_tile[32 keys x D] . Q^T[D x 32 queries]   (MFMA 32x32x16 BF16, A = K rows, B = Q rows)
//   O[query, d]    += P[32 queries x 32 keys] . V[32 keys x d]    (A = the probabilities, B = V^T rows)
// In a 32x32 accumulator lane l holds column l % 32 (of S^T: one query) and rows 8c + 4(l/32) + r (c, r = 0..3) in register
// 4c + r: all 32 keys of a query sit in the two lanes l and l ^ 32, so the row maximum, the row sum and the group
// maximum of the cast are 16 in-lane steps and one exchange, and registers 8j .. 8j+7 of S^T, converted to BF16, are
// already the A operand of k-step j of the second product, provided V^T was staged with its keys in that order
// (expand_kv_kernel). The queries are the rows of O, its registers: where the running maximum of a query moves, only the
// registers of its eight rows are multiplied (with the queries in the lanes it was all 64, in half of the tiles: 11 % of the
// kernel), by a factor that comes from the query's lane through LDS, behind the exponentials. Workgroup = kAttnWaves waves x
// 32 queries; the K and V fragments of a key tile are brought into LDS once per workgroup by direct-to-LDS loads.
#include "../../include/amxfp4.h"
#include "attention_tile.h"
#include "cast_math.h"
#include "dequant_regs.h"
#include "gemm_common.h"

namespace amx {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
// Waves per workgroup, 32 queries each. A wave's work on a tile is one long dependent chain (fragment reads -> eight
// chained MFMAs -> maximum, exponentials, sum, cast -> MFMAs), about 1 us where it has a SIMD to itself, and the barrier of a
// workgroup keeps its waves in the same phase of it, so what hides the chain's latencies is waves of OTHER workgroups on the
// same SIMD (of one wave, vector instructions and MFMAs add up; of three, an MFMA of 32 cycles is free beside 16 vector
// instructions): four waves per workgroup and a register budget of a third of the file put three workgroups on a compute
// unit. A grid that does not fill these is bound by the chain: there the kernel walks over pairs of key tiles with half of the
// register file, two workgroups to a compute unit, so that the latencies are paid once for two tiles (pairs_pay()).
constexpr int kAttnWaves = 4;
constexpr int kAttnQ = 32 * kAttnWaves;     // queries per workgroup
constexpr int kAttnD = 128;                 // the head dimension

// A key tile is kAttnD / 16 K fragments (one per 16 of D) and as many V^T fragments (D / 32 row blocks x 2 k-steps), dealt
// over the waves. All fragments of a product's operand are requested before its first MFMA (two at a time, as the compiler had
// them, each pair waited out its trip to LDS).
template <int SCALE_KIND, bool PAIRS>
__global__ __launch_bounds__(64 * kAttnWaves) __attribute__((amdgpu_waves_per_eu(PAIRS ? 2 : 3, PAIRS ? 2 : 3))) void attention_fused_kernel(
    const uint8_t* __restrict__ Q_codes, const uint8_t* __restrict__ Q_scales, int asym, const uint16_t* __restrict__ Kp,
    const uint16_t* __restrict__ Vp, float* __restrict__ out, int Sq, int Sk, int Sqp, int Skv, int kv_group,
    float scale_log2, int causal, int merged_bf16) {
  // FP8-E5M2 scales: the second product runs on FP16 operands. The cast leaves the probabilities as FP16 times 2^8
  // (the scale byte is the upper byte of an FP16: a conversion and a packed multiply per pair instead of a conversion,
  // two multiplies and a permute), V^T comes as an FP16 panel biased by 2^-3, and the 2^5 is taken out with the row
  // sum at the end. Same values, same sums.
  constexpr bool kPF16 = SCALE_KIND == kScaleE5M2;
  constexpr int kAttnKFrags = kAttnD / 16, kAttnVFrags = (kAttnD / 32) * 2;
  static_assert(kAttnKFrags == kAttnVFrags && kAttnKFrags % kAttnWaves == 0, "fragments must divide over the waves");
  constexpr int kStageBytes = (kAttnKFrags + kAttnVFrags) * kFragBytes;
  __shared__ __attribute__((aligned(1024))) uint8_t lds[3 * kStageBytes];
  __shared__ __attribute__((aligned(16))) float alphas[kAttnWaves][2][32];  // a wave's own: no barrier

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // Workgroups are dealt to the 8 XCDs round-robin by their linear id (x fastest). x walks the query heads, so every
  // XCD gets the same mix of light and heavy query blocks of a causal problem, and (when the head count is a multiple
  // of 8) a contiguous range of heads, i.e. heads that share a key/value head share an L2. y walks the query blocks,
  // last block first: under a causal mask those have the most key tiles and should start first.
  const int nheads = (int)gridDim.x;
  const int h = (nheads & 7) == 0 ? (int)(blockIdx.x & 7) * (nheads >> 3) + (int)(blockIdx.x >> 3) : (int)blockIdx.x;
  const int g = h / kv_group;
  const int qblock = (int)(gridDim.y - 1 - blockIdx.y);
  const int q0 = qblock * kAttnQ, qw = q0 + wave * 32;
  const int off = Sk - Sq;  // causal: query i sees keys <= i + off
  const bool wave_active = qw < Sqp;

  // key tiles this workgroup / this wave walks over (uniform)
  const int tiles_all = Sk / 32;
  const int last_q_block = (q0 + kAttnQ < Sqp ? q0 + kAttnQ : Sqp) - 1;
  const int nt = causal ? min(tiles_all, (last_q_block + off) / 32 + 1) : tiles_all;
  const int nt_wave = !wave_active ? 0 : (causal ? min(tiles_all, (qw + 31 + off) / 32 + 1) : tiles_all);

  // K panel of this key/value head: tile t = 8 contiguous fragments; V^T panel: 4 row blocks of Skv / 16 fragments
  // (Skv = Sk rounded up to the panel's K granularity of 64). Raw buffers: reads past the end return zero.
  const int64_t kfrags_head = (int64_t)tiles_all * kAttnKFrags, vfrags_head = (int64_t)(kAttnD / 32) * (Skv / 16);
  const uint8_t* Kbase = reinterpret_cast<const uint8_t*>(Kp) + g * kfrags_head * kFragBytes;
  const uint8_t* Vbase = reinterpret_cast<const uint8_t*>(Vp) + g * vfrags_head * kFragBytes;
  auto window = [](const uint8_t* base, int64_t bytes) {
    const uint64_t p = reinterpret_cast<uint64_t>(base);
    return u32x4{(uint32_t)p, (uint32_t)(p >> 32), (uint32_t)bytes, 0x00020000u};
  };
  const u32x4 Kr = window(Kbase, kfrags_head * kFragBytes), Vr = window(Vbase, vfrags_head * kFragBytes);
  const int lane_off = lane * 16;

  // Loads of the key tiles' fragments, dealt over the waves: wave w brings fragments w, w + kAttnWaves, .. of a tile (or of a
  // pair of tiles). They are written out so that the compiler, which cannot tell the stages of a ring apart, does not wait
  // for the newest of them in front of every fragment read; they write no registers, and the loops below wait by count.
  // `past`: 0, or an offset beyond any panel, which brings zeros without a trip to memory.
  constexpr int kLoads = (kAttnKFrags + kAttnVFrags) / kAttnWaves;  // of a wave and key tile
  constexpr uint32_t kPast = 0x80000000u;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_ptr_t)lds;
  // (m0 is a reserved register: that the compiler does not keep it across the statement, of which it warns, is what is meant)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
  auto load_fragment = [&](const u32x4& window, uint32_t to, uint32_t offset) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                 :: "s"(to), "v"(lane_off), "s"(window), "s"(offset) : "memory", "m0");
  };
#pragma clang diagnostic pop
  auto load_k = [&](int tile, uint32_t to, int i, uint32_t past) {  // number i of this wave's; a pair's two tiles are adjacent
    const int f = wave + kAttnWaves * i;
    load_fragment(Kr, to + f * kFragBytes, past | (uint32_t)((tile * kAttnKFrags + f) * kFragBytes));
  };
  auto load_v = [&](int tile, uint32_t to, int i, uint32_t past) {  // fragment f: row block f / 2, k-step f % 2
    const int n = wave + kAttnWaves * i, f = n % kAttnVFrags;
    load_fragment(Vr, to + n * kFragBytes,
                  past | (uint32_t)(((f >> 1) * (Skv / 16) + (f & 1) + 2 * (tile + n / kAttnVFrags)) * kFragBytes));
  };

  // this wave's 32 queries as the B operand of the first product: 8 k-steps over D, resident in registers. They are
  // dequantized here, once, from their codes (BF16: element * scale has at most 6 significant bits); expanding Q to a
  // panel first was a pass over memory and a launch (32 heads x 4064: 9 us of the call). Rows past Sq repeat the last one.
  bf16x8 qf[kAttnKFrags];
  {
    const int q = qw + (lane & 31) < Sq ? qw + (lane & 31) : Sq - 1;
    const int64_t row = (int64_t)h * Sq + q;
    const u32x4* codes = reinterpret_cast<const u32x4*>(Q_codes + row * (kAttnD / 2));
    const uint8_t* sb = Q_scales + row * (kAttnD / 32) * (asym ? 2 : 1);
#pragma unroll
    for (int g = 0; g < kAttnD / 32; ++g) {  // a group of 32: k-steps 2 g and 2 g + 1; lane half h takes words h, 2 + h
      const u32x4 w = codes[g];
      const uint32_t bp = sb[asym ? 2 * g : g], bn = asym ? sb[2 * g + 1] : bp;
      const uint32_t s_pos = f2u(scale_value<SCALE_KIND>(bp)), s_neg = f2u(scale_value<SCALE_KIND>(bn));
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const uint32_t word = (lane >> 5) ? w[2 * k + 1] : w[2 * k];
        qf[2 * g + k] = __builtin_bit_cast(
            bf16x8, u32x4{dequant2_f32<true, 0>(word, s_pos, s_neg), dequant2_f32<true, 1>(word, s_pos, s_neg),
                          dequant2_f32<true, 2>(word, s_pos, s_neg), dequant2_f32<true, 3>(word, s_pos, s_neg)});
      }
    }
  }

  f32x16 o[kAttnD / 32];
#pragma unroll
  for (int db = 0; db < kAttnD / 32; ++db)
#pragma unroll
    for (int v = 0; v < 16; ++v) o[db][v] = 0.f;
  float m = -__builtin_inff(), l = 0.f;  // running maximum (scaled score, in units of log2) and sum of this lane's query
  const int limit = causal ? qw + (lane & 31) + off : Sk - 1;  // last key this lane's query may attend to
  const int first_limit = causal ? qw + off : Sk - 1;         // the smallest of the wave's
  const int row_in_tile = 4 * (lane >> 5);                    // key of register v: 8 (v / 4) + row_in_tile + v % 4

  // o *= alpha by accumulator row, where the maximum moved: MOVED has a bit per query, AL the factors of the lane's rows
#define AMX_ATTN_RESCALE(MOVED, AL)                                                                                \
  if ((MOVED) != 0) {                                                                                              \
    _Pragma("unroll") for (int c = 0; c < 4; ++c) {                                                                \
      if ((MOVED) & (0xFFu << (8 * c))) { /* uniform: rows 8 c .. 8 c + 7 */                                       \
        asm volatile(""); /* (keeps the branch: without it all rows are multiplied and selected) */                \
        _Pragma("unroll") for (int db = 0; db < kAttnD / 32; ++db) {                                               \
          o[db][4 * c] *= (AL)[c].x, o[db][4 * c + 1] *= (AL)[c].y;                                                \
          o[db][4 * c + 2] *= (AL)[c].z, o[db][4 * c + 3] *= (AL)[c].w;                                            \
        }                                                                                                          \
      }                                                                                                            \
    }                                                                                                              \
  }
  // the factors of the lane's accumulator rows from those of the queries, through LDS of the wave's own
#define AMX_ATTN_BY_ROW(AL, ALPHA, SLOT)                                                                           \
  float4 AL[4];                                                                                                    \
  alphas[wave][SLOT][lane & 31] = (ALPHA);                                                                         \
  _Pragma("unroll") for (int c = 0; c < 4; ++c) AL[c] = *reinterpret_cast<const float4*>(&alphas[wave][SLOT][8 * c + row_in_tile]);
#define AMX_ATTN_PV(P, VF, J, STEP) /* k-step J: registers 4 J .. of the probabilities, V fragments J, STEP + J, .. */ \
  {                                                                                                                \
    const u32x4 p = {(P)[4 * (J)], (P)[4 * (J) + 1], (P)[4 * (J) + 2], (P)[4 * (J) + 3]};                          \
    _Pragma("unroll") for (int db = 0; db < kAttnD / 32; ++db) {                                                   \
      const u32x4 v = (VF)[(STEP) * db + (J)];                                                                     \
      if constexpr (kPF16)                                                                                         \
        o[db] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, p), __builtin_bit_cast(f16x8, v), \
                                                       o[db], 0, 0, 0);                                            \
      else                                                                                                         \
        o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, p), __builtin_bit_cast(bf16x8, v), \
                                                        o[db], 0, 0, 0);                                           \
    }                                                                                                              \
  }

  if constexpr (PAIRS) {
    // K of a pair of tiles in one slot, V in two: V(t + 2) is requested when pair t starts, K(t + 2) when its scores are
    // done; two barriers to a pair.
    constexpr uint32_t kPairV = 2 * kAttnVFrags * kFragBytes;
    uint32_t v_now = 2 * kAttnKFrags * kFragBytes, v_next = v_now + kPairV;
#pragma unroll
    for (int i = 0; i < kLoads; ++i) load_k(0, lds0, i, 0u);
#pragma unroll
    for (int i = 0; i < kLoads; ++i) load_v(0, lds0 + v_now, i, 0u);
    for (int t = 0; t < nt; t += 2) {
      __builtin_amdgcn_s_waitcnt(0x0070);  // vmcnt(0) lgkmcnt(0)
      AMX_BARRIER();
      const uint32_t past = t + 2 < nt ? 0u : kPast;
#pragma unroll
      for (int i = 0; i < kLoads; ++i) load_v(t + 2, lds0 + v_next, i, past);
      const bool active = t < nt_wave;  // uniform
      f32x16 s[2];
      if (active) {
        bf16x8 kf[2][kAttnKFrags];  // all requested before the first is used
#pragma unroll
        for (int kb = 0; kb < kAttnKFrags; ++kb)
#pragma unroll
          for (int i = 0; i < 2; ++i)
            kf[i][kb] = *reinterpret_cast<const bf16x8*>(lds + (i * kAttnKFrags + kb) * kFragBytes + lane_off);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int v = 0; v < 16; ++v) s[i][v] = 0.f;
#pragma unroll
        for (int kb = 0; kb < kAttnKFrags; ++kb)
#pragma unroll
          for (int i = 0; i < 2; ++i) s[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[i][kb], qf[kb], s[i], 0, 0, 0);
      }
      __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
      AMX_BARRIER();                       // every wave is past its reads of K
#pragma unroll
      for (int i = 0; i < kLoads; ++i) load_k(t + 2, lds0, i, past);
      if (active) {
        // AMX_ATTENTION_TILE_MAX and _EXP for both tiles at a time: the second one's maximum follows the first one's
        float x[2][16], mx[2];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int v = 0; v < 16; ++v) x[i][v] = s[i][v] * scale_log2;
        if (t * 32 + 63 > first_limit) {  // uniform: some key of the pair is masked for some query, or past the last one
#pragma unroll
          for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v)
              if ((t + i) * 32 + row_in_tile + 8 * (v >> 2) + (v & 3) > limit) x[i][v] = -__builtin_inff();
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          mx[i] = -__builtin_inff();
#pragma unroll
          for (int v = 0; v < 16; ++v) mx[i] = fmaxf(mx[i], x[i][v]);
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) mx[i] = fmaxf(mx[i], __shfl_xor(mx[i], 32, 64));
        const float m0 = fmaxf(m, mx[0]), m1 = fmaxf(m0, mx[1]);
        const float alpha0 = __builtin_amdgcn_exp2f(m - m0), alpha1 = __builtin_amdgcn_exp2f(m0 - m1);
        AMX_ATTN_BY_ROW(al0, alpha0, 0)
        AMX_ATTN_BY_ROW(al1, alpha1, 1)
        const uint32_t moved0 = (uint32_t)__builtin_amdgcn_ballot_w64(alpha0 != 1.0f);
        const uint32_t moved1 = (uint32_t)__builtin_amdgcn_ballot_w64(alpha1 != 1.0f);
        float psum[2] = {0.f, 0.f}, pmax[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const float mi = i ? m1 : m0;
          pmax[i] = __builtin_amdgcn_exp2f(mx[i] - mi);
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            x[i][v] = __builtin_amdgcn_exp2f(x[i][v] - mi);
            psum[i] += x[i][v];
          }
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) psum[i] += __shfl_xor(psum[i], 32, 64);
        l = (l * alpha0 + psum[0]) * alpha1 + psum[1];
        m = m1;
        uint32_t pb0[8], pb1[8];
        AMX_ATTENTION_TILE_CAST(x[0], pmax[0], pb0, kPF16)
        AMX_ATTENTION_TILE_CAST(x[1], pmax[1], pb1, kPF16)
        u32x4 vf[kAttnVFrags];
#pragma unroll
        for (int f = 0; f < kAttnVFrags; ++f) vf[f] = *reinterpret_cast<const u32x4*>(lds + v_now + f * kFragBytes + lane_off);
        AMX_ATTN_RESCALE(moved0, al0)
        AMX_ATTN_PV(pb0, vf, 0, 2)
        AMX_ATTN_PV(pb0, vf, 1, 2)
        if (t + 1 < nt_wave) {  // (otherwise all its probabilities are 0)
#pragma unroll
          for (int f = 0; f < kAttnVFrags; ++f)
            vf[f] = *reinterpret_cast<const u32x4*>(lds + v_now + (kAttnVFrags + f) * kFragBytes + lane_off);
          AMX_ATTN_RESCALE(moved1, al1)
          AMX_ATTN_PV(pb1, vf, 0, 2)
          AMX_ATTN_PV(pb1, vf, 1, 2)
        }
      }
      const uint32_t other = v_now;
      v_now = v_next;
      v_next = other;
    }
  } else {
    // Three stages of (K tile, V tile): tile t + 2 is requested during tile t, piece by piece, into the stage of t - 1. Past
    // the last tile the loads bring zeros instead of being skipped: a branch around each of them cost 5 %.
    static_assert(kLoads == 4, "places of the loads in a tile");
#pragma unroll
    for (int st = 0; st < 2; ++st)
#pragma unroll
      for (int i = 0; i < kLoads / 2; ++i) {
        load_k(st, lds0 + st * kStageBytes, i, st < nt ? 0u : kPast);
        load_v(st, lds0 + st * kStageBytes + kAttnKFrags * kFragBytes, i, st < nt ? 0u : kPast);
      }
    uint32_t stage = 0, free_stage = 2 * kStageBytes;
    for (int t = 0; t < nt; ++t) {
      // tile t has landed (t + 1 stays in flight), and every wave is past tile t - 1
      __builtin_amdgcn_s_waitcnt(0x0070 | kLoads);  // vmcnt(kLoads) lgkmcnt(0)
      AMX_BARRIER();
      const uint32_t past = t + 2 < nt ? 0u : kPast, to = lds0 + free_stage;
      const uint8_t* cur = lds + stage;
      if (t < nt_wave) {
        f32x16 s;
#pragma unroll
        for (int v = 0; v < 16; ++v) s[v] = 0.f;
        bf16x8 kf[kAttnKFrags];  // all requested before the first is used
#pragma unroll
        for (int kb = 0; kb < kAttnKFrags; ++kb) kf[kb] = *reinterpret_cast<const bf16x8*>(cur + kb * kFragBytes + lane_off);
        __builtin_amdgcn_sched_barrier(0);
        load_k(t + 2, to, 0, past);
        load_k(t + 2, to, 1, past);
#pragma unroll
        for (int kb = 0; kb < kAttnKFrags; ++kb) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[kb], qf[kb], s, 0, 0, 0);
        const bool masked = t * 32 + 31 > first_limit;  // some key of the tile is masked for some query
        AMX_ATTENTION_TILE_MAX(false, s, scale_log2, masked, t * 32 + row_in_tile, limit, m, alpha)
        AMX_ATTN_BY_ROW(al, alpha, 0)  // travels behind the exponentials
        const uint32_t moved = (uint32_t)__builtin_amdgcn_ballot_w64(alpha != 1.0f);
        __builtin_amdgcn_sched_barrier(0);
        load_v(t + 2, to + kAttnKFrags * kFragBytes, 0, past);
        AMX_ATTENTION_TILE_EXP(false, m, l, alpha)
        AMX_ATTN_RESCALE(moved, al)
        u32x4 vf[kAttnVFrags];
#pragma unroll
        for (int f = 0; f < kAttnVFrags; f += 2)
          vf[f] = *reinterpret_cast<const u32x4*>(cur + (kAttnKFrags + f) * kFragBytes + lane_off);
        __builtin_amdgcn_sched_barrier(0);
        uint32_t pb[8];
        AMX_ATTENTION_TILE_CAST(x, pmax, pb, kPF16)
        load_v(t + 2, to + kAttnKFrags * kFragBytes, 1, past);
#pragma unroll
        for (int f = 1; f < kAttnVFrags; f += 2)
          vf[f] = *reinterpret_cast<const u32x4*>(cur + (kAttnKFrags + f) * kFragBytes + lane_off);
        AMX_ATTN_PV(pb, vf, 0, 2)
        AMX_ATTN_PV(pb, vf, 1, 2)
      } else {
#pragma unroll
        for (int i = 0; i < kLoads / 2; ++i) {
          load_k(t + 2, to, i, past);
          load_v(t + 2, to + kAttnKFrags * kFragBytes, i, past);
        }
      }
      free_stage = stage;
      stage = stage == 2 * kStageBytes ? 0 : stage + kStageBytes;
    }
  }
  AMX_WAIT_VMCNT(0);  // nothing may still be writing this workgroup's LDS when it retires
#undef AMX_ATTN_RESCALE
#undef AMX_ATTN_PV

  // out[h][query][d] = O[query][d] / l; register 4c + r of column block db is query 8 c + 4 (lane / 32) + r, d = 32 db +
  // lane % 32.
  // merged_bf16: the same values rounded to BF16 and written token-major, out[query][h * D + d] (the layout the output
  // projection's cast reads: no head-merge pass over an FP32 copy); a lane packs the values of registers v and v + 1 and swaps
  // the pair with its neighbour's, of which the even one stores two columns of register v's row and the odd one the same two of
  // register v + 1's (swapped before they were rounded, twice the instructions: 0.5 us of a call of 96 tokens).
  // The stores go through a window of the wave's valid rows: rows past Sq fall outside it and are dropped, without a branch
  // around every store.
  if (!wave_active) return;
  // (the reciprocals by row through LDS at once: a lane exchange in front of every row's stores was one trip after the other, 0.8
  // us of a call of 96 tokens)
  AMX_ATTN_BY_ROW(inv, (kPF16 ? 0.03125f : 1.0f) / l, 0)
#undef AMX_ATTN_BY_ROW
  const int rows = Sq - qw < 32 ? Sq - qw : 32;
  if (merged_bf16) {
    const int odd = lane & 1, pitch = nheads * kAttnD * 2;
    const __amdgpu_buffer_rsrc_t window = __builtin_amdgcn_make_buffer_rsrc(
        reinterpret_cast<uint16_t*>(out) + ((int64_t)qw * nheads + h) * kAttnD, 0, (rows - 1) * pitch + kAttnD * 2, 0x00020000);
    const int lane_to = (row_in_tile + odd) * pitch + (lane & 30) * 2;
    const uint32_t pick = odd ? 0x03020706u : 0x05040100u;  // of (the neighbour's pair, one's own): which halves
#pragma unroll
    for (int v = 0; v < 16; v += 2) {
      const int qr = 8 * (v >> 2) + (v & 3);
      const float inv0 = v & 2 ? inv[v >> 2].z : inv[v >> 2].x, inv1 = v & 2 ? inv[v >> 2].w : inv[v >> 2].y;
#pragma unroll
      for (int db = 0; db < kAttnD / 32; ++db) {
        const uint32_t own = pack2(o[db][v] * inv0, o[db][v + 1] * inv1);
        const uint32_t other = __builtin_amdgcn_mov_dpp(own, 0xB1 /* quad_perm 1 0 3 2 */, 0xF, 0xF, true);
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_amdgcn_perm(other, own, pick), window, lane_to + db * 64, qr * pitch, 0);
      }
      __builtin_amdgcn_sched_barrier(0);  // (all rows at once would spill)
    }
  } else {
    constexpr int kPitch = kAttnD * 4;
    const __amdgpu_buffer_rsrc_t window =
        __builtin_amdgcn_make_buffer_rsrc(out + ((int64_t)h * Sq + qw) * kAttnD, 0, rows * kPitch, 0x00020000);
    const int lane_to = row_in_tile * kPitch + (lane & 31) * 4;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int qr = 8 * (v >> 2) + (v & 3);
      const float inv_row = v & 2 ? (v & 1 ? inv[v >> 2].w : inv[v >> 2].z) : (v & 1 ? inv[v >> 2].y : inv[v >> 2].x);
#pragma unroll
      for (int db = 0; db < kAttnD / 32; ++db)
        __builtin_amdgcn_raw_buffer_store_b32(f2u(o[db][v] * inv_row), window, lane_to + db * 128, qr * kPitch, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

size_t attention_workspace_bytes(int64_t Hq, int64_t Hkv, int64_t Sq, int64_t Sk, int64_t head_dim) {
  return (size_t)((Hq * round_up(Sq, 32) + Hkv * Sk + Hkv * round_up(Sk, 64)) * head_dim * 2);
}

// Whether pairs of key tiles are the faster walk: up to 704 workgroups of a causal call, whose later query blocks start first
// and whose short ones fill up what is left, but only while all run at once, 512 of them, where they are of much the same
// length: without a mask, or with more than an eighth of the keys in front of the first query. Us per call, AMXFP4-E5M2, tile by
// tile / pairs, 32 / 8 heads, causal: 512 tokens 23.3 / 22.6, 1504 53.5 / 51.3, 2688 (672 workgroups) 93.1 / 87.5, 3008 (768)
// 114 / 119, 4064 180 / 197; without a mask, 40 / 8 heads x 1920 (600 workgroups) 101 / 118, 64 / 8 x 1344 (704) 77 / 89, up to
// 512 ratios of 0.95 to 1.01; 513 to 704 workgroups with 1.5 to 4 times the keys 1.08 to 1.25, with 1.25 times 0.95 to 1.12. An
// odd number of key tiles costs pairs a whole empty one, which up to nine of them is more than they save (96 keys: tile by tile
// 0.95 to 0.98 of the pairs' time).
bool pairs_pay(int64_t workgroups, int64_t Sq, int64_t Sk, int causal) {
  if ((Sk / 32) % 2 == 1 && Sk / 32 <= 9) return false;
  return workgroups <= (causal && 8 * (Sk - Sq) <= Sk ? 704 : 512);
}

template <int SK>
static hipError_t launch_attn(const uint8_t* Qc, const uint8_t* Qs, bool asym, const uint16_t* Kp, const uint16_t* Vp,
                              float* out, int64_t Hq, int64_t Hkv, int64_t Sq, int64_t Sk, float scale, int causal, int merged_bf16,
                              hipStream_t s) {
  const int64_t Sqp = round_up(Sq, 32);
  const dim3 grid((unsigned)Hq, (unsigned)((Sqp + kAttnQ - 1) / kAttnQ));
  auto go = [&]<bool PAIRS>() {
    hipLaunchKernelGGL((attention_fused_kernel<SK, PAIRS>), grid, dim3(64 * kAttnWaves), 0, s, Qc, Qs, asym ? 1 : 0,
                       Kp, Vp, out, (int)Sq, (int)Sk, (int)Sqp, (int)round_up(Sk, 64), (int)(Hq / Hkv),
                       scale * 1.4426950408889634f, causal, merged_bf16);
    return hipGetLastError();
  };
  return pairs_pay((int64_t)grid.x * grid.y, Sq, Sk, causal) ? go.template operator()<true>() : go.template operator()<false>();
}

hipError_t launch_attention_fused(int scale_kind, bool asym, int64_t Hq, int64_t Hkv, int64_t Sq, int64_t Sk,
                                  int64_t head_dim, const uint8_t* Q_codes, const uint8_t* Q_scales,
                                  const uint8_t* K_codes, const uint8_t* K_scales, const uint8_t* V_codes,
                                  const uint8_t* V_scales, float scale, int causal, float* out, bool merged_bf16,
                                  void* workspace, hipStream_t s, const KernelTimer& timer) {
  if (head_dim != 128 && head_dim != 64) return hipErrorInvalidValue;
  uint16_t* Kp = reinterpret_cast<uint16_t*>(workspace);
  uint16_t* Vp = Kp + Hkv * Sk * head_dim;
  // K: rows = tokens, K = head dimension; V^T: rows = head dimension, K = keys, in the accumulator's key order
  hipError_t e = launch_expand_kv(scale_kind, asym, K_codes, K_scales, Kp, V_codes, V_scales, Vp, Sk, head_dim, Hkv, s);
  if (e != hipSuccess) return e;
  if (timer.start && (e = hipEventRecord(timer.start, s)) != hipSuccess) return e;
  auto go = [&]<int SK>() {
    return launch_attn<SK>(Q_codes, Q_scales, asym, Kp, Vp, out, Hq, Hkv, Sq, Sk, scale, causal, merged_bf16, s);
  };
  if (head_dim == 64)
    e = launch_attention_64(scale_kind, asym, Hq, Hkv, Sq, Sk, Q_codes, Q_scales, Kp, Vp, scale, causal, out, merged_bf16, s);
  else
    switch (scale_kind) {
      case kScaleE5M2: e = go.template operator()<kScaleE5M2>(); break;
      case kScaleE4M3: e = go.template operator()<kScaleE4M3>(); break;
      case kScaleE8M0Floor: e = go.template operator()<kScaleE8M0Floor>(); break;
      case kScaleE8M0Round: e = go.template operator()<kScaleE8M0Round>(); break;
      default: return hipErrorInvalidValue;
    }
  if (e != hipSuccess) return e;
  if (timer.stop) e = hipEventRecord(timer.stop, s);
  return e;
}

}  // namespace amx
