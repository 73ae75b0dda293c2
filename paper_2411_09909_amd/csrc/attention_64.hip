// Fused quantized attention for heads of 64 dimensions: the arithmetic of attention.hip, whose arrangement is for heads of
// 128. Here the matrix products are half as long beside the same softmax and cast, so the vector instructions of a tile are
// most of it, and what hides the latencies of a wave's chain is many waves: this form, with both products transposed and two
// stages of tiles, needs 89 registers and 16 KiB of LDS, five workgroups to a compute unit. The other one, whose fragments are
// all requested ahead, needs 162 registers (240 for pairs of tiles): 32 / 8 heads, causal, AMXFP4-E5M2, us per call, this form /
// that one: 512 tokens 17.9 / 20.8, 1504 39.3 / 46.6, 2688 68.7 / 77.3, 4064 118 / 160, 8192 394 / 507; with the other's
// registers cut to 94 (five workgroups) 19.5, 43.4, 71.8, 117, 370.
//
//   S^T[key, query] = K_tile[32 keys x 64] . Q^T[64 x 32 queries]      (MFMA 32x32x16 BF16, A = K rows, B = Q rows)
//   O^T[d, query]  += V^T[d x 32 keys]     . P^T[32 keys x 32 queries] (A = V^T rows, B = the probabilities)
// In a 32x32 accumulator lane l holds column l % 32 (one query) and rows 8c + 4(l/32) + r (c, r = 0..3) in register 4c + r:
// registers 8j .. 8j+7 of S^T, converted, are the B operand of k-step j of the second product, with V^T staged in that key
// order (expand_kv_kernel). Workgroup = 4 waves x 32 queries; a key tile's 4 K and 4 V fragments are brought into LDS once per
// workgroup by direct-to-LDS loads, double buffered.
#include "../../include/amxfp4.h"
#include "attention_tile.h"
#include "cast_math.h"
#include "dequant_regs.h"
#include "gemm_common.h"
#include "kernels.h"

namespace amx {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
constexpr int kD = 64, kWaves = 4, kQueries = 32 * kWaves;  // of a head; waves and queries of a workgroup
constexpr int kFrags = kD / 16;                             // K fragments of a key tile, and V fragments: one of each per wave

template <int SCALE_KIND>
__global__ __launch_bounds__(64 * kWaves) __attribute__((amdgpu_waves_per_eu(3, 3))) void attention_fused_64_kernel(
    const uint8_t* __restrict__ Q_codes, const uint8_t* __restrict__ Q_scales, int asym, const uint16_t* __restrict__ Kp,
    const uint16_t* __restrict__ Vp, float* __restrict__ out, int Sq, int Sk, int Sqp, int Skv, int kv_group,
    float scale_log2, int causal, int merged_bf16) {
  // FP8-E5M2 scales: probabilities as FP16 times 2^8, V^T biased by 2^-3, the 2^5 taken out with the row sum at the end
  constexpr bool kPF16 = SCALE_KIND == kScaleE5M2;
  static_assert(kFrags == kWaves, "one fragment of K and one of V per wave");
  // two stages of (K tile, V tile), separate arrays so that loads into one stage are known not to alias reads of the other
  __shared__ __attribute__((aligned(1024))) uint8_t ldsK0[kFrags * kFragBytes];
  __shared__ __attribute__((aligned(1024))) uint8_t ldsV0[kFrags * kFragBytes];
  __shared__ __attribute__((aligned(1024))) uint8_t ldsK1[kFrags * kFragBytes];
  __shared__ __attribute__((aligned(1024))) uint8_t ldsV1[kFrags * kFragBytes];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // x walks the query heads, a contiguous range of them per XCD where their number is a multiple of 8; y the query blocks,
  // the last ones, which have the most key tiles under a causal mask, first
  const int nheads = (int)gridDim.x;
  const int h = (nheads & 7) == 0 ? (int)(blockIdx.x & 7) * (nheads >> 3) + (int)(blockIdx.x >> 3) : (int)blockIdx.x;
  const int g = h / kv_group;
  const int q0 = (int)(gridDim.y - 1 - blockIdx.y) * kQueries, qw = q0 + wave * 32;
  const int off = Sk - Sq;  // causal: query i sees keys <= i + off
  const bool wave_active = qw < Sqp;

  // key tiles this workgroup / this wave walks over (uniform)
  const int tiles_all = Sk / 32;
  const int last_query = (q0 + kQueries < Sqp ? q0 + kQueries : Sqp) - 1;
  const int nt = causal ? min(tiles_all, (last_query + off) / 32 + 1) : tiles_all;
  const int nt_wave = !wave_active ? 0 : (causal ? min(tiles_all, (qw + 31 + off) / 32 + 1) : tiles_all);

  // K panel of this key/value head: tile t = 4 contiguous fragments; V^T panel: 2 row blocks of Skv / 16 fragments (Skv = Sk
  // rounded up to the panel's K granularity of 64)
  const int64_t frags_k = (int64_t)tiles_all * kFrags, frags_v = (int64_t)(kD / 32) * (Skv / 16);
  const __amdgpu_buffer_rsrc_t Kr = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint8_t*>(reinterpret_cast<const uint8_t*>(Kp) + g * frags_k * kFragBytes), 0, (int)(frags_k * kFragBytes), 0x00020000);
  const __amdgpu_buffer_rsrc_t Vr = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint8_t*>(reinterpret_cast<const uint8_t*>(Vp) + g * frags_v * kFragBytes), 0, (int)(frags_v * kFragBytes), 0x00020000);
  const int lane_off = lane * 16;

  // this wave's share of tile T into stage (DK, DV): K fragment `wave`, and the V fragment of row block wave / 2, k-step wave % 2
#define AMX_ATTN_LOAD(T, DK, DV)                                                                                   \
  do {                                                                                                             \
    __builtin_amdgcn_raw_ptr_buffer_load_lds(Kr, (lds_ptr_t)((DK) + wave * kFragBytes), 16, lane_off,              \
                                             ((T) * kFrags + wave) * kFragBytes, 0, 0);                            \
    __builtin_amdgcn_raw_ptr_buffer_load_lds(Vr, (lds_ptr_t)((DV) + wave * kFragBytes), 16, lane_off,              \
                                             ((wave >> 1) * (Skv / 16) + (wave & 1) + 2 * (T)) * kFragBytes, 0, 0); \
  } while (0)

  // this wave's 32 queries as the B operand of the first product, dequantized here from their codes. Rows past Sq repeat the
  // last one.
  bf16x8 qf[kFrags];
  {
    const int q = qw + (lane & 31) < Sq ? qw + (lane & 31) : Sq - 1;
    const int64_t row = (int64_t)h * Sq + q;
    const u32x4* codes = reinterpret_cast<const u32x4*>(Q_codes + row * (kD / 2));
    const uint8_t* sb = Q_scales + row * (kD / 32) * (asym ? 2 : 1);
#pragma unroll
    for (int g = 0; g < kD / 32; ++g) {  // a group of 32: k-steps 2 g and 2 g + 1; lane half h takes words h, 2 + h
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

  f32x16 o[kD / 32];
#pragma unroll
  for (int db = 0; db < kD / 32; ++db)
#pragma unroll
    for (int v = 0; v < 16; ++v) o[db][v] = 0.f;
  float m = -__builtin_inff(), l = 0.f;  // running maximum (scaled score, in units of log2) and sum of this lane's query
  const int limit = causal ? qw + (lane & 31) + off : Sk - 1;  // last key this lane's query may attend to
  const int row_in_tile = 4 * (lane >> 5);                    // key of register v: 8 (v / 4) + row_in_tile + v % 4

  // one key tile from stage (CK, CV)
#define AMX_ATTN_TILE(T, CK, CV)                                                                                   \
  if ((T) < nt_wave) {                                                                                             \
    f32x16 s;                                                                                                      \
    _Pragma("unroll") for (int v = 0; v < 16; ++v) s[v] = 0.f;                                                     \
    _Pragma("unroll") for (int kb = 0; kb < kFrags; ++kb) {                                                        \
      const bf16x8 a = *reinterpret_cast<const bf16x8*>((CK) + kb * kFragBytes + lane_off);                        \
      s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qf[kb], s, 0, 0, 0);                                          \
    }                                                                                                              \
    const bool diagonal = causal && (T) * 32 + 31 > qw + off; /* some key of the tile is masked for some query */ \
    AMX_ATTENTION_TILE_PROBS(false, s, scale_log2, diagonal, (T) * 32 + row_in_tile, limit, m, l, pb, alpha, kPF16) \
    if (__builtin_amdgcn_ballot_w64(alpha != 1.0f) != 0) { /* the maximum moved for some query: rescale */        \
      _Pragma("unroll") for (int db = 0; db < kD / 32; ++db)                                                       \
        _Pragma("unroll") for (int v = 0; v < 16; ++v) o[db][v] *= alpha;                                          \
    }                                                                                                              \
    _Pragma("unroll") for (int j = 0; j < 2; ++j) {                                                                \
      const u32x4 b = {pb[4 * j], pb[4 * j + 1], pb[4 * j + 2], pb[4 * j + 3]};                                    \
      _Pragma("unroll") for (int db = 0; db < kD / 32; ++db) {                                                     \
        const u32x4 a = *reinterpret_cast<const u32x4*>((CV) + (db * 2 + j) * kFragBytes + lane_off);              \
        if constexpr (kPF16)                                                                                       \
          o[db] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), \
                                                         o[db], 0, 0, 0);                                          \
        else                                                                                                       \
          o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),                           \
                                                          __builtin_bit_cast(bf16x8, b), o[db], 0, 0, 0);          \
      }                                                                                                            \
    }                                                                                                              \
  }

  AMX_ATTN_LOAD(0, ldsK0, ldsV0);
  AMX_WAIT_VMCNT(0);
  AMX_BARRIER();
  for (int t = 0; t < nt; t += 2) {
    // stage 1 was last read during tile t - 1; the barrier that ended it lets every wave refill it now
    if (t + 1 < nt) AMX_ATTN_LOAD(t + 1, ldsK1, ldsV1);
    AMX_ATTN_TILE(t, ldsK0, ldsV0);
    AMX_WAIT_VMCNT(0);
    AMX_BARRIER();
    if (t + 1 < nt) {  // uniform over the workgroup
      if (t + 2 < nt) AMX_ATTN_LOAD(t + 2, ldsK0, ldsV0);
      AMX_ATTN_TILE(t + 1, ldsK1, ldsV1);
      AMX_WAIT_VMCNT(0);
      AMX_BARRIER();
    }
  }
#undef AMX_ATTN_TILE
#undef AMX_ATTN_LOAD

  // out[h][query][d] = O^T[d][query] / l; register 4c + r of row block db is d = 32 db + 8 c + 4 (lane / 32) + r. merged_bf16:
  // the same values rounded to BF16 and written token-major, out[query][h * 64 + d]. (The reciprocal stands in either branch on
  // purpose: in front of both it costs ten registers, and with them the fifth workgroup.)
  const int q = qw + (lane & 31);
  if (wave_active && q < Sq && merged_bf16) {
    const float inv = (kPF16 ? 0.03125f : 1.0f) / l;
    uint16_t* dst = reinterpret_cast<uint16_t*>(out) + ((int64_t)q * nheads + h) * kD + row_in_tile;
#pragma unroll
    for (int db = 0; db < kD / 32; ++db)
#pragma unroll
      for (int c = 0; c < 4; ++c)
        *reinterpret_cast<uint2*>(dst + db * 32 + c * 8) = make_uint2(
            pack2(o[db][4 * c] * inv, o[db][4 * c + 1] * inv), pack2(o[db][4 * c + 2] * inv, o[db][4 * c + 3] * inv));
  } else if (wave_active && q < Sq) {
    const float inv = (kPF16 ? 0.03125f : 1.0f) / l;
    float* dst = out + ((int64_t)h * Sq + q) * kD + row_in_tile;
#pragma unroll
    for (int db = 0; db < kD / 32; ++db)
#pragma unroll
      for (int c = 0; c < 4; ++c)
        *reinterpret_cast<float4*>(dst + db * 32 + c * 8) =
            make_float4(o[db][4 * c] * inv, o[db][4 * c + 1] * inv, o[db][4 * c + 2] * inv, o[db][4 * c + 3] * inv);
  }
}

hipError_t launch_attention_64(int scale_kind, bool asym, int64_t Hq, int64_t Hkv, int64_t Sq, int64_t Sk,
                               const uint8_t* Q_codes, const uint8_t* Q_scales, const uint16_t* K_panel,
                               const uint16_t* V_panel, float scale, int causal, float* out, bool merged_bf16, hipStream_t s) {
  const int64_t Sqp = round_up(Sq, 32);
  auto go = [&]<int SK>() {
    hipLaunchKernelGGL((attention_fused_64_kernel<SK>), dim3((unsigned)Hq, (unsigned)((Sqp + kQueries - 1) / kQueries)),
                       dim3(64 * kWaves), 0, s, Q_codes, Q_scales, asym ? 1 : 0, K_panel, V_panel, out, (int)Sq, (int)Sk, (int)Sqp,
                       (int)round_up(Sk, 64), (int)(Hq / Hkv), scale * 1.4426950408889634f, causal, merged_bf16 ? 1 : 0);
    return hipGetLastError();
  };
  switch (scale_kind) {
    case kScaleE5M2: return go.template operator()<kScaleE5M2>();
    case kScaleE4M3: return go.template operator()<kScaleE4M3>();
    case kScaleE8M0Floor: return go.template operator()<kScaleE8M0Floor>();
    case kScaleE8M0Round: return go.template operator()<kScaleE8M0Round>();
    default: return hipErrorInvalidValue;
  }
}

}  // namespace amx
