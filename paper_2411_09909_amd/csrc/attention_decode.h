// The operands of the fused attention for few queries in registers (attention_decode.hip, attention_decode_16.hip): codes and
// scale bytes as they are stored -> exact 16-bit floats.
#pragma once
#include "attention_tile.h"
#include "dequant_regs.h"
#include "kernels.h"

namespace amx {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// The 16-bit type the operands are dequantized to. FP8-E5M2 scales: FP16 with a bias of 2^-3 (every element * scale / 8
// lies in [2^-20, 43008] with at most 5 significant bits: an FP16 number, subnormals included; the scale byte is the
// upper byte of an FP16, so the dequantization is a conversion and one packed multiply); everything else: BF16.
template <int SCALE_KIND>
constexpr bool kDecodeF16 = SCALE_KIND == kScaleE5M2;

// Eight codes (one word) of one group -> eight exact 16-bit floats (element * scale has at most 6 significant bits).
// FP8-E5M2 scales: FP16, biased (above). Power-of-two scales: the FP4 -> BF16 conversion applies the scale itself (it
// reads the exponent field of a float). FP8-E4M3 scales: FP32 decode, times the scale of the element's sign class as a
// float, truncated to BF16.
template <int SCALE_KIND, bool ASYM>
__device__ __forceinline__ u32x4 decode_word(uint32_t word, uint32_t byte_pos, uint32_t byte_neg) {
  u32x4 r;
  if constexpr (kDecodeF16<SCALE_KIND>) {
    const uint32_t sp = ((byte_pos << 8) | (byte_pos << 24)) & 0x7F007F00u, sn = ((byte_neg << 8) | (byte_neg << 24)) & 0x7F007F00u;
    r = u32x4{dequant2_f16<ASYM, 0>(word, sp, sn), dequant2_f16<ASYM, 1>(word, sp, sn),
              dequant2_f16<ASYM, 2>(word, sp, sn), dequant2_f16<ASYM, 3>(word, sp, sn)};
  } else if constexpr (SCALE_KIND == kScaleE8M0Floor || SCALE_KIND == kScaleE8M0Round) {
    const uint32_t sp = byte_pos << 23, sn = byte_neg << 23;
    r = u32x4{dequant2_pot<ASYM, 0>(word, sp, sn), dequant2_pot<ASYM, 1>(word, sp, sn),
              dequant2_pot<ASYM, 2>(word, sp, sn), dequant2_pot<ASYM, 3>(word, sp, sn)};
  } else {
    const uint32_t sp = f2u(scale_value<SCALE_KIND>(byte_pos)), sn = ASYM ? f2u(scale_value<SCALE_KIND>(byte_neg)) : sp;
    r = u32x4{dequant2_f32<ASYM, 0>(word, sp, sn), dequant2_f32<ASYM, 1>(word, sp, sn),
              dequant2_f32<ASYM, 2>(word, sp, sn), dequant2_f32<ASYM, 3>(word, sp, sn)};
  }
  return r;
}

// The same with the group's scale bytes as one value: S_p in the low byte, S_n in the next (E5M2: sign bits cleared; ASYM == false:
// S_p alone).
template <int SCALE_KIND, bool ASYM>
__device__ __forceinline__ u32x4 decode_word_of_pair(uint32_t word, uint32_t pair) {
  if constexpr (kDecodeF16<SCALE_KIND>) {
    // each scale as two FP16, by one byte permute (shifts become a 32-bit multiplication, which takes four times as long)
    const uint32_t sp = __builtin_amdgcn_perm(0, pair, 0x000C000C), sn = ASYM ? __builtin_amdgcn_perm(0, pair, 0x010C010C) : sp;
    return u32x4{dequant2_f16<ASYM, 0>(word, sp, sn), dequant2_f16<ASYM, 1>(word, sp, sn),
                 dequant2_f16<ASYM, 2>(word, sp, sn), dequant2_f16<ASYM, 3>(word, sp, sn)};
  } else {
    return decode_word<SCALE_KIND, ASYM>(word, pair & 255u, ASYM ? pair >> 8 : pair);
  }
}

constexpr int kDecodeCols = 32;  // query columns of a key / value head in the workspace of the ranges' partial results

}  // namespace amx
