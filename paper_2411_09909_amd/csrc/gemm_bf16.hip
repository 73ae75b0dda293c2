// Fully quantized GEMM for scale formats whose values are not powers of two (FP8 E5M2, Sec. 4.2) and for the
// sign-asymmetric formats (Eq. 1, Sec. 4.3).
//
// A dequantized element is elem * S_class with elem in {0,.5,1,1.5,2,3,4,6} and S = (1 + m/4) * 2^e: up to 5
// significant bits (3 * 7 = 21; 6 bits with the 3 mantissa bits of an E4M3 scale, 3 * 15 = 45), which FP8/FP6/FP4
// MFMA operands cannot hold but BF16 holds exactly. Groups of 16, 64 or 128 elements, which do not match the 32-long
// blocks of the block-scaled instructions, also come here whatever their scale format. The GEMM is
// therefore run on the BF16 MFMA (v_mfma_f32_32x32x16_bf16) with exact operands and FP32 accumulation:
//
//   1. expand kernel: codes + scale pair -> BF16, written into "fragment-major" panels in the workspace:
//        panel[row_block of 32][k_block of 16][lane 0..63][8 BF16],  lane = 32 * (k / 8 % 2) + row % 32,
//      which is exactly the register image of one MFMA operand (lane l holds row l%32, k = 8*(l/32) .. +7).
//      Rows are padded to a multiple of 256 and K to a multiple of 128 with zeros.
//   2. GEMM kernel: every operand fragment is one contiguous KiB in the workspace, so staging global -> LDS is a
//      linear copy and LDS -> register reads are conflict-free 128-bit reads at lane * 16.

#include "device_formats.h"
#include "gemm_common.h"

namespace amx {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

size_t bf16_path_workspace_bytes(int64_t M, int64_t N, int64_t K, int64_t batch) {
  const int64_t Kp = round_up(K, kPanelK);
  return (size_t)(batch * (round_up(M, kPanelRows) + round_up(N, kPanelRows)) * Kp * 2);
}

size_t bf16_panel_bytes(int64_t rows, int64_t K) { return (size_t)(round_up(rows, kPanelRows) * round_up(K, kPanelK) * 2); }

// ------------------------------------------------------------------------------------------------ expand ----------
// grid: (ceil(Kp / 256), Rp / 32, batch); block 256 = 4 waves. A workgroup expands one 32-row block over a K span of
// 256, i.e. whole 128-byte lines of every code row (neighbouring workgroups run on different XCDs with separate L2s,
// so a line split between two of them would be fetched from HBM twice); wave w takes the 64-wide slice w of the span:
// lane = 32 * group_in_slice + row_in_block. The 16 fragments a workgroup writes are contiguous in the panel.
// F16: the panel holds FP16 values biased by 2^-3 instead of BF16 (FP8-E5M2 scales only: every such value lies in
// [2^-20, 43008] and has at most 5 significant bits, so it is an FP16 number, subnormals included).
// PERMUTE: within every block of 32 along K, the fragment of k-step j (0, 1) holds, in lane half h, the elements
// 16 j + 4 h + {0, 1, 2, 3, 8, 9, 10, 11} instead of 16 j + 8 h + {0 .. 7}. That is the order in which the rows of a
// 32x32 MFMA accumulator sit in a lane's registers, so an accumulator tile can be fed back as the other operand of a
// product over those rows without a transpose (the fused attention kernel multiplies probabilities with V this way).
// HALF_LINE: within every block of 256 along K (8 groups), k-step s (0 .. 15) holds, in lane half h, the 8 elements
// s % 4 of group 4 h + s / 4 instead of the 8 elements h of the 16 that follow 16 s: a lane half then draws all its
// 16 k-steps from one contiguous half (64 bytes of codes) of the block. The few-rows kernel reads its B operand in
// that order straight from the packed codes and needs A to match (a product sums over k in any order).
// One operand of an expansion: codes and scales of [batch][R][K] -> panel [batch][Rp / 32][Kp / 16] fragments.
struct ExpandJob {
  const uint8_t* codes;
  const uint8_t* scales;
  uint16_t* panel;
  int64_t R, K, Rp, Kp;
};

// One wave's share: 64-wide slice `slice` of row block rb of batch entry b.
template <int SCALE_KIND, bool ASYM, bool F16, bool PERMUTE, bool HALF_LINE>
__device__ __forceinline__ void expand_slice(const ExpandJob& job, int gs_log2, int64_t slice, int64_t rb, int64_t b) {
  const uint8_t* codes = job.codes;
  const uint8_t* scales = job.scales;
  uint16_t* panel = job.panel;
  const int64_t R = job.R, K = job.K, Rp = job.Rp, Kp = job.Kp;
  const int lane = threadIdx.x & 63;
  if (slice * 64 >= Kp) return;
  const int64_t r = rb * 32 + (lane & 31);
  const int64_t g = slice * 2 + (lane >> 5);  // the lane's block of 32 elements
  uint32_t w[4] = {0, 0, 0, 0};
  // scales of the first and of the second 16 elements of the block (they differ only for groups of 16)
  float s_pos[2] = {0.f, 0.f}, s_neg[2] = {0.f, 0.f};
  if (r < R && g < (K >> 5)) {
    const uint4 c = *reinterpret_cast<const uint4*>(codes + (b * R + r) * (K >> 1) + g * 16);
    w[0] = c.x, w[1] = c.y, w[2] = c.z, w[3] = c.w;
    const int64_t row_groups = (b * R + r) * groups_per_row(K, gs_log2);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if (h == 1 && gs_log2 != 4) {
        s_pos[1] = s_pos[0], s_neg[1] = s_neg[0];
        break;
      }
      const int64_t gi = row_groups + ((g * 32 + h * 16) >> gs_log2);
      if constexpr (ASYM) {
        const uint32_t sb = *reinterpret_cast<const uint16_t*>(scales + gi * 2);
        s_pos[h] = scale_value<SCALE_KIND>(sb & 255u);
        s_neg[h] = scale_value<SCALE_KIND>(sb >> 8);
      } else {
        s_pos[h] = s_neg[h] = scale_value<SCALE_KIND>(scales[gi]);
      }
    }
  }
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    s_pos[h] *= F16 ? 0.0625f : 0.5f;
    s_neg[h] *= F16 ? -0.0625f : -0.5f;
  }
  uint16_t* dst = panel + ((b * (Rp >> 5) + rb) * (Kp >> 4) + slice * 4 + (lane >> 5) * 2) * 512;
  uint32_t o[4][4];  // run t of 8 elements of the block -> 4 registers of 2 values
#pragma unroll
  for (int t = 0; t < 4; ++t) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t n0 = (w[t] >> (8 * j)) & 15u, n1 = (w[t] >> (8 * j + 4)) & 15u;
      const float v0 = (float)e2m1_twice(n0 & 7u) * ((n0 & 8u) ? s_neg[t >> 1] : s_pos[t >> 1]);
      const float v1 = (float)e2m1_twice(n1 & 7u) * ((n1 & 8u) ? s_neg[t >> 1] : s_pos[t >> 1]);
      if constexpr (F16)
        o[t][j] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(v0, v1));  // exact, see above
      else
        o[t][j] = (f2u(v0) >> 16) | (f2u(v1) & 0xFFFF0000u);  // truncation is exact: <= 6 significant bits
    }
  }
  if constexpr (HALF_LINE) {
    const int64_t blk = g >> 3;
    const int gl = (int)(g & 7);
    uint16_t* d2 = panel + ((b * (Rp >> 5) + rb) * (Kp >> 4) + blk * 16 + (gl & 3) * 4) * 512 +
                   ((gl >> 2) * 32 + (lane & 31)) * 8;
#pragma unroll
    for (int t = 0; t < 4; ++t) *reinterpret_cast<uint4*>(d2 + t * 512) = make_uint4(o[t][0], o[t][1], o[t][2], o[t][3]);
    return;
  }
#pragma unroll
  for (int t = 0; t < 4; ++t) {  // k block (t / 2), lane half (t % 2) of the block's two fragments
    uint4 out;
    if constexpr (PERMUTE)
      out = make_uint4(o[t & 2][2 * (t & 1)], o[t & 2][2 * (t & 1) + 1], o[(t & 2) + 1][2 * (t & 1)],
                       o[(t & 2) + 1][2 * (t & 1) + 1]);
    else
      out = make_uint4(o[t][0], o[t][1], o[t][2], o[t][3]);
    *reinterpret_cast<uint4*>(dst + (t >> 1) * 512 + ((t & 1) * 32 + (lane & 31)) * 8) = out;
  }
}

template <int SCALE_KIND, bool ASYM, bool F16, bool PERMUTE = false, bool HALF_LINE = false>
__global__ __launch_bounds__(256) void expand_kernel(ExpandJob job, int gs_log2) {
  expand_slice<SCALE_KIND, ASYM, F16, PERMUTE, HALF_LINE>(job, gs_log2, (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6),
                                                          blockIdx.y, blockIdx.z);
}

// Both operands of a product in one launch: row blocks of A, then of B (same K). A launch of its own for A's expansion cost
// the call 4 to 5 us, whatever A's size.
template <int SCALE_KIND, bool ASYM>
__global__ __launch_bounds__(256) void expand_pair_kernel(ExpandJob ja, ExpandJob jb, int gs_log2) {
  const int64_t blocks_a = ja.Rp >> 5, rb = blockIdx.y;
  const bool second = rb >= blocks_a;
  expand_slice<SCALE_KIND, ASYM, false, false, false>(second ? jb : ja, gs_log2, (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6),
                                                      second ? rb - blocks_a : rb, blockIdx.z);
}

// ------------------------------------------------------------------------------------------------ GEMM ------------
// Tile configuration, stage ring and supertile order: gemm_common.h. Here one stage is a K slice of 32.

// SCALED: the result is multiplied by the product of the operands' tensor-wise scales alpha_a[0] * alpha_b[0]
// (Sec. 5.3, double scaling), read from device memory after the main loop.
// GLU: the gated-activation epilogue of store_glu_tiles() instead of the FP32 store: C is then the BF16 output
// [M][ldc] with N / 2 columns.
template <int WM, int WN, int FM, int FN, bool SCALED, bool GLU = false, StoreWay WAY = kStoreRows>
__global__ __launch_bounds__(64 * WM * WN) void gemm_bf16_kernel(const uint16_t* __restrict__ Ap,
                                                                 const uint16_t* __restrict__ Bp, float* __restrict__ C,
                                                                 int64_t M, int64_t N, int64_t Mp, int64_t Np,
                                                                 int64_t Kp, int64_t ldc, int tiles_m, int tiles_n,
                                                                 int super_m, const float* __restrict__ alpha_a,
                                                                 const float* __restrict__ alpha_b) {
  using Cfg = TileCfg<WM, WN, FM, FN>;
  // Four separate arrays rather than one ring buffer: the compiler then knows that a direct-to-LDS load into one
  // stage cannot alias the fragment reads of another and does not serialise them.
  __shared__ __attribute__((aligned(1024))) uint8_t lds0[Cfg::kStageBytes];
  __shared__ __attribute__((aligned(1024))) uint8_t lds1[Cfg::kStageBytes];
  __shared__ __attribute__((aligned(1024))) uint8_t lds2[Cfg::kStageBytes];
  __shared__ __attribute__((aligned(1024))) uint8_t lds3[Cfg::kStageBytes];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int64_t b = blockIdx.z;

  int tm, tn;
  if (!tile_of_workgroup(blockIdx.x, tiles_m, tiles_n, super_m, tm, tn)) return;  // uniform, before any barrier

  // Buffer descriptors over this tile's slice of each panel: (tile rows / 32) row blocks x kblocks fragments of 1 KiB.
  // Raw buffer (stride 0), so reads past num_records return zero instead of faulting.
  const int kblocks = (int)(Kp >> 4);
  const uint8_t* Abase = reinterpret_cast<const uint8_t*>(Ap) +
                         ((b * (Mp >> 5) + (int64_t)tm * (Cfg::kTileM / 32)) * kblocks) * kFragBytes;
  const uint8_t* Bbase = reinterpret_cast<const uint8_t*>(Bp) +
                         ((b * (Np >> 5) + (int64_t)tn * (Cfg::kTileN / 32)) * kblocks) * kFragBytes;
  // (tiles of 192 rows or columns do not divide the panels' 256: the last one may reach beyond its panel)
  const int left_a = (int)(Mp >> 5) - tm * (Cfg::kTileM / 32), left_b = (int)(Np >> 5) - tn * (Cfg::kTileN / 32);
  const __amdgpu_buffer_rsrc_t Ar = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint8_t*>(Abase), 0, (left_a < Cfg::kTileM / 32 ? left_a : Cfg::kTileM / 32) * kblocks * kFragBytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t Br = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint8_t*>(Bbase), 0, (left_b < Cfg::kTileN / 32 ? left_b : Cfg::kTileN / 32) * kblocks * kFragBytes, 0x00020000);
  const int lane_off = lane * 16;

  f32x16 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  // Load number L (0 .. kLoads-1) of this wave for K stage ST into ring slot array DST: fragment f = wave + kWaves * L
  // of the stage; f < kFragsA: A row block f / 2, k block f % 2; otherwise the same for B. One contiguous KiB of the
  // panel goes to DST + f KiB (the hardware adds lane * 16 on the LDS side).
  // (local copies of the tile constants: naming Cfg:: members directly inside the builtin's arguments trips the host
  // pass of the compiler, which then drops the kernel's launch stub)
  constexpr int kWaves = Cfg::kWaves, kFragsA = Cfg::kFragsA, kLoads = Cfg::kLoads;
#define AMX_ISSUE_LOAD(L, ST, DST)                                                                         \
  {                                                                                                        \
    const int f_ = wave + kWaves * (L);                                                                    \
    if ((L) < kFragsA / kWaves) /* decided at compile time once the loops are unrolled */                  \
      __builtin_amdgcn_raw_ptr_buffer_load_lds(Ar, (lds_ptr_t)((DST) + f_ * kFragBytes), 16, lane_off,     \
                                               ((f_ >> 1) * kblocks + (ST) * 2 + (f_ & 1)) * kFragBytes,   \
                                               0, 0);                                                      \
    else                                                                                                   \
      __builtin_amdgcn_raw_ptr_buffer_load_lds(                                                            \
          Br, (lds_ptr_t)((DST) + f_ * kFragBytes), 16, lane_off,                                          \
          (((f_ - kFragsA) >> 1) * kblocks + (ST) * 2 + (f_ & 1)) * kFragBytes, 0, 0);                     \
  }

  const int nstages = (int)(Kp / 32);  // one stage = a K slice of 32 BF16 (2 MFMA k-steps); multiple of 4
  // prologue: 3 stages in flight; stages 0 and 1 must have landed before the first fragment reads
#pragma unroll
  for (int l = 0; l < kLoads; ++l) AMX_ISSUE_LOAD(l, 0, lds0);
#pragma unroll
  for (int l = 0; l < kLoads; ++l) AMX_ISSUE_LOAD(l, 1, lds1);
#pragma unroll
  for (int l = 0; l < kLoads; ++l) AMX_ISSUE_LOAD(l, 2, lds2);
  AMX_WAIT_VMCNT(kLoads);
  AMX_BARRIER();

  // register rings: the A fragment for step t lives in aR[t & 3] (read two steps ahead; t counts on through the four stages
  // of the loop below, T0 being a stage's first step), the B fragments of k-step ks in bR[ks & 1] (read during the previous
  // k-step)
  bf16x8 aR[4], bR[2][FN];
  const int offA = lane_off + (wm * FM) * 2 * kFragBytes;
  const int offB = lane_off + (Cfg::kFragsA + (wn * FN) * 2) * kFragBytes;
  aR[0] = *reinterpret_cast<const bf16x8*>(lds0 + offA);
  aR[1] = *reinterpret_cast<const bf16x8*>(lds0 + offA + 2 * kFragBytes);
#pragma unroll
  for (int j = 0; j < FN; ++j) bR[0][j] = *reinterpret_cast<const bf16x8*>(lds0 + offB + j * 2 * kFragBytes);

  // One stage: 2 k-steps x FM steps; a step issues the fragment reads needed two steps (A) or one k-step (B) later,
  // its share of the direct-to-LDS loads for stage S + 3, then FN MFMAs. CUR / NXT are the ring arrays of stage S and
  // S + 1, FETCH the one stage S + 3 lands in (last read during stage S - 1). Past the end of K the fetch is pointed
  // at the last real stage instead of being skipped: it lands in a slot nobody reads any more and the body stays free
  // of branches.
#define AMX_STAGE(S, CUR, NXT, FETCH, T0)                                                                                \
  {                                                                                                                  \
    const int fetch_ = (S) + 3 < nstages ? (S) + 3 : nstages - 1;                                                    \
    _Pragma("unroll") for (int ks = 0; ks < 2; ++ks) {                                                               \
      _Pragma("unroll") for (int i = 0; i < FM; ++i) {                                                               \
        const int t = ks * FM + i;                                                                                   \
        {                                                                                                            \
          const int t2 = t + 2, ks2 = t2 / FM, i2 = t2 % FM;                                                         \
          const uint8_t* src_ = ks2 < 2 ? (CUR) : (NXT);                                                             \
          aR[(T0 + t2) & 3] = *reinterpret_cast<const bf16x8*>(src_ + offA + (i2 * 2 + (ks2 & 1)) * kFragBytes);    \
        }                                                                                                            \
        _Pragma("unroll") for (int jj = 2 * i; jj < 2 * i + 2; ++jj) {                                               \
          if (jj < FN) {                                                                                             \
            const uint8_t* src_ = ks == 0 ? (CUR) : (NXT);                                                           \
            bR[(ks + 1) & 1][jj] =                                                                                   \
                *reinterpret_cast<const bf16x8*>(src_ + offB + (jj * 2 + ((ks + 1) & 1)) * kFragBytes);             \
          }                                                                                                          \
        }                                                                                                            \
        _Pragma("unroll") for (int l = t; l < kLoads; l += 2 * FM) AMX_ISSUE_LOAD(l, fetch_, FETCH);            \
        _Pragma("unroll") for (int j = 0; j < FN; ++j) acc[i][j] =                                                   \
            __builtin_amdgcn_mfma_f32_32x32x16_bf16(aR[(T0 + t) & 3], bR[ks & 1][j], acc[i][j], 0, 0, 0);            \
        __builtin_amdgcn_sched_barrier(0);                                                                           \
      }                                                                                                              \
    }                                                                                                                \
    /* stage S + 2 must be complete in LDS for every wave before stage S + 1 starts reading ahead into it; the same  \
       barrier tells every wave that stage S is no longer read, so its slot may be refilled during stage S + 1 */    \
    AMX_WAIT_VMCNT(kLoads);                                                                                     \
    AMX_BARRIER();                                                                                                   \
  }

  for (int s = 0; s < nstages; s += 4) {
    AMX_STAGE(s, lds0, lds1, lds3, 0);
    AMX_STAGE(s + 1, lds1, lds2, lds0, 2 * FM);
    AMX_STAGE(s + 2, lds2, lds3, lds1, 4 * FM);
    AMX_STAGE(s + 3, lds3, lds0, lds2, 6 * FM);
  }
  AMX_WAIT_VMCNT(0);  // nothing may still be writing this workgroup's LDS when it retires
#undef AMX_STAGE
#undef AMX_ISSUE_LOAD

  if constexpr (GLU) {
    // every wave is past its last fragment read: the operand stages become the waves' transposition space
    static_assert(glu_stage_bytes<FM, FN>() * ((Cfg::kWaves + 3) / 4) <= Cfg::kStageBytes, "stage too small");
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
    AMX_BARRIER();
    const int w = wm * WN + wn;
    uint8_t* stage = ((w & 3) == 0 ? lds0 : (w & 3) == 1 ? lds1 : (w & 3) == 2 ? lds2 : lds3) +
                     (w >> 2) * glu_stage_bytes<FM, FN>();
    store_glu_tiles<FM, FN>(acc, stage, reinterpret_cast<uint16_t*>(C) + b * M * ldc, M, N >> 1, ldc,
                            (int64_t)tm * Cfg::kTileM + wm * FM * 32, (int64_t)tn * Cfg::kTileN + wn * FN * 32);
  } else if constexpr (SCALED)
    store_c_tiles<FM, FN, WAY, 0, true>(acc, C + b * M * ldc, M, N, ldc, (int64_t)tm * Cfg::kTileM + wm * FM * 32,
                                        (int64_t)tn * Cfg::kTileN + wn * FN * 32, alpha_a[0] * alpha_b[0]);
  else
    store_c_tiles<FM, FN, WAY>(acc, C + b * M * ldc, M, N, ldc, (int64_t)tm * Cfg::kTileM + wm * FM * 32,
                                         (int64_t)tn * Cfg::kTileN + wn * FN * 32);
}

template <int SK, bool ASYM, bool F16 = false>
static hipError_t launch_expand(const uint8_t* codes, const uint8_t* scales, int64_t R, int64_t K, int64_t Rp,
                                int64_t Kp, int gs_log2, int64_t batch, uint16_t* panel, hipStream_t s) {
  hipLaunchKernelGGL((expand_kernel<SK, ASYM, F16>), dim3((unsigned)((Kp + 255) / 256), (unsigned)(Rp / 32), (unsigned)batch),
                     dim3(256), 0, s, (ExpandJob{codes, scales, panel, R, K, Rp, Kp}), gs_log2);
  return hipGetLastError();
}

static hipError_t expand_dispatch(int scale_kind, bool asym, int gs_log2, const uint8_t* codes, const uint8_t* scales,
                                  int64_t R, int64_t K, int64_t Rp, int64_t Kp, int64_t batch, uint16_t* panel,
                                  hipStream_t s) {
  if (scale_kind == kScaleE5M2)
    return asym ? launch_expand<kScaleE5M2, true>(codes, scales, R, K, Rp, Kp, gs_log2, batch, panel, s)
                : launch_expand<kScaleE5M2, false>(codes, scales, R, K, Rp, Kp, gs_log2, batch, panel, s);
  if (scale_kind == kScaleE4M3)
    return asym ? launch_expand<kScaleE4M3, true>(codes, scales, R, K, Rp, Kp, gs_log2, batch, panel, s)
                : launch_expand<kScaleE4M3, false>(codes, scales, R, K, Rp, Kp, gs_log2, batch, panel, s);
  return asym ? launch_expand<kScaleE8M0Floor, true>(codes, scales, R, K, Rp, Kp, gs_log2, batch, panel, s)
              : launch_expand<kScaleE8M0Floor, false>(codes, scales, R, K, Rp, Kp, gs_log2, batch, panel, s);
}

// The K and V panels of an attention in one launch: a wave takes one 64-wide slice of one 32-row block, the slices of K
// (rows = keys, along the head dimension) in front of those of V (rows = head dimension, along the keys, permuted).
// E5M2 scales: V as FP16 with a bias of 2^-3 (every element * scale / 8 is an FP16 number): the probabilities it is
// multiplied with come out of the attention kernel's cast as FP16 for this scale format.
template <int SCALE_KIND, bool ASYM>
__global__ __launch_bounds__(256) void expand_kv_kernel(ExpandJob jk, ExpandJob jv, int slices_k, int slices_v, int blocks_k) {
  const bool is_v = (int)blockIdx.x >= blocks_k;
  const int unit = ((int)blockIdx.x - (is_v ? blocks_k : 0)) * 4 + (int)(threadIdx.x >> 6);
  const int per_row_block = is_v ? slices_v : slices_k, rb = unit / per_row_block, slice = unit % per_row_block;
  if (rb >= (int)((is_v ? jv.Rp : jk.Rp) >> 5)) return;
  if (is_v)
    expand_slice<SCALE_KIND, ASYM, SCALE_KIND == kScaleE5M2, true, false>(jv, 5, slice, rb, blockIdx.y);
  else
    expand_slice<SCALE_KIND, ASYM, false, false, false>(jk, 5, slice, rb, blockIdx.y);
}

hipError_t launch_expand_kv(int scale_kind, bool asym, const uint8_t* K_codes, const uint8_t* K_scales, uint16_t* K_panel,
                            const uint8_t* V_codes, const uint8_t* V_scales, uint16_t* V_panel, int64_t Sk,
                            int64_t head_dim, int64_t heads, hipStream_t s) {
  if (Sk % 32 != 0 || head_dim % 64 != 0) return hipErrorInvalidValue;
  const int64_t Skv = round_up(Sk, 64);
  const ExpandJob jk = {K_codes, K_scales, K_panel, Sk, head_dim, Sk, head_dim};
  const ExpandJob jv = {V_codes, V_scales, V_panel, head_dim, Sk, head_dim, Skv};
  const int slices_k = (int)(head_dim / 64), slices_v = (int)(Skv / 64);
  const int blocks_k = (int)((Sk / 32 * slices_k + 3) / 4), blocks_v = (int)((head_dim / 32 * slices_v + 3) / 4);
  const dim3 grid((unsigned)(blocks_k + blocks_v), (unsigned)heads);
  auto go = [&]<int SK>() {
    if (asym)
      hipLaunchKernelGGL((expand_kv_kernel<SK, true>), grid, dim3(256), 0, s, jk, jv, slices_k, slices_v, blocks_k);
    else
      hipLaunchKernelGGL((expand_kv_kernel<SK, false>), grid, dim3(256), 0, s, jk, jv, slices_k, slices_v, blocks_k);
    return hipGetLastError();
  };
  if (scale_kind == kScaleE5M2) return go.template operator()<kScaleE5M2>();
  if (scale_kind == kScaleE4M3) return go.template operator()<kScaleE4M3>();
  return go.template operator()<kScaleE8M0Floor>();  // (floor and round share the byte encoding)
}

hipError_t launch_expand_half_line(int scale_kind, bool asym, const uint8_t* codes, const uint8_t* scales, int64_t R,
                                   int64_t K, int64_t Rp, int64_t batch, uint16_t* panel, hipStream_t s) {
  if (K % 256 != 0 || Rp % 32 != 0) return hipErrorInvalidValue;
  const dim3 grid((unsigned)(K / 256), (unsigned)(Rp / 32), (unsigned)batch);
  auto go = [&]<int SK, bool ASYM, bool F16>() {
    hipLaunchKernelGGL((expand_kernel<SK, ASYM, F16, false, true>), grid, dim3(256), 0, s,
                       (ExpandJob{codes, scales, panel, R, K, Rp, K}), 5);
    return hipGetLastError();
  };
  if (scale_kind == kScaleE5M2)
    return asym ? go.template operator()<kScaleE5M2, true, true>() : go.template operator()<kScaleE5M2, false, true>();
  if (scale_kind == kScaleE4M3)
    return asym ? go.template operator()<kScaleE4M3, true, false>() : go.template operator()<kScaleE4M3, false, false>();
  return asym ? go.template operator()<kScaleE8M0Floor, true, false>()
              : go.template operator()<kScaleE8M0Floor, false, false>();
}

hipError_t launch_expand_f16_e5m2(bool asym, const uint8_t* codes, const uint8_t* scales, int64_t R, int64_t K,
                                  int64_t Rp, int64_t Kp, int64_t batch, uint16_t* panel, hipStream_t s) {
  return asym ? launch_expand<kScaleE5M2, true, true>(codes, scales, R, K, Rp, Kp, 5, batch, panel, s)
              : launch_expand<kScaleE5M2, false, true>(codes, scales, R, K, Rp, Kp, 5, batch, panel, s);
}

// Tiles of every XCD, and of the one with the most, where whole supertiles are dealt.
struct SupertileShare {
  int64_t tiles[8], most;
};
static SupertileShare supertile_share(int tiles_m, int tiles_n) {
  const int super_m = (tiles_m + kSuperM - 1) / kSuperM, super_n = (tiles_n + kSuperN - 1) / kSuperN;
  SupertileShare r = {};
  for (int st = 0; st < super_m * super_n; ++st) {
    const int m = tiles_m - st % super_m * kSuperM, n = tiles_n - st / super_m * kSuperN;
    int64_t& t = r.tiles[st & 7];
    t += (m < kSuperM ? m : kSuperM) * (n < kSuperN ? n : kSuperN);
    r.most = t > r.most ? t : r.most;
  }
  return r;
}

// Whether equal runs of tiles of 256 x tile_cols, per_xcd to an XCD, end sooner than supertiles where those leave a fifth
// of their slots empty. What counts is the tiles that an XCD really has (its share; 32 CUs: one round of 32 at a time),
// measured in both orders over 1 .. 16 rows and 2 .. 251 columns of tiles, us of the kernel, supertiles / runs:
//   fewer rounds: runs (12 x 20 tiles, K 13824, a share of 64 tiles or 30: 520 / 292;  9 x 112, K 4096, 224 or 126: 556 / 392)
//   one round either way: runs, which spread the tiles over all XCDs (8 x 16, K 4096, 32 or 16: 98 / 76;  1 x 126: 193 / 123),
//     but with a partial row of supertiles, whose XCDs alternate between full and nearly empty, only for much smaller shares
//     (9 x 16, K 4096, 32 or 18: 87 / 77;  12 x 16 tiles of 256 x 128, K 2048, 32 or 24: 28 / 29)
//   several rounds, as many either way: runs
//     up to two rows of tiles (2 x 112, K 4096: 174 / 117), and three of 256 x 128 (3 x 172, the call: 177 / 150)
//     where no more than two XCDs carry the largest share or 8 tiles less (8 x 40, K 8192, 64 or 40: 358 / 311;  14 x 20 of FP6,
//       the call: 238 / 214)
//     without a partial row of supertiles where the last round of that share is nearly full (6 x 112, K 4096, 96 or 84: 340 / 292)
//   otherwise they only make every XCD take a last round that few took (6 x 86 of 256 x 128, 72 or 65: 132 / 143;  4 x 224 of
//     them, 112 either way: 222 / 244;  10 x 32, K 8192, 64 or 40: 289 / 309;  12 x 43, K 4096, 96 or 65: 248 / 261, FP4 100 /
//     106;  14 x 43 of FP4, the call: 107 / 113;  3 x 86 of it, gated, 59 / 64)
//   one or two columns and many rows: a run shares fewer rows of A (32 x 2 FP4 tiles, K 28672, the call: 175 / 189)
static bool equal_runs_pay(int tiles_m, int tiles_n, int tile_cols, int64_t per_xcd) {
  if (tiles_n <= 2 && tiles_m > 2 * kSuperM) return false;
  const SupertileShare shares = supertile_share(tiles_m, tiles_n);
  const int64_t share = shares.most;
  constexpr int kRound = kSuperM * kSuperN;
  const bool partial_row = tiles_m > kSuperM && tiles_m % kSuperM != 0;
  if ((per_xcd + kRound - 1) / kRound < (share + kRound - 1) / kRound || tiles_m <= (tile_cols < 256 ? 3 : 2))
    return true;
  if (share <= kRound) return !partial_row || 8 * per_xcd <= 5 * share;
  int fullest = 0;
  for (int64_t t : shares.tiles) fullest += t >= share - 8;
  return fullest <= 2 || (!partial_row && (share - 1) % kRound >= 19);
}

// Grid size (x) for a tiles_m x tiles_n problem, and the order of its tiles (super_m, for tile_of_workgroup()).
// Supertiles are dealt 8 at a time, one per XCD. Where tiles_m is no multiple of 8, or the last 8 supertiles are not all
// there, an XCD has whole supertiles of work while others have none or leave CUs empty: then equal runs of tiles are dealt
// where they pay (bands of fewer than 8 rows share the staged panels a little less). The rule above is for one problem of tiles
// that fill a CU; with tiles of fewer rows, and in a batch, whose entries all start at the same XCD, the runs are dealt
// wherever a fifth of the slots is empty (8 x 1024 x 1024 x 128 on FP4: 41 / 12.5; 1504 x 1024 x 1024 on 64-row tiles: 20 / 18).
// Per call, E5M2 asymmetric on the panel kernel: 3000 x 5120 x 13824, 12 x 20 tiles, 543 -> 345 us; 2300 x 13824 x 5120, 9 x
// 54, 387 -> 269; 1504 x 28672 x 4096, 6 x 112, 400 -> 347; 1504 x 6144 x 4096, 6 x 24, 92 -> 87; 4067 x 4544 x 4544, 16 x 36
// of the 256 x 128 tiles, 183 -> 173. Merged FP6, 3000 x 10240 x 8192: 228 -> 179. Where few slots are empty, supertiles: 4096
// x 28672 x 8192 stays at 1430-1440.
unsigned supertile_grid(int tiles_m, int tiles_n, int tile_rows, int tile_cols, int64_t batch, int& super_m) {
  super_m = (tiles_m + kSuperM - 1) / kSuperM;
  const int super_n = (tiles_n + kSuperN - 1) / kSuperN;
  const int rounds = (super_m * super_n + 7) / 8;
  const int64_t tiles = (int64_t)tiles_m * tiles_n, per_xcd = (tiles + 7) / 8;
  if (tiles < (int64_t(1) << 30) && 5 * per_xcd <= 4 * (int64_t)rounds * kSuperM * kSuperN &&
      (batch > 1 || tile_rows < 256 || equal_runs_pay(tiles_m, tiles_n, tile_cols, per_xcd))) {
    super_m = 0;
    return (unsigned)(per_xcd * 8);
  }
  return (unsigned)(rounds * 8 * kSuperM * kSuperN);
}

// The most tiles that one XCD has in the order that supertile_grid() gives.
static int64_t largest_share(int tiles_m, int tiles_n, int tile_rows, int tile_cols) {
  int super_m;
  const unsigned grid = supertile_grid(tiles_m, tiles_n, tile_rows, tile_cols, 1, super_m);
  return super_m == 0 ? grid / 8 : supertile_share(tiles_m, tiles_n).most;
}

// Row by row, the column tiles of a row one after the other: where rows are no whole lines, a line is written by two stores, and they
// meet in L2 only if they are close. Streaming, except for rows that are not even half lines, a C below 80 MB and a K up to 4096: the two
// halves of a line then wait for each other in the caches; with a deeper K the operands need those (panels, 1400 x 2161 x 8192 73.4 /
// 72.5 / 75.3). us, column by column / row by row / row by row through the caches: FP4 3000 x 5001 x 4096 76 / 49 / 41, 4096 x 10001 x
// 1024 160 / 83 / 75, 4096 x 32001 x 4096 532 / 297 / 354, FP6 4096 x 4545 x 4544 141 / 109 / 104, BF16 panels 4096 x 32001 x 4096 1126 /
// 917 / 892, 1400 x 50257 x 2048 423 / 319 / 364. The 80 MB are of one problem of a batch: its problems are written one after
// the other (FP4 64 x 512 x 1001 x 256 116 / 57 / 39, 32 x 1000 x 2001 x 512, 256 MB in all, 222 / 102 / 95, panels 32 x 512 x
// 4097 x 128 238 / 116 / 97).
// Whole lines, too, are stored faster row by row (FP4 4096 x 4096 x 512 23.8 / 22.3, 2048 x 11008 x 4096 68.3 / 67.2, 4096 x 32000 x
// 4096 273 / 269, panels 4096 x 11008 x 512 77.0 / 75.6; through the caches they take a tenth longer), but not at a pitch of 8192,
// 16384 or 32768 elements, where the rows of a tile lie on few memory channels: FP4 2048 x 8192 x 512 24.0 / 30.1, 4096 x 8192 x
// 4096 83 / 91, 4096 x 16384 x 512 77 / 81, 4096 x 32768 x 512 158 / 169, panels 2048 x 8192 x 1024 49.6 / 53.5, half lines at such a
// pitch FP4 4096 x 8192 x 1024 53 / 66 (but 3000 x 16384 x 2048 86.3 / 85.4; at 4096 elements 26.6 / 25.4 for 3000 x 4096 x 2048, at 24576
// 55.2 / 50.6 for 2048 x 24576 x 512; not even half lines 119 / 86).
StoreWay store_way(const float* C, int64_t M, int64_t K, int64_t pitch) {
  const bool half_lines = ((reinterpret_cast<uintptr_t>(C) | (uintptr_t)pitch) & 63) == 0;
  if (half_lines && pitch >= 32768 && (pitch & (pitch - 1)) == 0) return kStoreColumns;
  return half_lines || K > 4096 || M * pitch >= 80000000 ? kStoreRows : kStoreRowsCached;
}

template <int WM, int WN, int FM, int FN>
static hipError_t launch_tiles(const uint16_t* Ap, const uint16_t* Bp, float* C, int64_t M, int64_t N, int64_t Mp,
                               int64_t Np, int64_t Kp, int64_t ldc, int64_t batch, const float* alpha_a,
                               const float* alpha_b, bool glu, hipStream_t s) {
  using Cfg = TileCfg<WM, WN, FM, FN>;
  const int tiles_m = (int)((M + Cfg::kTileM - 1) / Cfg::kTileM), tiles_n = (int)((N + Cfg::kTileN - 1) / Cfg::kTileN);
  int super_m;
  const unsigned grid = supertile_grid(tiles_m, tiles_n, Cfg::kTileM, Cfg::kTileN, batch, super_m);
  if (glu) {
    if constexpr (FN % 2 == 0)  // (gate and up columns alternate in blocks of 32)
      hipLaunchKernelGGL((gemm_bf16_kernel<WM, WN, FM, FN, false, true>), dim3(grid, 1, (unsigned)batch),
                         dim3(Cfg::kThreads), 0, s, Ap, Bp, C, M, N, Mp, Np, Kp, ldc, tiles_m, tiles_n, super_m, alpha_a,
                         alpha_b);
    else
      return hipErrorInvalidValue;
  } else if (alpha_a && alpha_b)
    in_store_way(C, M, Kp, ldc, [&]<StoreWay WAY>() {
      hipLaunchKernelGGL((gemm_bf16_kernel<WM, WN, FM, FN, true, false, WAY>), dim3(grid, 1, (unsigned)batch), dim3(Cfg::kThreads), 0, s,
                         Ap, Bp, C, M, N, Mp, Np, Kp, ldc, tiles_m, tiles_n, super_m, alpha_a, alpha_b);
    });
  else
    in_store_way(C, M, Kp, ldc, [&]<StoreWay WAY>() {
      hipLaunchKernelGGL((gemm_bf16_kernel<WM, WN, FM, FN, false, false, WAY>), dim3(grid, 1, (unsigned)batch), dim3(Cfg::kThreads), 0, s,
                         Ap, Bp, C, M, N, Mp, Np, Kp, ldc, tiles_m, tiles_n, super_m, alpha_a, alpha_b);
    });
  return hipGetLastError();
}

// Tile shape (1: 256 x 256, 2: 256 x 128, 3: 64 x 256). 256 x 256 (4 waves of 128 x 128) has the least operand traffic and
// LDS reads per MFMA and is what large problems use; a problem with fewer such tiles than the chip has CUs, or with one
// side much smaller than a tile, finishes sooner with 256 x 128 or 64 x 256 tiles that fill the CUs. The choice minimises
// (rounds of 256 workgroups) x (measured cost of one tile relative to a 256 x 256 one: 0.6 and 0.4), and leaves
// 256 x 256 only for a predicted gain: of more than 15 % for 64 x 256, of more than 8 % for 256 x 128, which takes in the
// problems of 257 to 384 large tiles: two rounds of those, three of the halves. Us per call, 256 x 256 / 256 x 128:
// 2048 x 11008 x 4096 213-219 / 183, 1700 x 11008 x 4096 196-198 / 170, 1900 x 10240 x 8192 403 / 339, 2600 x 8192 x 8192
// 355 / 337, 3800 x 4544 x 4544 201 / 186, 1300 x 13824 x 5120 221 / 220. With no more than three rows of tiles that needs a
// second round of hardly any large tiles (768 x 22016 x 4096, 258 tiles, gated, prepared, 167 / 150; but 768 x 28672 x 8192,
// 336 tiles, 490 / 522, gated x 4096, prepared, 170 / 182; 640 x 32001 x 4096, 378 tiles, prepared, 214 / 221).
int bf16_tile_choice(int64_t M, int64_t N, int64_t batch) {
  auto rounds = [&](int64_t tile_m, int64_t tile_n) {
    const int64_t tiles = ((M + tile_m - 1) / tile_m) * ((N + tile_n - 1) / tile_n) * batch;
    return (double)((tiles + 255) / 256);
  };
  const double est1 = rounds(256, 256), est2 = 0.6 * rounds(256, 128), est3 = 0.4 * rounds(64, 256);
  const bool ok3 = est3 < 0.85 * est1;
  const bool two_rounds = M > 768 || (M + 255) / 256 * ((N + 255) / 256) * batch <= 288;
  // (with a single row of 256-row tiles the 64-row tile was never worse)
  const bool ok2 = est2 < (two_rounds ? 0.92 : 0.85) * est1 && M > 256;
  return ok3 && (!ok2 || est3 <= est2) ? 3 : ok2 ? 2 : 1;
}

// The same for a single problem with the shapes between those three: 4: 192 x 256, 5: 192 x 128, 6: 128 x 128, 7: 192 x 192
// (not gated: gate and up columns alternate in blocks of 32, so a wave's column tiles come in pairs). `choice` stays unless
// one of them is estimated to be 3 % faster. The estimate, us of the kernel: the rounds of the XCD with the most tiles (32
// CUs; the shapes with two workgroups on a CU take less for the second round) at the time of a lone tile per unit of K, which
// grows with the share of the chip that is busy (the clock falls: a lone 256 x 256 tile takes 15 ns per unit of K, a full
// chip of them 20), or all tiles at the rate the shape reaches on a full chip, and the store of C. Fitted to 280 sizes of
// 40 to 4097 rows, mean error 5 %; the smaller shapes in the first rounds only, beyond which the larger tiles' lower traffic
// decides (954 x 28672 x 4096: 256 x 256 195, 192 x 192 228), and 128 x 128 not for a K below 2048 (813 x 1024 x 1024, the
// call: 64 x 256 13.9, 128 x 128 14.6). Us per call on three sets of buffers in turn, E5M2 asymmetric, before / with the chosen
// one: 1504 x 6144 x 4096 86 / 73 (192 x 192: 256 tiles instead of 144), 1563 x 10240 x 8192 364 / 307 (192 x 256), 1504 x 4096
// x 14336 255 / 223 and 1024 x 5120 x 13824 228 / 207 (192 x 128), 2048 x 11008 x 4096 180 / 165 and 3000 x 4096 x 4096 94 /
// 87 (192 x 256); 281 x 8192 x 8192 67 / 58 (the kernel; 128 x 128).
// Where the estimate was wrong over 2660 more sizes (257 to 4096 rows, plain, gated and prepared; before / with the other):
// 192 x 256 in more rounds than 256 x 256 takes (1148 x 25920 x 2432, gated, prepared, 120 / 140; 2071 x 13824 x 5120, gated,
// 260 / 281), and instead of 64 x 256 with a K up to 1024 (1408 x 5632 x 1024, gated, 25.1 / 25.7), in a second round up to 2048
// (1311 x 11072 x 1792, gated, 65 / 72; 574 x 24704 x 1792 82 / 87; a gated layer of 1312 tokens x 11264 x 2048 276 / 280). All shapes add the products of an output in the same order: their bits are the same.
struct TileEstimates {
  double us[8];
  int64_t rounds[8];
  bool ok[8];
};

static TileEstimates tile_estimates(int64_t M, int64_t N, int64_t K, bool gated) {
  struct Shape {
    int tile, rows, cols, rounds;    // at most so many rounds
    double lone, pair, grows, rate;  // ns per unit of K: one round, two; slower by this share on a full chip; TFLOP/s
  };
  static constexpr Shape kShapes[] = {
      {1, 256, 256, 0, 14.4, 28.8, 0.30, 1500}, {2, 256, 128, 0, 7.6, 15.2, 0.23, 1330}, {3, 64, 256, 0, 6.1, 11.0, 0.23, 1080},
      {4, 192, 256, 3, 10.7, 21.4, 0.26, 1440}, {5, 192, 128, 1, 6.4, 12.5, 0.21, 1500}, {6, 128, 128, 1, 5.4, 9.0, 0.24, 1370},
      {7, 192, 192, 1, 8.2, 16.4, 0.25, 1530}};
  TileEstimates e = {};
  for (const Shape& s : kShapes) {
    const int tiles_m = (int)((M + s.rows - 1) / s.rows), tiles_n = (int)((N + s.cols - 1) / s.cols);
    const int64_t r = (largest_share(tiles_m, tiles_n, s.rows, s.cols) + 31) / 32, tiles = (int64_t)tiles_m * tiles_n;
    const double per = (double)(r / 2) * s.pair + (double)(r % 2) * s.lone;
    const double own = per * (1.0 + s.grows * (double)tiles / (256.0 * (double)r)) * 1e-3 * (double)K;
    const double full = (double)(tiles * s.rows * s.cols) * 2e-6 * (double)K / s.rate;
    e.us[s.tile] = 7.0 + (own > full ? own : full) + 0.6 * 4.0 * (double)(M * N) / 5.1e6;
    e.rounds[s.tile] = r;
    e.ok[s.tile] = r <= s.rounds && !(gated && s.tile == 7) && !(s.tile == 6 && K < 2048);
  }
  return e;
}

int bf16_tile_refined(int choice, int64_t M, int64_t N, int64_t K, int64_t batch, bool gated) {
  if (batch != 1 || ((M + 255) / 256) * ((N + 255) / 256) > 3 * 256) return choice;
  TileEstimates e = tile_estimates(M, N, K, gated);
  if ((choice == 1 && e.rounds[4] > e.rounds[1]) || (choice == 3 && K <= (e.rounds[4] > 1 ? 2048 : 1024))) e.ok[4] = false;
  int best = choice;
  double limit = 0.97 * e.us[choice];
  for (int t = 4; t <= 7; ++t)
    if (e.ok[t] && e.us[t] < limit) best = t, limit = e.us[t];
  return best;
}

// The shape of a product that leaves it to the library. 192 x 192 takes the place of 256 x 128 tiles that all run at once only
// where it is the faster one: for weights whose panel has just been written (prepared ones come from memory, and the
// smaller tiles read them once more: 803 x 8192 x 8192 124 / 136, 696 x 10240 x 8192 126 / 138, 1577 x 4096 x 11008 159 / 162),
// from six rows of 256 on (836 x 8192 x 28672 571 / 584; 752 x 10240 x 8192 184 / 187), with a K beyond 4096 (1805 x 4096 x 14336
// ratio 0.88, 1611 x 4096 x 11008 0.94, 1493 x 4544 x 4544 0.98; but 2029 x 4096 x 4096 64 / 66, 1600 x 4096 x 4096 56.5 / 57.2,
// 3503 x 2048 x 2048 35.2 / 35.6). 192 x 256 does not take that of 256 x 128 in a gated product of up to 768 rows, which are as many
// in tiles of either height (768 x 22016 x 4096 189 / 196).
// whole_lines: every row of C is whole 128-byte lines, or C is BF16. Stores of rows that are not take longer, and in the larger
// tiles there is less beside them: 192 x 256 then takes the place of 64 x 256 only with a K beyond 4096 (1323 x 11008 x 4096 167
// / 183, 2570 x 6144 x 4096 170 / 177;  1124 x 13824 x 5120 ratio 0.93), that of 256 x 128 with one beyond 2048 (1349 x 16384 x
// 2048 144 / 149). (These figures are from before such rows were stored row by row and through the caches; on both sides of
// the lines for them, here and below, 10 of 145 sizes then differed by more than 3 %, in either direction.)
int bf16_tile(int64_t M, int64_t N, int64_t K, int64_t batch, bool gated, bool prepared, bool whole_lines) {
  const int choice = bf16_tile_choice(M, N, batch), refined = bf16_tile_refined(choice, M, N, K, batch, gated);
  const bool one_round = ((M + 255) / 256) * ((N + 127) / 128) <= 256;
  if (choice == 2 && refined == 7 && one_round && (prepared || M <= 1280 || K <= 4096)) return choice;
  if (choice == 2 && refined == 4 && gated && !prepared && M <= 768) return choice;
  if (!whole_lines && refined == 4 && ((choice == 3 && K <= 4096) || (choice == 2 && K <= 2048))) return choice;
  return refined;
}

// Columns of the product (rows of B) that are expanded and multiplied at a time; N: all of them at once. A panel of B of two
// thirds of the last-level cache (256 MB) or more does not stay there until it is read: it is written to memory and read back
// from it. Cut into pieces that go through the same workspace one after the other, more of it stays. A piece is whole rounds of
// tiles, so that the pieces take no more rounds than the whole, as many as fit into 144 MB, or else into 280 MB (not for up to
// four rows of tiles: 800 x 28672 x 8192 483 / 488). whole_lines: every row of C is whole 128-byte lines, or C is BF16. Us per
// call on three sets of buffers in turn, AMXFP4-E5M2, whole / in pieces: 4096 x 28672 x 8192 (448 MB, three pieces of 128 and one
// of 64) 1437 / 1392, 2048 of these rows 870 / 824; 1504 x 28672 x 4096 (224 MB) 352 / 326, 3094 rows 693 / 604; 736 x 22016 x
// 4096 (172 MB) 216 / 201. Five rows of tiles gain most (1192 x 28672 x 8192, pieces of 204, 204 and 40 MB, 783 / 624; 1200 x
// 28672 x 4096 404 / 321), but by their order: the uncut grid of 5 x 112 is dealt in supertiles, whose every XCD leaves three
// rows of eight empty, and in equal runs it takes 637 and 328.
// Every piece ends in a round of stores that nothing overlaps. Whole therefore stay, ratio in pieces / whole over 2846 sizes of
// 520 to 4096 rows (a row of tiles: 256):
//   panels up to 200 MB beyond five rows of tiles (22016 x 4096 1.02 to 1.06; up to there 0.89 to 0.95), but for those near it
//     with a K of 6144 or more (16384 x 6144 0.94 to 1.01, 12288 x 8192 0.92 to 1.00); below 170 MB 0.98 to 1.02
//   products whose last round has hardly any tiles, which overlaps the one before it unless it is a piece of its own (beyond five
//     rows of tiles: 26624 x 4096, 10 x 104 tiles, 1.07;  12288 x 8192, 12 x 48, 1.05;  27648 x 5120, 12 x 108, 1.02)
//   rows of an FP32 C that are no whole lines, whose stores take longer: 28672 x 4096 1.03 to 1.10 at six to twelve rows of tiles,
//     32000 x 4096 1.00 to 1.08, 32001 x 4096 at four rows 1.02 to 1.04; except, for panels of 200 MB and more, three rows and five
//     (0.84 to 1.02) and a K of 8192 (14336 x 8192 0.90 to 1.03, 28672 x 8192 0.84 to 1.02)
// Each output's sum is the same.
int64_t bf16_columns_at_a_time(int tile, int64_t M, int64_t N, int64_t K, int64_t batch, bool whole_lines) {
  const int64_t rows = tile == 4 ? 192 : 256, tiles_m = (M + rows - 1) / rows, tiles_n = (N + 255) / 256;
  const int64_t column_bytes = 256 * round_up(K, kPanelK) * 2;  // of the panel, per column of tiles
  const int64_t panel = tiles_n * column_bytes, mb = int64_t(1) << 20, large_m = (M + 255) / 256;
  if (batch != 1 || (tile != 1 && tile != 4) || panel < 170 * mb) return N;
  if (panel < 200 * mb && large_m > 5 && (panel < 190 * mb || K < 6144)) return N;
  if (large_m > 5 && (tiles_m * tiles_n - 1) % 256 < 64) return N;
  if (!whole_lines && (panel < 200 * mb || (large_m > 3 && large_m != 5 && K < 8192))) return N;
  const int64_t rounds = (tiles_m * tiles_n + 255) / 256;
  for (int64_t most : {144 * mb, 280 * mb}) {
    if (most > 144 * mb && tiles_m < 5) break;
    int64_t best = 0;
    for (int64_t k = 1; k < rounds; ++k) {
      const int64_t cols = 256 * k / tiles_m;  // columns of tiles in k rounds
      if (cols >= tiles_n || cols * column_bytes > most) break;
      const int64_t last = cols == 0 ? 0 : (tiles_n - 1) % cols + 1;
      if (cols > 0 && (tiles_n - last) / cols * k + (tiles_m * last + 255) / 256 <= rounds) best = cols;
    }
    if (best > 0) return best * 256;
  }
  return N;
}

// Estimate of the kernel on prepared weights that stay in the caches, us: the estimate above of the tile that it runs.
double bf16_prepared_us(int64_t M, int64_t N, int64_t K) {
  return tile_estimates(M, N, K, false).us[bf16_tile(M, N, K, 1, false, true, N % 32 == 0)];
}

// Estimate of a call that expands both operands, us, for up to some 800 rows (with what beats_panels() in gemm_stream.hip adds to it, up to
// 1500): B's expansion at the copy rate, and the rounds
// of tiles at the rate of a lone tile (256 x 256 14 ns per unit of K, 256 x 128 9.3, 64 x 256 6.6 to 8 as they fill the
// chip) or the chip's, and half of the store of C, c_bytes per element of M x N. It prices the shape of bf16_tile_choice(), not
// the one between those three that most of these sizes run on. Measured (the same buffers again and again, on that one) /
// estimated: 512 x 4096 x 4096 42 / 44, 512 x 11008 x 4096 65 / 68, 768 x 8192 x 8192 113 / 124, 512 x 13824 x 5120 92 / 102, 512 x
// 4096 x 11008 101 / 109, 448 x 4544 x 4544 48 / 50; with weights that come from memory 39, 69, 150, 127, 114 and 47.
double bf16_path_us(int64_t M, int64_t N, int64_t K, double c_bytes) {
  const int tile = bf16_tile_choice(M, N, 1);
  const int64_t tile_m = tile == 3 ? 64 : 256, tile_n = tile == 2 ? 128 : 256;
  const int64_t tiles = ((M + tile_m - 1) / tile_m) * ((N + tile_n - 1) / tile_n);
  const double fill = tiles < 256 ? (double)tiles / 256.0 : 1.0;
  const double lone = (tile == 1 ? 14.0 : tile == 2 ? 9.3 : 6.6 + 1.4 * fill) * 1e-3 * (double)((tiles + 255) / 256);
  const double full = (double)(tiles * tile_m * tile_n) * 2.0 / 1.25e9;
  return 5.0 + 0.51e-6 * (double)(N * K) + (lone > full ? lone : full) * (double)K + 0.5 * c_bytes * (double)(M * N) / 5.1e6;
}

hipError_t launch_gemm_bf16_path(int scale_kind, bool asym, int64_t group_size, int64_t M, int64_t N, int64_t K,
                                 const uint8_t* A_codes, const uint8_t* A_scales, const uint8_t* B_codes,
                                 const uint8_t* B_scales, const float* A_tensor_pair, const float* B_tensor_pair,
                                 float* C, int64_t ldc, int64_t batch, void* workspace, int tile, hipStream_t s,
                                 const KernelTimer& timer, bool glu, const void* B_panel) {
  const int gs_log2 = group_log2(group_size);
  if (gs_log2 < 0 || !group_divides(K, group_size) || K % 32 != 0) return hipErrorInvalidValue;
  const int64_t Mp = round_up(M, kPanelRows), Np = round_up(N, kPanelRows), Kp = round_up(K, kPanelK);
  uint16_t* Ap = reinterpret_cast<uint16_t*>(workspace);
  uint16_t* own_b = Ap + batch * Mp * Kp;
  hipError_t e = hipSuccess;
  // Expands A and columns n0 .. n0 + n - 1 of the product (rows of B), either, or neither.
  auto expand = [&](bool with_a, bool with_b, int64_t n0, int64_t n) {
    const int64_t Npn = round_up(n, kPanelRows);
    const uint8_t* bc = B_codes + n0 * (K >> 1);
    const uint8_t* bs = B_scales + n0 * groups_per_row(K, gs_log2) * (asym ? 2 : 1);
    if (!with_a || !with_b || (Mp + Npn) / 32 > 65535) {  // one of them, or a grid too tall
      hipError_t r = hipSuccess;
      if (with_a) r = expand_dispatch(scale_kind, asym, gs_log2, A_codes, A_scales, M, K, Mp, Kp, batch, Ap, s);
      if (with_b && r == hipSuccess) r = expand_dispatch(scale_kind, asym, gs_log2, bc, bs, n, K, Npn, Kp, batch, own_b, s);
      return r;
    }
    const ExpandJob ja = {A_codes, A_scales, Ap, M, K, Mp, Kp}, jb = {bc, bs, own_b, n, K, Npn, Kp};
    const dim3 grid((unsigned)((Kp + 255) / 256), (unsigned)((Mp + Npn) / 32), (unsigned)batch);
    auto go = [&]<int SK>() {
      if (asym)
        hipLaunchKernelGGL((expand_pair_kernel<SK, true>), grid, dim3(256), 0, s, ja, jb, gs_log2);
      else
        hipLaunchKernelGGL((expand_pair_kernel<SK, false>), grid, dim3(256), 0, s, ja, jb, gs_log2);
      return hipGetLastError();
    };
    return scale_kind == kScaleE5M2   ? go.template operator()<kScaleE5M2>()
           : scale_kind == kScaleE4M3 ? go.template operator()<kScaleE4M3>()
                                      : go.template operator()<kScaleE8M0Floor>();
  };
  const bool whole_lines = glu || ((reinterpret_cast<uintptr_t>(C) | (uint64_t)ldc * 4) & 127) == 0;
  if (tile == 0) tile = bf16_tile(M, N, K, batch, glu, B_panel != nullptr, whole_lines);  // (an option overrides it)
  const int64_t columns = B_panel ? N : bf16_columns_at_a_time(tile, M, N, K, batch, whole_lines);
  for (int64_t n0 = 0; n0 < N; n0 += columns) {
    const int64_t n = N - n0 < columns ? N - n0 : columns, Npn = columns < N ? round_up(n, kPanelRows) : Np;
    if ((e = expand(n0 == 0, !B_panel, n0, n)) != hipSuccess) return e;
    if (n0 == 0 && timer.start && (e = hipEventRecord(timer.start, s)) != hipSuccess) return e;
    const uint16_t* Bp = B_panel ? reinterpret_cast<const uint16_t*>(B_panel) : own_b;
    float* Cn = glu ? reinterpret_cast<float*>(reinterpret_cast<uint16_t*>(C) + (n0 >> 1)) : C + n0;
    auto go = [&]<int WM, int WN, int FM, int FN>() {
      return launch_tiles<WM, WN, FM, FN>(Ap, Bp, Cn, M, n, Mp, Npn, Kp, ldc, batch, A_tensor_pair, B_tensor_pair, glu, s);
    };
    switch (tile) {
      case 2: e = go.template operator()<4, 1, 2, 4>(); break;  // 256 x 128
      case 3: e = go.template operator()<1, 4, 2, 2>(); break;  // 64 x 256
      case 4: e = go.template operator()<2, 2, 3, 4>(); break;  // 192 x 256
      case 5: e = go.template operator()<2, 2, 3, 2>(); break;  // 192 x 128
      case 6: e = go.template operator()<2, 2, 2, 2>(); break;  // 128 x 128
      case 7: e = go.template operator()<2, 2, 3, 3>(); break;  // 192 x 192
      default: e = go.template operator()<2, 2, 4, 4>();        // 256 x 256
    }
    if (e != hipSuccess) return e;
  }
  if (timer.stop) e = hipEventRecord(timer.stop, s);
  return e;
}

hipError_t launch_expand_b_panel(int scale_kind, bool asym, int64_t group_size, int64_t N, int64_t K,
                                 const uint8_t* B_codes, const uint8_t* B_scales, void* panel, hipStream_t s) {
  const int gs_log2 = group_log2(group_size);
  if (gs_log2 < 0 || !group_divides(K, group_size) || K % 32 != 0) return hipErrorInvalidValue;
  return expand_dispatch(scale_kind, asym, gs_log2, B_codes, B_scales, N, K, round_up(N, kPanelRows), round_up(K, kPanelK),
                         1, reinterpret_cast<uint16_t*>(panel), s);
}

}  // namespace amx
