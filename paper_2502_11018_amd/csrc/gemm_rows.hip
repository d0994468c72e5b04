// GEMM of the verify pass over several 64-row tiles (batched trees):
// out = X W^T with X in split bf16 (hi + lo).  From 128 rows on a weight byte
// feeds 256 flop and more, so the matrix cores bound the launch and not the
// weight stream, and the kernel is shaped around keeping them fed:
//
// * Eight waves a workgroup, two per SIMD at 256 registers each, so that one
//   wave's waits and address work run under the other's MFMAs.  Each wave owns
//   a 64-row x 128-column tile (8 accumulators of 32x32) of one K slice:
//   WM x WN x KS = 8 waves cover 64 WM rows x 128 WN columns with KS waves
//   sharing the K range of a tile, merged in slice order in LDS at the end.
//   The tile shape is chosen per step from the number of row tiles
//   (plan_rows in host.cpp) so that the launch fills the 256 CUs.
// * Weights and activations both travel by LDS DMA into a ring of S stages.  A
//   stage is one 16-deep MFMA step of every slice (1 KB pieces in fragment
//   order: each operand is one conflict-free ds_read_b128).  Per stage a wave
//   reads 4 weight and 4 activation pieces for 16 MFMAs, half of what LDS
//   delivers in that time.
// * The fragments of stage t + 1 are read while stage t multiplies, and stages
//   t + 2 .. t + S are in flight from memory.
//
// Weights are packed per group of 128 rows (PackShape::group_major): group g,
// K step t, block b at ((g * ks + t) * 4 + b) * 2048, in the fragment order of
// gemm.hip.  The layout does not depend on the tile shape or on K splits, so
// one packing serves every step of a context.  One K step of a group is 16 KB,
// as is one K step of a row tile of split activations: all DMA sources advance
// by the same stride.

// Measured per launch at the Llama-3-8B shapes, against gemm.hip's two-tile
// form (four column blocks a wave, one wave per SIMD at 476 registers, a fixed
// tile shape) that this replaced: gate/up at 256 rows 203 -> 105 us, at 512
// rows 235 -> 204 us; LM head 485 -> 438 and 975 -> 932 us; the fixed shape had
// 112 workgroups at 256 rows.  Back to back the launches run at 1.1-1.25
// PFLOP/s of executed MFMA work with the shader clock down to 1.6-1.8 GHz; the
// same loop without its DMA reaches 1.42, one wave per SIMD over 128 x 128
// tiles or weights loaded past LDS into registers 0.95-1.16.

#include "gemm_common.h"

namespace griffin {

template <int WM, int WN, int KS, bool XLO>
struct RowsShape {
  static constexpr int XH = XLO ? 2 : 1;
  static constexpr int XPC = WM * XH * 2 * KS;  // activation pieces per stage
  static constexpr int WPC = WN * 4 * KS;       // weight pieces per stage
  static constexpr int PC = XPC + WPC;
  static constexpr int PPW = PC / 8;            // pieces each wave moves per stage
  static constexpr int S = 144 / PC > 6 ? 6 : 144 / PC;
  static constexpr int SUB = 4 / KS;            // stages per 64-deep K step
  static_assert(WM * WN * KS == 8 && PC % 8 == 0 && S >= 3, "eight waves, whole pieces per wave");
  static_assert(KS == 1 || WM * WN * 32 <= S * PC, "the slice merge fits the ring");
};

template <int EPI, int WM, int WN, int KS, bool XLO>
__global__ __launch_bounds__(512, 2) void gemm_rows_kernel(GemmArgs a) {
  using R = RowsShape<WM, WN, KS, XLO>;
  constexpr int XH = R::XH, S = R::S, PPW = R::PPW, SUB = R::SUB;
  __shared__ u32x4 ring[S][R::PC][64];

  stamp_begin(a.stamp);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int kh = wave / (WM * WN), wt = wave % (WM * WN);
  const int wm = wt / WN, wn = wt % WN;
  // XCD-aware decode as in gemm.hip: the row groups that stream the same
  // weights get the same id % 8
  const int groups = (a.m_tiles + WM - 1) / WM;
  int mg = 0, wg = blockIdx.x;
  if (groups > 1) {
    const int grp = blockIdx.x / (8 * groups), r = blockIdx.x % (8 * groups);
    mg = r >> 3;
    wg = grp * 8 + (r & 7);
    if (wg >= a.n_wgs) return;  // padding of the grid to a multiple of 8 (uniform)
  }
  const int zsplit = blockIdx.z;
  const int tile0 = mg * WM;
  const int step0 = zsplit * a.len;
  const int steps = min(a.len, a.ks - step0);  // K steps of this split
  const int NT = steps * SUB;                  // stages

  // sources of the pieces this wave moves, at stage 0
  const uint16_t* src[PPW];
#pragma unroll
  for (int i = 0; i < PPW; ++i) {
    const int p = wave * PPW + i;
    if (p < R::XPC) {  // [tile][plane][row half][slice]
      const int k = p % KS, mb = p / KS % 2, h = p / (KS * 2) % XH, t = p / (KS * 2 * XH);
      src[i] = a.X + ((long long)min(tile0 + t, a.m_tiles - 1) * a.x_ks + step0) * XPACK_STEP + h * XPACK_LO +
               mb * 2048 + k * 512;
    } else {  // [column group][block][slice]
      const int pw = p - R::XPC;
      const int k = pw % KS, b = pw / KS % 4, g = pw / (KS * 4);
      src[i] = a.W + ((long long)(wg * WN + g) * a.ks + step0) * 8192 + b * 2048 + k * 512;
    }
  }
  auto issue = [&](int slot, int t) {
    t = min(t, NT - 1);  // past the end: re-read the last stage into a slot that is not read again
    const int off = (t / SUB) * XPACK_STEP + (t % SUB) * (KS * 512);
#pragma unroll
    for (int i = 0; i < PPW; ++i)
      __builtin_amdgcn_global_load_lds((const void*)(src[i] + off + lane * 8),
                                       (lds_void*)&ring[slot][wave * PPW + i][0], 16, 0, 0);
  };

  f32x16 acc[4][2];
#pragma unroll
  for (int b = 0; b < 4; ++b)
#pragma unroll
    for (int mb = 0; mb < 2; ++mb)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[b][mb][i] = 0.f;

  u32x4 wf[2][4], xf[2][XH][2];
  auto read = [&](int set, int slot) {
#pragma unroll
    for (int h = 0; h < XH; ++h)
#pragma unroll
      for (int mb = 0; mb < 2; ++mb) xf[set][h][mb] = ring[slot][((wm * XH + h) * 2 + mb) * KS + kh][lane];
#pragma unroll
    for (int b = 0; b < 4; ++b) wf[set][b] = ring[slot][R::XPC + (wn * 4 + b) * KS + kh][lane];
  };
  auto multiply = [&](int set) {
#pragma unroll
    for (int h = 0; h < XH; ++h)
#pragma unroll
      for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int mb = 0; mb < 2; ++mb)
          acc[b][mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(wf[set][b]), as_bf16x8(xf[set][h][mb]),
                                                               acc[b][mb], 0, 0, 0);
  };

  // Stages 0 .. S-1 go out at once.  At the top of stage t a wave waits for its
  // fragments of stage t (read during stage t - 1) and for its own DMA of
  // stage t + 1; the barrier then publishes stage t + 1 and frees slot t % S,
  // whose readers all hold their fragments, for stage t + S.
#pragma unroll
  for (int s = 0; s < S; ++s) issue(s, s);
  wait_vmcnt_lds<(S - 1) * PPW>();
  __builtin_amdgcn_s_barrier();
  read(0, 0);
  int slot = 0;  // t % S
  auto stage = [&](int set, int t) {
    wait_vmcnt_lds<(S - 2) * PPW>();
    __builtin_amdgcn_s_barrier();
    const int next = slot + 1 == S ? 0 : slot + 1;
    read(set ^ 1, next);  // past the end: a slot that holds old or repeated data, never multiplied
    issue(slot, t + S);
    multiply(set);
    // issue order: left alone the compiler moves the reads behind the MFMAs,
    // next to their use, and every stage then waits for LDS.  The DMA, which
    // has S - 1 stages to land, goes behind the reads (1-2 % over before them).
#pragma unroll
    for (int i = 0; i < 4 + 2 * XH; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);  // an LDS read
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // an MFMA
    }
#pragma unroll
    for (int i = 0; i < PPW; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);  // a DMA
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    slot = next;
  };
  int t = 0;
  for (; t + 2 <= NT; t += 2) {
    stage(0, t);
    stage(1, t + 1);
  }
  if (t < NT) stage(0, t);  // uniform
  wait_vmcnt_lds<0>();  // every DMA has landed before the ring is reused or released

  if constexpr (KS > 1) {
    ks_merge<4, WM * WN, KS>(acc, reinterpret_cast<float*>(&ring[0][0][0]), kh, wt, lane);
    if (kh != 0) return;
  }
  if (tile0 + wm < a.m_tiles)
    gemm_epilogue<EPI, 4, 1>(a, acc, 0, (tile0 + wm) * 64, wg * WN + wn, 0, zsplit, a.m_tiles * 64, lane);
  stamp_end(a.stamp);
}

template <int EPI, int WM, int WN, int KS>
static hipError_t launch_shape(const GemmArgs& a, hipStream_t s) {
  const int groups = (a.m_tiles + WM - 1) / WM;
  const dim3 grid(groups > 1 ? (a.n_wgs + 7) / 8 * 8 * groups : a.n_wgs, 1, a.splits);
  if (a.xlo)
    hipLaunchKernelGGL((gemm_rows_kernel<EPI, WM, WN, KS, true>), grid, dim3(512), 0, s, a);
  else
    hipLaunchKernelGGL((gemm_rows_kernel<EPI, WM, WN, KS, false>), grid, dim3(512), 0, s, a);
  return hipGetLastError();
}

template <int EPI>
static hipError_t launch_epi(const GemmArgs& a, hipStream_t s) {
  switch (a.rows_wm * 10 + a.rows_wn) {
    case 42: return launch_shape<EPI, 4, 2, 1>(a, s);
    case 22: return launch_shape<EPI, 2, 2, 2>(a, s);
    case 21: return launch_shape<EPI, 2, 1, 4>(a, s);
    case 12: return launch_shape<EPI, 1, 2, 4>(a, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_gemm_rows(const GemmArgs& a, hipStream_t s) {
  // every split has at least one K step
  if (a.m_tiles < 1 || a.splits < 1 || a.len < 1 || (a.splits - 1) * a.len >= a.ks || a.x_ks < a.ks)
    return hipErrorInvalidValue;
  switch (a.epi) {
    case EPI_STORE: return launch_epi<EPI_STORE>(a, s);
    case EPI_SWIGLU: return launch_epi<EPI_SWIGLU>(a, s);
    case EPI_ARGMAX: return launch_epi<EPI_ARGMAX>(a, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace griffin
