// Pieces shared by the GEMM kernels: the merge of a workgroup's K slices and
// the epilogues.
#pragma once

#include "device_common.h"
#include "griffin_internal.h"

namespace griffin {

// Merge the KS K slices of a workgroup in slice order through LDS (red: at
// least WN * NB * MB * 4 KB, free: every wave's reads of it have returned).  Every
// wave of the workgroup calls it (its barriers are uniform); waves whose kh
// is not a slice index only take part in the barriers.  Slice 0 ends with the
// sum.
template <int NB, int WN, int KS, int MB>
__device__ __forceinline__ void ks_merge(f32x16 (&acc)[NB][MB], float* red, int kh, int wc, int lane) {
  wait_vmcnt_lds<0>();
  __builtin_amdgcn_s_barrier();
  for (int k = 1; k < KS; ++k) {
    if (kh == k) {
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
          for (int i = 0; i < 16; ++i) red[(((wc * NB + b) * MB + mb) * 16 + i) * 64 + lane] = acc[b][mb][i];
    }
    wait_vmcnt_lds<0>();
    __builtin_amdgcn_s_barrier();
    if (kh == 0) {
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
          for (int i = 0; i < 16; ++i) acc[b][mb][i] += red[(((wc * NB + b) * MB + mb) * 16 + i) * 64 + lane];
    }
    wait_vmcnt_lds<0>();
    __builtin_amdgcn_s_barrier();
  }
}

// Columns n .. n + 3 (n a multiple of 4) of an output row of N: as one store, or
// where rows of N values are no whole number of 16-byte groups (a vocabulary or
// a fusion width that is no multiple of 4) one by one, since the row's last group
// would reach into the next row, or past the caller's buffer.
__device__ __forceinline__ void store_cols(float* row, int n, int N, float x, float y, float z, float w) {
  if (N % 4 == 0) {  // uniform
    if (n < N) *reinterpret_cast<float4*>(row + n) = make_float4(x, y, z, w);
    return;
  }
  if (n < N) row[n] = x;
  if (n + 1 < N) row[n + 1] = y;
  if (n + 2 < N) row[n + 2] = z;
  if (n + 3 < N) row[n + 3] = w;
}

// The epilogues, every wave for its own NB column blocks of the 32 MB rows from row0.
template <int EPI, int NB, int WN, int MB>
__device__ __forceinline__ void gemm_epilogue(const GemmArgs& a, f32x16 (&acc)[NB][MB], int e, int row0, int wg,
                                              int wc, int zsplit, int rows_e, int lane) {
  const int lr = lane & 31, g = lane >> 5;
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
    const int ml = row0 + mb * 32 + lr;  // row of the (expert's) operand
    const bool row_ok = ml < rows_e;
    const long long orow = (long long)e * a.o_erows + ml;
    if constexpr (EPI == EPI_STORE) {
      if (!row_ok) continue;
      float* out = a.out + (long long)zsplit * a.out_split_stride + orow * a.ldo;
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int rg = 0; rg < 4; ++rg) {
          const int n = ((wg * WN + wc) * NB + b) * 32 + 8 * rg + 4 * g;
          store_cols(out, n, a.N, acc[b][mb][4 * rg], acc[b][mb][4 * rg + 1], acc[b][mb][4 * rg + 2],
                     acc[b][mb][4 * rg + 3]);
        }
    } else if constexpr (EPI == EPI_SWIGLU) {
      // blocks [0, NB/2) hold gate rows, block b + NB/2 the up rows of block b
      static_assert(EPI != EPI_SWIGLU || NB % 2 == 0, "SwiGLU pairs gate and up blocks");
      constexpr int HB = NB / 2;
      if (!row_ok) continue;
#pragma unroll
      for (int hb = 0; hb < HB; ++hb)
#pragma unroll
        for (int rg = 0; rg < 4; ++rg) {
          const int n = ((wg * WN + wc) * HB + hb) * 32 + 8 * rg + 4 * g;
          if (n < a.N) {
            // the product rounds before its split into hi + lo: contracted into
            // the subtraction, or not, as the compiler chooses per kernel form,
            // a row's bits would depend on the form that computed it
#pragma clang fp contract(off)
            float h[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) h[i] = silu_f32(acc[hb][mb][4 * rg + i]) * acc[hb + HB][mb][4 * rg + i];
            uint16_t* dst = a.act + xpack_off(orow, n, a.act_ks);
            const Hilo2 p0 = pack_hilo2(h[0], h[1]), p1 = pack_hilo2(h[2], h[3]);
            *reinterpret_cast<uint2*>(dst) = make_uint2(p0.hi, p1.hi);
            *reinterpret_cast<uint2*>(dst + XPACK_LO) = make_uint2(p0.lo, p1.lo);
          }
        }
    } else {  // EPI_ARGMAX: partial (max, argmax, second max, NaN count) over this wave's columns
      float best = -INFINITY, second = -INFINITY;
      int bidx = 0x7fffffff;
      int nan_cnt = 0;
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int rg = 0; rg < 4; ++rg)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int n = ((wg * WN + wc) * NB + b) * 32 + 8 * rg + 4 * g + i;
            const float v = acc[b][mb][4 * rg + i];
            if (n < a.N) {
              if (v != v) ++nan_cnt;
              else top2_push(best, bidx, second, v, n);
            }
          }
      const float ob = __shfl_xor(best, 32, 64);
      const int oi = __shfl_xor(bidx, 32, 64);
      const float os = __shfl_xor(second, 32, 64);
      nan_cnt += __shfl_xor(nan_cnt, 32, 64);
      top2_merge(best, bidx, second, ob, oi, os);
      const int part = wg * WN + wc;
      if (g == 0) {
        a.pmax[orow * a.ld_part + part] = best;
        a.pmax2[orow * a.ld_part + part] = second;
        a.pidx[orow * a.ld_part + part] = bidx;
        a.pnan[orow * a.ld_part + part] = nan_cnt;
      }
      if (a.logits && orow < a.logit_rows && orow % a.max_tree < a.n_nodes[orow / a.max_tree]) {
        float* out = a.logits + orow * a.ld_logits;
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
          for (int rg = 0; rg < 4; ++rg) {
            const int n = ((wg * WN + wc) * NB + b) * 32 + 8 * rg + 4 * g;
            store_cols(out, n, a.N, acc[b][mb][4 * rg], acc[b][mb][4 * rg + 1], acc[b][mb][4 * rg + 2],
                       acc[b][mb][4 * rg + 3]);
          }
      }
    }
  }
}

}  // namespace griffin
