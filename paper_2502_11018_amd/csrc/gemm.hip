// Skinny bf16 GEMM of the verify pass: out = X W^T, X the activations of the
// tree rows ([rows][K], 64 rows per tile) and W a weight matrix [N][K] that is
// streamed once from HBM.  With ~64 rows the weights carry almost all the
// traffic (64 flop per weight byte, far below the MFMA ridge), so the kernel is
// shaped around keeping HBM busy:
//
// * Weights are repacked once (at context creation) into fragment order: a
//   block of 32 rows x 64 K (4 KB) holds, for piece j = 0..3 and lane
//   l = r + 32 g, the 8 values W[32 nb + r][64 s + 32 g + 8 j + 0..7] at
//   element j * 512 + 8 l, so one wave instruction reads one contiguous KB that
//   is directly an MFMA operand.  Blocks are laid out step-major over the
//   launch's wave streams (block (t, q, b) at ((t * Q + q) * NB + b) * 2048),
//   so at any moment all waves read one compact window of the matrix, the way
//   a plain streaming copy does.
// * Activations are produced in the same fragment order by the kernels that
//   write them (RMSNorm, attention merge, SwiGLU epilogue).  A workgroup's WN
//   waves own different weight rows over the same K range, so each 8 KB
//   activation stage is loaded once per workgroup into an LDS ring of PF slots
//   and read by all waves.
// * Each wave keeps PF - 1 stages of weight loads in flight in registers; the
//   main loop has no data-dependent branches.
//
// MFMA: v_mfma_f32_32x32x16_bf16 with A = weight rows, B = activation rows.
// Piece j of lane (r, g) feeds MFMA j, so MFMA j sums k in
// {64 s + 8 j + [0,8)} U {64 s + 32 + 8 j + [0,8)}: both operands use the same
// permutation of K and every dot product is unchanged.  Output layout (lane l,
// register i): m = l % 32, n = 8 (i / 4) + 4 (l / 32) + (i % 4).
//
// K is split across `splits` workgroups; each split writes fp32 partial sums
// that the consumer kernel adds in split order (no atomics, reproducible).

#include "gemm_common.h"

namespace griffin {

// Half tiles: a step with at most 32 live rows (short chains, small trees, a
// draft's frontier, plain decoding) or an expert that was routed no more
// stages and multiplies one 32-row half.  The activation pieces come through
// the same L1 queue as the weights, byte for byte as many of them in a full
// tile, so halving them is worth more than the MFMAs they feed: Mixtral-8x7B
// shape, 61 rows over 8 experts, 4 layers: step 2516 -> 2392 us; a draft's
// catch-up on 5 tokens 98.8 -> 88.4 us, its 60-token tree (with only the new
// nodes' half per pass) 3398 -> 3073 us.  An expert's count is only known on
// the device, so its kernel holds both forms and picks by the count.

// LDS bytes of the activation ring: per slot and slice {hi, lo} (XLO) or {hi}
// x MB row halves x 4 pieces of 1 KB.
template <int PF, int KS, bool XLO, int MB>
constexpr int kRingPieces = PF * KS * 4 * MB * (XLO ? 2 : 1);

// One workgroup's part of the product for MB 32-row halves from half mb0 of
// row tile m_tile.
template <int EPI, int NB, int WN, int PF, int KS, bool XLO, bool NT_W, int MB>
__device__ __forceinline__ void gemm_body(const GemmArgs& a, u32x4* ring, int e, int m_tile, int mb0, int wg,
                                          int rows_e) {
  constexpr int XH = XLO ? 2 : 1;
  constexpr int XPIECES = 4 * MB * XH;
  constexpr int XP = XPIECES / WN;          // activation pieces each wave stages per step
  constexpr int LOADS = NB * 4 + XP;        // vector-memory instructions per stage per wave
  static_assert(LOADS * (PF - 2) < 64, "wait count out of range");
  static_assert(PF >= 2 && XPIECES % WN == 0, "pipeline shape");
  static_assert(WN * NB * 4 * MB <= PF * KS * XPIECES || KS == 1, "K-split merge buffer");
  u32x4(&xs)[PF][KS][XPIECES][64] = *reinterpret_cast<u32x4(*)[PF][KS][XPIECES][64]>(ring);

  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wc = wave % WN;            // column group of this wave
  const int kh = wave / WN;            // K slice of this wave inside the workgroup
  const int zsplit = blockIdx.z;       // output split (its KS slices are merged in the workgroup)
  const int split = zsplit * KS + kh;  // K slice of this wave's weight stream

  const long long Q = (long long)a.n_wgs * a.splits * WN;
  const long long q = ((long long)split * a.n_wgs + wg) * WN + wc;
  const uint16_t* W = a.W + (long long)e * a.w_estride + q * NB * 2048 + lane * 8;
  const long long wstep = Q * NB * 2048;  // elements between consecutive steps of a stream
  const uint16_t* X = a.X + ((long long)(e * a.x_etiles + m_tile) * a.x_ks + (long long)zsplit * KS * a.len) * XPACK_STEP +
                      mb0 * 2048 + lane * 8;

  f32x16 acc[NB][MB];
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[b][mb][i] = 0.f;

  // Stage t: this wave's weight blocks into registers, its share of the
  // activation stage straight into LDS slot t % PF (lane l's 16
  // bytes land at the piece base + 16 l, which is the fragment order).
  // NT_W: non-temporal weight loads (see launch_gemm for where they are used)
  u32x4 wb[PF][NB][4];
  auto issue = [&](u32x4 (&wv)[NB][4], int slot, int t) {
    const uint16_t* wp = W + t * wstep;
    if constexpr (NT_W) {
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int b = 0; b < NB; ++b) wv[b][j] = ld_u4_nt(wp + b * 2048 + j * 512);
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int b = 0; b < NB; ++b) wv[b][j] = ld_u4(wp + b * 2048 + j * 512);
    }
#pragma unroll
    for (int p = 0; p < XP; ++p) {
      const int pp = wave * XP + p, sk = pp / XPIECES, pc = pp % XPIECES;  // slice, piece
      const int src = pc / (4 * MB) * XPACK_LO + pc % (4 * MB) * 512;       // plane, half and piece in the packed step
      __builtin_amdgcn_global_load_lds((const void*)(X + ((long long)sk * a.len + t) * XPACK_STEP + src),
                                       (lds_void*)&xs[slot][sk][pc][0], 16, 0, 0);
    }
  };
  // Consume stage t from slot u: the weights times the activation's bf16 high
  // part plus, with XLO, its bf16 low part (two MFMAs into one accumulator).
  auto compute = [&](int u) {
    u32x4 xv[XH][MB][4];
#pragma unroll
    for (int h = 0; h < XH; ++h)
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int j = 0; j < 4; ++j) xv[h][mb][j] = xs[u][kh][(h * MB + mb) * 4 + j][lane];
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int h = 0; h < XH; ++h)
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
          for (int mb = 0; mb < MB; ++mb)
            acc[b][mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(wb[u][b][j]), as_bf16x8(xv[h][mb][j]),
                                                                 acc[b][mb], 0, 0, 0);
  };

  // Pipeline: stages t+1 .. t+PF-2 stay in flight while stage t is consumed.
  // At the top of iteration t the wave waits for its own stage-t loads
  // (vector-memory counters retire in issue order) and for its LDS reads of
  // slot (t-1) % PF; the barrier then makes every wave's share of stage t
  // visible and guarantees that no wave still reads slot (t-1) % PF, which
  // stage t+PF-1 overwrites.  A plain s_barrier: the explicit waits are the
  // only ones needed (a fence would drain all loads in flight).
  const int len = a.len;
#pragma unroll
  for (int p = 0; p < PF - 1; ++p) issue(wb[p], p, min(p, len - 1));
  int base = 0;
  for (; base + PF <= len; base += PF) {
#pragma unroll
    for (int u = 0; u < PF; ++u) {
      wait_vmcnt_lds<(PF - 2) * LOADS>();
      __builtin_amdgcn_s_barrier();
      issue(wb[(u + PF - 1) % PF], (u + PF - 1) % PF, min(base + u + PF - 1, len - 1));
      compute(u);
    }
  }
  const int rem = len - base;  // < PF steps, already issued into slots 0 .. rem-1 (uniform)
  wait_vmcnt_lds<0>();
  __builtin_amdgcn_s_barrier();
#pragma unroll
  for (int u = 0; u < PF - 1; ++u)
    if (u < rem) compute(u);

  if constexpr (KS > 1) {
    ks_merge<NB, WN, KS>(acc, reinterpret_cast<float*>(&xs[0][0][0][0]), kh, wc, lane);
    if (kh != 0) return;
  }
  gemm_epilogue<EPI, NB, WN>(a, acc, e, m_tile * 64 + mb0 * 32, wg, wc, zsplit, rows_e, lane);
}

enum GemmRows { FULL_TILES, HALF_TILE, BY_COUNT };

template <int EPI, int NB, int WN, int PF, int KS, bool XLO, bool NT_W, int ROWS>
__global__ __launch_bounds__(64 * WN * KS) void gemm_kernel(GemmArgs a) {
  __shared__ u32x4 ring[kRingPieces<PF, KS, XLO, ROWS == HALF_TILE ? 1 : 2>][64];
  stamp_begin(a.stamp);
  const int e = blockIdx.y;
  // XCD-aware decode: workgroups are dispatched round-robin over the 8 XCDs
  // (linear id % 8, and the grid's x extent is a multiple of 8), so the
  // workgroups of the row tiles that stream the same weights get the same
  // id % 8 and the re-reads of those weights hit that XCD's L2.
  int m_tile = 0, wg = blockIdx.x;
  if (a.m_tiles > 1) {
    const int grp = blockIdx.x / (8 * a.m_tiles), r = blockIdx.x % (8 * a.m_tiles);
    m_tile = r >> 3;
    wg = grp * 8 + (r & 7);
    if (wg >= a.n_wgs) return;  // padding of the grid to a multiple of 8 (uniform)
  }
  const int rows_e = ROWS == BY_COUNT ? a.count[e] : a.m_tiles * 64;
  if (m_tile * 64 >= rows_e) return;  // uniform over the workgroup
  u32x4* r0 = &ring[0][0];
  if constexpr (ROWS == HALF_TILE) {
    gemm_body<EPI, NB, WN, PF, KS, XLO, NT_W, 1>(a, r0, e, m_tile, a.half - 1, wg, rows_e);
  } else {
    if (ROWS == BY_COUNT && rows_e - m_tile * 64 <= 32)  // uniform
      gemm_body<EPI, NB, WN, PF, KS, XLO, NT_W, 1>(a, r0, e, m_tile, 0, wg, rows_e);
    else
      gemm_body<EPI, NB, WN, PF, KS, XLO, NT_W, 2>(a, r0, e, m_tile, 0, wg, rows_e);
  }
  stamp_end(a.stamp);
}

template <int EPI, int NB, int WN, int PF, int KS, bool XLO, bool NT_W, int ROWS>
static hipError_t launch_rows(const GemmArgs& a, int experts, hipStream_t s) {
  const int gx = a.m_tiles > 1 ? (a.n_wgs + 7) / 8 * 8 * a.m_tiles : a.n_wgs;
  dim3 grid(gx, experts, a.splits / KS);
  hipLaunchKernelGGL((gemm_kernel<EPI, NB, WN, PF, KS, XLO, NT_W, ROWS>), grid, dim3(64 * WN * KS), 0, s, a);
  return hipGetLastError();
}

template <int EPI, int NB, int WN, int PF, int KS, bool XLO, bool NT_W>
static hipError_t launch_one(const GemmArgs& a, int experts, hipStream_t s) {
  if (a.count) {  // experts: no LM head
    if constexpr (EPI != EPI_ARGMAX) return launch_rows<EPI, NB, WN, PF, KS, XLO, NT_W, BY_COUNT>(a, experts, s);
    return hipErrorInvalidValue;
  }
  if (a.half) return launch_rows<EPI, NB, WN, PF, KS, XLO, NT_W, HALF_TILE>(a, experts, s);
  return launch_rows<EPI, NB, WN, PF, KS, XLO, NT_W, FULL_TILES>(a, experts, s);
}

hipError_t launch_gemm(const GemmArgs& a, int experts, hipStream_t s) {
  const int epi = a.epi, nb = a.nb, wn = a.wn, pf = a.pf, ks = a.kslices;
  if (ks < 1 || a.splits % ks != 0) return hipErrorInvalidValue;
  if (a.half < 0 || a.half > 2 || (a.half && (a.m_tiles != 1 || a.count))) return hipErrorInvalidValue;
  // Non-temporal weight loads where they measured faster: the two-slice store
  // form (down) and the LM head (189 -> 182 us).  The one-slice store and the
  // SwiGLU forms measured slower with them.
#define GRIFFIN_GEMM_CASE(E, B, N_, P, K_)                                                             \
  if (epi == (E) && nb == (B) && wn == (N_) && pf == (P) && ks == (K_)) {                             \
    constexpr bool nt = (E) == EPI_ARGMAX || ((E) == EPI_STORE && (K_) == 2);                         \
    return a.xlo ? launch_one<E, B, N_, P, K_, true, nt>(a, experts, s)                               \
                 : launch_one<E, B, N_, P, K_, false, nt>(a, experts, s);                             \
  }
  GRIFFIN_GEMM_CASE(EPI_STORE, 1, 4, 4, 1)
  GRIFFIN_GEMM_CASE(EPI_STORE, 1, 4, 2, 1)
  GRIFFIN_GEMM_CASE(EPI_STORE, 1, 4, 3, 2)
  GRIFFIN_GEMM_CASE(EPI_SWIGLU, 2, 2, 3, 2)
  GRIFFIN_GEMM_CASE(EPI_SWIGLU, 2, 2, 2, 2)
  GRIFFIN_GEMM_CASE(EPI_SWIGLU, 2, 2, 2, 1)
  GRIFFIN_GEMM_CASE(EPI_ARGMAX, 2, 4, 4, 1)
  GRIFFIN_GEMM_CASE(EPI_ARGMAX, 2, 4, 2, 1)
#undef GRIFFIN_GEMM_CASE
  return hipErrorInvalidValue;
}

// ---------------------------------------------------------- weight packing ----
// One thread per 16-byte piece of the packed matrix: decode its (step, stream,
// block, piece, lane), read the 8 source values (zero outside [rows, K)).
__global__ __launch_bounds__(256) void pack_weight_kernel(const uint16_t* __restrict__ src, int rows, int K,
                                                          PackShape p, uint16_t* __restrict__ dst,
                                                          long long pieces) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= pieces) return;
  const int lane = (int)(i & 63);
  const int j = (int)((i >> 6) & 3);
  long long blk = i >> 8;  // ((t * Q + q) * nb + b), or ((q * len + t) * nb + b) group-major
  const int b = (int)(blk % p.nb);
  blk /= p.nb;
  const long long Q = (long long)p.n_wgs * p.splits * p.wn;
  const int q = (int)(p.group_major ? blk / p.len : blk % Q);
  const int t = (int)(p.group_major ? blk % p.len : blk / Q);
  const int wave = q % p.wn;
  const int rest = q / p.wn;
  const int wg = rest % p.n_wgs;
  const int split = rest / p.n_wgs;
  const int s = split * p.len + t;
  const int r = lane & 31, gg = lane >> 5;
  long long row;
  bool ok;
  if (p.swiglu) {  // blocks [0, nb/2): gate rows of the wave's column blocks; b + nb/2: their up rows
    const int hb = p.nb / 2;
    const int c = ((wg * p.wn + wave) * hb + b % hb) * 32 + r;
    ok = c < p.n_out;
    row = c + (b >= hb ? p.n_out : 0);
  } else {
    row = ((long long)(wg * p.wn + wave) * p.nb + b) * 32 + r;
    ok = row < rows;
  }
  const int k = s * 64 + 32 * gg + 8 * j;
  ok = ok && k < K;
  u32x4 v = zero_u4();
  if (ok && K % 8 == 0) {
    v = *reinterpret_cast<const u32x4*>(src + row * K + k);
  } else if (ok) {  // rows of any length (a draft's fusion width): the last piece ends inside the row
#pragma unroll
    for (int e = 0; e < 8; ++e)
      if (k + e < K) v[e / 2] |= (uint32_t)src[row * K + k + e] << (e % 2 * 16);
  }
  *reinterpret_cast<u32x4*>(dst + i * 8) = v;
}

hipError_t launch_pack_weight(const uint16_t* src, int rows, int K, const PackShape& p, uint16_t* dst,
                              hipStream_t s) {
  const long long pieces = packed_elems(p) / 8;
  const long long grid = (pieces + 255) / 256;
  hipLaunchKernelGGL(pack_weight_kernel, dim3((unsigned)grid), dim3(256), 0, s, src, rows, K, p, dst, pieces);
  return hipGetLastError();
}

}  // namespace griffin
