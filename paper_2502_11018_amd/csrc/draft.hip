// GRIFFIN-style draft model: the kernels around its decoder layer.
//
// The draft (Sec. 4.2) fuses an input feature F with the token embedding e in
// Token-Guided Fusion, runs one decoder layer, and splits the result in the
// Token-Enhanced Head:
//   h = [F, e] W_m + b_m;  z = [LN(h), LN(e)] W_u + b_u;  o = SiLU(z) W_d + b_d + h
//   y = decoder layer(o);  F^P = y W_p + b_p;  F^R = y W_r + b_r
//   logits = RMSNorm(F^P) (the target's final norm) times the target's LM head
// The four matrices go through the library's GEMM (split-K partials, fp32);
// the kernels here sum those partials in split order, add biases, normalise
// and write the next GEMM's split-bf16 operand.  Rows are b * max_tree + i;
// rows of absent nodes get zero operands.  A node's input feature is its
// parent's regress feature from the previous draft pass (the root's is the
// caller's), unless the caller gives every node's feature (a draft catching
// up on accepted tokens with the target's features).

#include "device_common.h"
#include "draft.h"
#include "griffin_internal.h"

namespace griffin {

constexpr int DT = 256;   // threads per workgroup of the elementwise kernels
constexpr int DR = 1024;  // threads per workgroup of the per-row reductions (LayerNorm, RMSNorm)

__device__ __forceinline__ bool draft_live(const StepMeta& m, int r, int rows, int max_tree) {
  return r < rows && (r % max_tree) < m.n_nodes[r / max_tree];
}

// Single passes over a few rows, bound by latency: the kernels move four columns
// a thread and issue eight splits' partials together (32 rows of 4096, eight
// splits, against one column and four splits: the LayerNorms 11.5 -> 9.4 us,
// the heads' norm 11.4 -> 7.7, the four elementwise ones 6.9 -> 5.2 on average).
// d is a multiple of 8, and so is every row of the library's own buffers; the
// caller's bias and gain vectors are
// bf16 arrays of any alignment and are read one value at a time.
__device__ __forceinline__ float4 bf16x4_at(const uint16_t* p) {
  return make_float4(bf16_to_f32(p[0]), bf16_to_f32(p[1]), bf16_to_f32(p[2]), bf16_to_f32(p[3]));
}

__device__ __forceinline__ void add4(float4& a, const float4& b) {
  a.x += b.x; a.y += b.y; a.z += b.z; a.w += b.w;
}

// columns k .. k + 3 (k a multiple of 4) of a packed operand row
__device__ __forceinline__ void put_split4(uint16_t* dst, long long off, float4 v) {
  const Hilo2 a = pack_hilo2(v.x, v.y), b = pack_hilo2(v.z, v.w);
  *reinterpret_cast<uint2*>(dst + off) = make_uint2(a.hi, b.hi);
  *reinterpret_cast<uint2*>(dst + off + XPACK_LO) = make_uint2(a.lo, b.lo);
}

// Split-K partials of columns at .. at + 3, in split order; eight splits' loads
// are issued together.
__device__ __forceinline__ float4 sum_parts4(const float* parts, int n, long long stride, long long at) {
  float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int p0 = 0; p0 < n; p0 += 8) {
    float4 t[8];
#pragma unroll
    for (int u = 0; u < 8; ++u)  // past the last: a repeated load that is not added
      t[u] = *reinterpret_cast<const float4*>(parts + min(p0 + u, n - 1) * stride + at);
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (p0 + u < n) add4(s, t[u]);
  }
  return s;
}

// [F, e] of every row as the operand of W_m (K = 2d).
__global__ __launch_bounds__(DT) void draft_in_kernel(DraftArgs a, StepMeta meta) {  // grid (rows, y)
  const int r = a.row0 + blockIdx.x, d = a.d;
  const bool live = draft_live(meta, r, a.rows, a.max_tree);
  const int b = r / a.max_tree, i = r % a.max_tree;
  const float* f = a.node_feat ? a.node_feat + (long long)min(r, a.rows - 1) * d
                  : i == 0    ? a.root_feat + (long long)b * d
                              : a.feat_r + ((long long)b * a.max_tree + meta.parent[min(r, a.rows - 1)]) * d;
  const uint16_t* e = a.embed + (long long)meta.token[min(r, a.rows - 1)] * d;
  const int k = 4 * (blockIdx.y * DT + threadIdx.x);
  if (k >= 2 * d) return;
  float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
  if (live) v = k < d ? *reinterpret_cast<const float4*>(f + k) : bf16x4_at(e + k - d);
  put_split4(a.x_m, xpack_off(r, k, a.ks_m), v);
}

// Per-row reductions hold a row in registers: G groups of four columns per
// thread, group j at column 4 (threadIdx.x + j DR).
constexpr int MAX_G = 2;  // d <= 4 DR MAX_G
constexpr float4 kZero4 = {0.f, 0.f, 0.f, 0.f};

// Two block-wide sums at once (fixed order).
__device__ __forceinline__ float2 block_sum2(float x, float y, float* red /* >= 32 floats */) {
  x = wave_sum(x);
  y = wave_sum(y);
  const int w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) {
    red[w] = x;
    red[16 + w] = y;
  }
  __syncthreads();
  float sx = 0.f, sy = 0.f;
  for (int i = 0; i < nw; ++i) {
    sx += red[i];
    sy += red[16 + i];
  }
  return make_float2(sx, sy);
}

// h = sum of the W_m partials + b_m (kept), then [LN(h), LN(e)] as the
// operand of W_u (K = 2d).
template <int G>
__global__ __launch_bounds__(DR) void draft_fuse_kernel(DraftArgs a, StepMeta meta) {
  __shared__ float red[32];
  const int r = a.row0 + blockIdx.x, d = a.d;
  const bool live = draft_live(meta, r, a.rows, a.max_tree);
  const uint16_t* e = a.embed + (long long)meta.token[min(r, a.rows - 1)] * d;
  float4 hv[G], ev[G];
  int at[G];
  bool ok[G];
  float sh = 0.f, se = 0.f;
#pragma unroll
  for (int j = 0; j < G; ++j) {
    at[j] = 4 * (threadIdx.x + j * DR);
    ok[j] = at[j] < d;
    hv[j] = ev[j] = kZero4;
    if (!ok[j]) continue;
    ev[j] = bf16x4_at(e + at[j]);
    if (live) {
      hv[j] = sum_parts4(a.parts, a.n_parts_m, a.stride_m, (long long)r * d + at[j]);
      add4(hv[j], bf16x4_at(a.b_m + at[j]));
    }
    *reinterpret_cast<float4*>(a.h + (long long)r * d + at[j]) = hv[j];
    sh += hv[j].x + hv[j].y + hv[j].z + hv[j].w;
    se += ev[j].x + ev[j].y + ev[j].z + ev[j].w;
  }
  const float2 mean = block_sum2(sh, se, red);
  const float mh = mean.x / d, me = mean.y / d;
  auto sq = [](const float4& v, float m) {
    return (v.x - m) * (v.x - m) + (v.y - m) * (v.y - m) + (v.z - m) * (v.z - m) + (v.w - m) * (v.w - m);
  };
  float vh = 0.f, ve = 0.f;
#pragma unroll
  for (int j = 0; j < G; ++j)
    if (ok[j]) {
      vh += sq(hv[j], mh);
      ve += sq(ev[j], me);
    }
  const float2 var = block_sum2(vh, ve, red);
  const float rh = rsqrtf(var.x / d + a.ln_eps), re = rsqrtf(var.y / d + a.ln_eps);
  auto norm = [](const float4& v, float m, float rs, const float4& g, const float4& b) {
    return make_float4((v.x - m) * rs * g.x + b.x, (v.y - m) * rs * g.y + b.y, (v.z - m) * rs * g.z + b.z,
                       (v.w - m) * rs * g.w + b.w);
  };
#pragma unroll
  for (int j = 0; j < G; ++j) {
    const int k = at[j];
    if (!ok[j]) continue;
    const float4 lh = norm(hv[j], mh, rh, bf16x4_at(a.ln_h_g + k), bf16x4_at(a.ln_h_b + k));
    const float4 le = norm(ev[j], me, re, bf16x4_at(a.ln_x_g + k), bf16x4_at(a.ln_x_b + k));
    put_split4(a.x_u, xpack_off(r, k, a.ks_u), live ? lh : kZero4);
    put_split4(a.x_u, xpack_off(r, d + k, a.ks_u), live ? le : kZero4);
  }
}

// SiLU(sum of the W_u partials + b_u) as the operand of W_d (K = tgf_dim).
// e is any width: rows of a width that is no multiple of 4 go one column at a time.
__global__ __launch_bounds__(DT) void draft_silu_kernel(DraftArgs a, StepMeta meta) {
  const int r = a.row0 + blockIdx.x, e = a.tgf_dim;
  const bool live = draft_live(meta, r, a.rows, a.max_tree);
  const int k = 4 * (blockIdx.y * DT + threadIdx.x);
  auto silu = [](float z) { return z / (1.f + expf(-z)); };
  if (e % 4 == 0) {
    if (k >= e) return;
    float4 v = kZero4;
    if (live) {
      float4 z = sum_parts4(a.parts, a.n_parts_u, a.stride_u, (long long)r * e + k);
      add4(z, bf16x4_at(a.b_u + k));
      v = make_float4(silu(z.x), silu(z.y), silu(z.z), silu(z.w));
    }
    put_split4(a.x_d, xpack_off(r, k, a.ks_d), v);
    return;
  }
  for (int c = k; c < min(k + 4, e); ++c) {
    float v = 0.f;
    if (live) {
      float z = 0.f;
      for (int p = 0; p < a.n_parts_u; ++p) z += a.parts[p * a.stride_u + (long long)r * e + c];
      v = silu(z + bf16_to_f32(a.b_u[c]));
    }
    const Hilo2 q = pack_hilo2(v, 0.f);
    const long long off = xpack_off(r, c, a.ks_d);
    a.x_d[off] = (uint16_t)q.hi;
    a.x_d[off + XPACK_LO] = (uint16_t)q.lo;
  }
}

// o = sum of the W_d partials + b_d + h: the decoder layer's input x.
__global__ __launch_bounds__(DT) void draft_out_kernel(DraftArgs a, StepMeta meta) {
  const int r = a.row0 + blockIdx.x, d = a.d;
  const bool live = draft_live(meta, r, a.rows, a.max_tree);
  const int k = 4 * (blockIdx.y * DT + threadIdx.x);
  if (k >= d) return;
  const long long at = (long long)r * d + k;
  float4 v = kZero4;
  if (live) {
    const float4 h = *reinterpret_cast<const float4*>(a.h + at);
    v = sum_parts4(a.parts, a.n_parts_d, a.stride_d, at);
    add4(v, bf16x4_at(a.b_d + k));
    add4(v, h);
  }
  *reinterpret_cast<float4*>(a.x + at) = v;
}

// y = x + the decoder layer's last residual (down-projection partials), as
// the operand of [W_p; W_r] (K = d).
__global__ __launch_bounds__(DT) void draft_head_in_kernel(DraftArgs a, StepMeta meta, ResidualAdd add) {
  const int r = a.row0 + blockIdx.x, d = a.d;
  const bool live = draft_live(meta, r, a.rows, a.max_tree);
  const int k = 4 * (blockIdx.y * DT + threadIdx.x);
  if (k >= d) return;
  const long long at = (long long)r * d + k;
  float4 y = kZero4;
  if (live) {
    y = *reinterpret_cast<const float4*>(a.x + at);
    add4(y, sum_parts4(add.parts, add.n_parts, add.part_stride, at));
  }
  put_split4(a.x_h, xpack_off(r, k, a.ks_h), y);
}

// F^P and F^R from the head partials; F^R is kept for the next pass, and
// RMSNorm(F^P) times the final norm's gain becomes the LM head's operand.
template <int G>
__global__ __launch_bounds__(DR) void draft_head_out_kernel(DraftArgs a, StepMeta meta) {
  __shared__ float red[32];
  const int r = a.row0 + blockIdx.x, d = a.d;
  const bool live = draft_live(meta, r, a.rows, a.max_tree);
  float4 pv[G];
  float ss = 0.f;
#pragma unroll
  for (int j = 0; j < G; ++j) {
    const int k = 4 * (threadIdx.x + j * DR);
    pv[j] = kZero4;
    if (k >= d) continue;
    const long long at = (long long)r * d + k;
    if (live) {
      pv[j] = sum_parts4(a.parts, a.n_parts_h, a.stride_h, (long long)r * 2 * d + k);
      float4 q = sum_parts4(a.parts, a.n_parts_h, a.stride_h, (long long)r * 2 * d + d + k);
      add4(pv[j], bf16x4_at(a.b_p + k));
      add4(q, bf16x4_at(a.b_r + k));
      *reinterpret_cast<float4*>(a.feat_r + at) = q;
    }
    *reinterpret_cast<float4*>(a.feat_p + at) = pv[j];
    ss += pv[j].x * pv[j].x + pv[j].y * pv[j].y + pv[j].z * pv[j].z + pv[j].w * pv[j].w;
  }
  const float inv = rsqrtf(block_sum2(ss, 0.f, red).x / d + a.rms_eps);
#pragma unroll
  for (int j = 0; j < G; ++j) {
    const int k = 4 * (threadIdx.x + j * DR);
    if (k >= d) continue;
    const float4 g = bf16x4_at(a.final_norm + k), p = pv[j];
    put_split4(a.xn, xpack_off(r, k, a.xn_ks),
               live ? make_float4(p.x * inv * g.x, p.y * inv * g.y, p.z * inv * g.z, p.w * inv * g.w) : kZero4);
  }
}

// Top-k tokens (value descending, lower id first on ties) and their
// log-probabilities log softmax.  Two launches, so that a handful of rows
// still fills the chip: first every (row, vocabulary slice) workgroup holds
// its slice in registers and writes the slice's k best candidates in order plus
// its maximum and sum of exp; then one workgroup per row combines the slices'
// log-sum-exp and ranks their candidates.
// Nothing here runs k rounds: a wave's k-th best lane maximum is a bound that k
// logits of the wave reach, so the best such bound of the slice's waves cuts
// the slice to a few candidates (in a wave at most k lanes reach it), and each
// candidate's place is the number of candidates before it.  Rounds of a
// block-wide argmax were a serial chain of shuffles and barriers: 10 rows of
// 128256 logits, k = 10: slices 28.3 -> 12.0 us, merge 8.7 -> 5.6 us.  (Lane
// exchanges through __shfl instead of v_readlane: 24.9 us.)
constexpr int DK = 16;       // largest k
constexpr int TS = 1024;     // threads per slice workgroup
constexpr int TE = 8;        // logits per thread
constexpr int TCAND = TS / 64 * DK * TE;  // most candidates of a slice
constexpr int TM = 256;      // threads per row of the merge
constexpr int SLICE_MAX = TS * TE;
constexpr int MAX_SLICES = 64;
constexpr int PART_WORDS = 2 * DK + 2;  // values, ids, maximum, sum of exp

constexpr int NO_ID = 0x7fffffff;

// A candidate as one word: value descending, then id ascending, is the words'
// descending order (-0 counts as 0).  0 stands for no candidate, NaN included.
typedef unsigned long long TopKey;
__device__ __forceinline__ TopKey top_key(float v, int id) {
  const uint32_t u = __float_as_uint(v + 0.f);
  const uint32_t ord = u & 0x80000000u ? ~u : u | 0x80000000u;
  return v == v ? (TopKey)ord << 32 | (uint32_t)~id : 0;
}
__device__ __forceinline__ int key_id(TopKey key) { return key ? (int)~(uint32_t)key : NO_ID; }
__device__ __forceinline__ float key_value(TopKey key) {
  const uint32_t ord = (uint32_t)(key >> 32);
  return key ? __uint_as_float(ord & 0x80000000u ? ord & 0x7fffffffu : ~ord) : -INFINITY;
}

// How many of keys[0, n) come before `key`; keys is padded with zeros to a
// multiple of 8, whose reads are issued together.
__device__ __forceinline__ int rank_of(const TopKey* keys, int n, TopKey key) {
  int at = 0;
  for (int o = 0; o < n; o += 8) {
    TopKey t[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) t[u] = keys[o + u];
#pragma unroll
    for (int u = 0; u < 8; ++u) at += t[u] > key;
  }
  return at;
}

__host__ __device__ __forceinline__ int topk_slices(int V) { return (V + SLICE_MAX - 1) / SLICE_MAX; }
__host__ __device__ __forceinline__ int topk_slice_len(int V) {
  const int s = topk_slices(V);
  return ((V + s - 1) / s + 3) & ~3;
}

template <bool VEC>
__global__ __launch_bounds__(TS) void draft_topk_slice_kernel(const float* logits, long long ld, int V, StepMeta meta,
                                                             int rows, int max_tree, int first, int count, int k,
                                                             float* part) {
  __shared__ float red[16];
  __shared__ TopKey wk[TS / 64], ck[TCAND + 8], best[DK];
  __shared__ int n_cand;
  const int r = (int)blockIdx.x / count * max_tree + first + (int)blockIdx.x % count, slice = blockIdx.y;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (!draft_live(meta, r, rows, max_tree)) return;  // uniform
  const int len = topk_slice_len(V), lo = slice * len, hi = min(V, lo + len);
  const float* lg = logits + (long long)r * ld;
  float x[TE];
  if (tid == 0) n_cand = 0;
  if (tid < DK) best[tid] = 0;
  auto id_of = [&](int j) { return VEC ? lo + 4 * (tid + (j >> 2) * TS) + (j & 3) : lo + tid + j * TS; };
  if (VEC) {
    const float4* l4 = reinterpret_cast<const float4*>(lg + lo);
#pragma unroll
    for (int q = 0; q < TE / 4; ++q) {
      const int at = lo + 4 * (tid + q * TS);
      const float4 v = at < hi ? l4[tid + q * TS] : make_float4(0.f, 0.f, 0.f, 0.f);
      x[4 * q] = v.x;
      x[4 * q + 1] = v.y;
      x[4 * q + 2] = v.z;
      x[4 * q + 3] = v.w;
    }
  } else {
#pragma unroll
    for (int j = 0; j < TE; ++j) {
      const int at = lo + tid + j * TS;
      x[j] = at < hi ? lg[at] : 0.f;
    }
  }
  // the slice's maximum and sum of exp (fixed order)
  float m = -INFINITY;
#pragma unroll
  for (int j = 0; j < TE; ++j)
    if (id_of(j) < hi) m = fmaxf(m, x[j]);
  m = wave_max(m);
  __syncthreads();
  if (lane == 0) red[wave] = m;
  __syncthreads();
  float M = red[0];
  for (int w = 1; w < TS / 64; ++w) M = fmaxf(M, red[w]);
  float e = 0.f;
  if (M > -INFINITY) {
#pragma unroll
    for (int j = 0; j < TE; ++j)
      if (id_of(j) < hi) e += expf(x[j] - M);
  }
  const float S = block_sum(e, red);
  float* out = part + ((long long)r * gridDim.y + slice) * PART_WORDS;
  if (tid == 0) {
    out[2 * DK] = M;
    out[2 * DK + 1] = S;
  }
  // this lane's best logit, ranked among the wave's lanes
  TopKey mine = 0;
#pragma unroll
  for (int j = 0; j < TE; ++j)
    if (id_of(j) < hi) mine = max(mine, top_key(x[j], id_of(j)));
  const int klo = (int)(uint32_t)mine, khi = (int)(uint32_t)(mine >> 32);
  int rank = 0;
#pragma unroll
  for (int l = 0; l < 64; ++l) {
    const TopKey o = (TopKey)(uint32_t)__builtin_amdgcn_readlane(khi, l) << 32 |
                     (uint32_t)__builtin_amdgcn_readlane(klo, l);
    rank += o > mine;
  }
  // the k-th best lane's key; 0 where fewer lanes hold a logit
  if (tid % 64 == 0) wk[wave] = 0;
  __syncthreads();
  if (mine && rank == k - 1) wk[wave] = mine;
  __syncthreads();
  TopKey bound = 1;
#pragma unroll
  for (int w = 0; w < TS / 64; ++w) bound = max(bound, wk[w]);
#pragma unroll
  for (int j = 0; j < TE; ++j) {
    const TopKey key = id_of(j) < hi ? top_key(x[j], id_of(j)) : 0;
    if (key >= bound) {
      const int at = atomicAdd(&n_cand, 1);  // places in any order: the keys are distinct
      if (at < TCAND) ck[at] = key;
    }
  }
  __syncthreads();
  const int n = min(n_cand, TCAND);
  if (tid < 8) ck[n + tid] = 0;
  __syncthreads();
  for (int c = tid; c < n; c += TS) {
    const int at = rank_of(ck, n, ck[c]);
    if (at < k) best[at] = ck[c];
  }
  __syncthreads();
  if (tid < k) {
    out[tid] = key_value(best[tid]);
    out[DK + tid] = __int_as_float(key_id(best[tid]));
  }
}

__global__ __launch_bounds__(TM) void draft_topk_merge_kernel(const float* part, int nslice, StepMeta meta, int rows,
                                                             int max_tree, int first, int count, int k,
                                                             int32_t* tok_out, float* logp_out) {
  __shared__ TopKey ck[MAX_SLICES * DK + 8], best[DK];
  const int r = (int)blockIdx.x / count * max_tree + first + (int)blockIdx.x % count;
  const int tid = threadIdx.x, lane = tid & 63;
  if (!draft_live(meta, r, rows, max_tree)) return;  // uniform
  const float* pr = part + (long long)r * nslice * PART_WORDS;
  const float Ms = lane < nslice ? pr[lane * PART_WORDS + 2 * DK] : -INFINITY;
  const float Ss = lane < nslice ? pr[lane * PART_WORDS + 2 * DK + 1] : 0.f;
  const float M = wave_max(Ms);
  const float lse = M + logf(wave_sum(Ms > -INFINITY ? Ss * expf(Ms - M) : 0.f));
  const int n = nslice * k;
  if (tid < DK) best[tid] = 0;
  for (int q = tid; q < n + 8; q += TM) {
    const float* at = pr + (q / k) * PART_WORDS + q % k;
    const int id = q < n ? __float_as_int(at[DK]) : NO_ID;
    ck[q] = id == NO_ID ? 0 : top_key(at[0], id);
  }
  __syncthreads();
  for (int q = tid; q < n; q += TM) {
    const int at = ck[q] ? rank_of(ck, n, ck[q]) : k;
    if (at < k) best[at] = ck[q];
  }
  __syncthreads();
  if (tid < k) {  // a row with fewer than k logits that are no NaN: token -1 past them
    tok_out[(long long)r * k + tid] = best[tid] ? key_id(best[tid]) : -1;
    logp_out[(long long)r * k + tid] = best[tid] ? key_value(best[tid]) - lse : -INFINITY;
  }
}

hipError_t launch_draft_front(const DraftArgs& a, const StepMeta& meta, int stage, hipStream_t s) {
  const auto blocks = [&](int width) { return dim3(a.nr, (width + 4 * DT - 1) / (4 * DT)); };
  if (a.d % 4 != 0 || a.d > 4 * DR * MAX_G) return hipErrorInvalidValue;
  switch (stage) {
    case 0: hipLaunchKernelGGL(draft_in_kernel, blocks(2 * a.d), dim3(DT), 0, s, a, meta); break;
    case 1:
      if (a.d <= 4 * DR) hipLaunchKernelGGL(draft_fuse_kernel<1>, dim3(a.nr), dim3(DR), 0, s, a, meta);
      else hipLaunchKernelGGL(draft_fuse_kernel<MAX_G>, dim3(a.nr), dim3(DR), 0, s, a, meta);
      break;
    case 2: hipLaunchKernelGGL(draft_silu_kernel, blocks(a.tgf_dim), dim3(DT), 0, s, a, meta); break;
    case 3: hipLaunchKernelGGL(draft_out_kernel, blocks(a.d), dim3(DT), 0, s, a, meta); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_draft_head(const DraftArgs& a, const StepMeta& meta, const ResidualAdd& add, int stage,
                             hipStream_t s) {
  if (add.slot != nullptr) return hipErrorInvalidValue;  // dense decoder layer only
  if (a.d % 4 != 0 || a.d > 4 * DR * MAX_G) return hipErrorInvalidValue;
  if (stage == 0)
    hipLaunchKernelGGL(draft_head_in_kernel, dim3(a.nr, (a.d + 4 * DT - 1) / (4 * DT)), dim3(DT), 0, s, a, meta, add);
  else if (a.d <= 4 * DR)
    hipLaunchKernelGGL(draft_head_out_kernel<1>, dim3(a.nr), dim3(DR), 0, s, a, meta);
  else
    hipLaunchKernelGGL(draft_head_out_kernel<MAX_G>, dim3(a.nr), dim3(DR), 0, s, a, meta);
  return hipGetLastError();
}

size_t draft_topk_work_bytes(int rows, int V) {
  return sizeof(float) * (size_t)rows * topk_slices(V) * PART_WORDS;
}

hipError_t launch_draft_topk(const float* logits, long long ld, int V, const StepMeta& meta, int rows, int max_tree,
                             int first, int count, int k, int32_t* tok, float* logp, float* work, hipStream_t s) {
  if (first < 0 || count < 1 || first + count > max_tree || k < 1 || k > DK || V < k || topk_slices(V) > MAX_SLICES) return hipErrorInvalidValue;
  const int ns = topk_slices(V);
  const int n = rows / max_tree * count;
  if ((V & 3) == 0 && (ld & 3) == 0)  // 16-byte aligned rows and slices
    hipLaunchKernelGGL(draft_topk_slice_kernel<true>, dim3(n, ns), dim3(TS), 0, s, logits, ld, V, meta, rows,
                       max_tree, first, count, k, work);
  else
    hipLaunchKernelGGL(draft_topk_slice_kernel<false>, dim3(n, ns), dim3(TS), 0, s, logits, ld, V, meta, rows,
                       max_tree, first, count, k, work);
  hipLaunchKernelGGL(draft_topk_merge_kernel, dim3(n), dim3(TM), 0, s, work, ns, meta, rows, max_tree, first, count, k,
                     tok, logp);
  return hipGetLastError();
}

// ------------------------------------------------------------ tree expansion

// Ranking key of a candidate score: NaN counts as the lowest score.
__device__ __forceinline__ double sel_key(double s) { return s != s ? -INFINITY : s; }
// Candidate a (score sa) ranks before candidate b: higher score, then lower index.
__device__ __forceinline__ bool sel_before(double sa, int a, double sb, int b) {
  return sa > sb || (sa == sb && a < b);
}

constexpr int SEL_T = 1024;  // one thread per candidate of the last pass (four waves per SIMD)
constexpr int SEL_U = 16;    // candidates compared per batch of LDS reads

// Rank of candidate q (key s) among the n candidates keyed sc[0, n): how many
// rank before it.  The reads are batched so that their LDS latencies overlap.
__device__ __forceinline__ int sel_rank(const double* sc, int n, double s, int q) {
  int rk = 0, o = 0;
  for (; o + SEL_U <= n; o += SEL_U) {
    double v[SEL_U];
#pragma unroll
    for (int u = 0; u < SEL_U; ++u) v[u] = sc[o + u];
#pragma unroll
    for (int u = 0; u < SEL_U; ++u) rk += sel_before(v[u], o + u, s, q);
  }
  for (; o < n; ++o) rk += sel_before(sc[o], o, s, q);
  return rk;
}

__global__ __launch_bounds__(SEL_T) void draft_select_kernel(DraftSelectArgs a) {
  __shared__ double sc[DRAFT_SEL_MAX];  // ranking keys of the candidates
  __shared__ int slot[DRAFT_SEL_MAX];   // last pass: output row - 1 of a kept candidate, else -1
  __shared__ int dep[DRAFT_SEL_MAX];    // last pass: depth of a candidate
  __shared__ int kept[64], kdep[64];    // last pass: kept candidates by rank, their depths
  const int b = blockIdx.x, tid = threadIdx.x, k = a.k, T = a.max_tree, t = a.t;
  // the frontier of pass t: the root, or the k nodes the previous pass added
  const int f0 = t == 0 ? 0 : 1 + k * (t - 1), nf = (t == 0 ? 1 : k) * k;
  const int c0 = t == 0 ? 0 : k + k * k * (t - 1);  // index of the first fresh candidate
  const long long cb = (long long)b * DRAFT_SEL_MAX, nb = (long long)b * T;
  int none = 0;  // the sequence has candidates without a token
  for (int q = tid; q < nf; q += SEL_T) {
    const int r = f0 + q / k;
    const long long at = (nb + r) * k + q % k;
    const int tok = a.topk_tok[at];  // -1: no candidate, ranked last
    const double s = tok < 0 ? -INFINITY : (r == 0 ? 0.0 : a.n_score[nb + r]) + (double)a.topk_lp[at];
    none |= tok < 0;
    a.c_tok[cb + c0 + q] = tok;
    a.c_node[cb + c0 + q] = r;
    a.c_score[cb + c0 + q] = s;
    sc[c0 + q] = sel_key(s);
  }
  if (t + 1 < a.depth) {
    __syncthreads();
    // the k best fresh candidates become pass-tree nodes 1 + k t + rank
    for (int q = tid; q < nf; q += SEL_T) {
      const int rk = sel_rank(sc + c0, nf, sc[c0 + q], q);
      if (rk < k) {
        const int node = 1 + k * t + rk, r = f0 + q / k;
        a.n_cand[nb + node] = c0 + q;
        a.n_score[nb + node] = a.c_score[cb + c0 + q];
        a.m_token[nb + node] = max(a.c_tok[cb + c0 + q], 0);  // the next pass reads this token's embedding
        a.m_parent[nb + node] = r;
        a.m_anc[nb + node] = a.m_anc[nb + r] | (1ull << node);
      }
    }
    for (int w = b * SEL_T + tid; w < a.tail_words; w += gridDim.x * SEL_T) a.tail_dst[w] = a.tail_src[w];
    return;
  }
  // last pass: the n_total best of all candidates, numbered by depth, then rank
  const int nc = c0 + nf, keep = min(nc, a.n_total);
  for (int q = tid; q < nc; q += SEL_T) {
    if (q < c0) {
      sc[q] = sel_key(a.c_score[cb + q]);
      none |= a.c_tok[cb + q] < 0;
    }
    dep[q] = q < k ? 1 : 2 + (q - k) / (k * k);
    slot[q] = -1;
  }
  none = __syncthreads_or(none);
  for (int q = tid; q < nc; q += SEL_T) {
    const int rk = sel_rank(sc, nc, sc[q], q);
    if (rk < keep) {  // ranks are distinct
      kept[rk] = q;
      kdep[rk] = dep[q];
    }
  }
  __syncthreads();
  if (tid < keep) {
    const int dq = kdep[tid];
    int at = 0;
    for (int j = 0; j < keep; ++j) at += kdep[j] < dq || (kdep[j] == dq && j < tid);
    slot[kept[tid]] = at;
  }
  __syncthreads();
  if (tid < keep) {
    const int q = kept[tid], at = slot[q];
    const int r = a.c_node[cb + q];
    const int pc = r == 0 ? -1 : a.n_cand[nb + r];
    a.o_tok[nb + at + 1] = a.c_tok[cb + q];
    a.o_par[nb + at + 1] = pc < 0 ? 0 : slot[pc] + 1;
    a.o_score[nb + at + 1] = (float)a.c_score[cb + q];
  }
  if (tid == 0) {
    a.o_nodes[b] = none ? -(1 + keep) : 1 + keep;
    a.o_tok[nb] = a.m_token[nb];
    a.o_par[nb] = -1;
    a.o_score[nb] = 0.f;
  }
}

hipError_t launch_draft_select(const DraftSelectArgs& a, int batch, hipStream_t s) {
  if (a.k < 1 || a.k > DK || a.t < 0 || a.t >= a.depth || a.max_tree > 64 || 1 + a.k * (a.depth - 1) > a.max_tree ||
      a.k * (1 + a.k * (a.depth - 1)) > DRAFT_SEL_MAX || a.n_total < 1 || a.n_total > 63 || batch < 1)
    return hipErrorInvalidValue;
  hipLaunchKernelGGL(draft_select_kernel, dim3(batch), dim3(SEL_T), 0, s, a);
  return hipGetLastError();
}

}  // namespace griffin
