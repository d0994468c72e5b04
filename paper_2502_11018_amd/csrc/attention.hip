// Tree-masked attention of the verify pass.
//
// A tree node r of sequence b sees the cached prefix slots [0, P_b) and the
// tree slots P_b + j for every node j on its root path (bit j of anc[r]).
// The prefix part is the bulk of the work and is computed here; the few tree
// keys of each node (its ancestors) are added by attn_combine in fp32, from
// fp32 copies of the tree K/V, while it merges the prefix splits.
//
// tree_attention_kernel: a workgroup handles one (sequence, KV head, prefix
// split) for NW of the KV head's row tiles.  A row tile is 32 tree rows of one
// query head, or, where a sequence's rows of the whole head group fit one tile
// (max_tree * group <= 32: short chains), all of them (PACK).  The NW waves,
// one row tile each, share every 32-key block of K and V, which the workgroup
// stages once into an LDS ring with global_load_lds_dwordx4 (each wave issues
// an equal share of the block's 1 KB pieces), so the cache is read once per
// workgroup rather than once per head.
//
// Per 32-key block each wave computes S^T = K Q^T and O^T += V^T P^T with
// v_mfma_f32_32x32x16_bf16, so that each lane owns one query row (column of
// the MFMA output) and the softmax bookkeeping is lane-local:
//  * Keys are fed to the MFMA in a permuted row order so that accumulator
//    register q of lane half h holds key 16 h + q of the block; the P operand
//    of the second product is then the lane's own registers 8 t .. 8 t + 7.
//  * V is cached in 32-slot tiles stored transposed ([tile][dim][32]), so a
//    block's V^T is one contiguous 8 KB tile.
//  * The ring holds each block in MFMA fragment order (piece, lane, 8 values):
//    the DMA gathers every lane's 16 bytes from the cache, and the compute
//    side reads each operand with one conflict-free ds_read_b128.
//  * Q and K use the same head-dim permutation as the projection GEMMs: a lane
//    reads 32 consecutive head dims and feeds 8 of them to each of 4 MFMAs.
//  * Q and P enter the matrix cores as split bf16 (hi + lo, two MFMAs each),
//    so only the cached K/V carry bf16 rounding.
// Scores are kept in the log2 domain (scaled by log2(e)/sqrt(dh)) and exp2 is
// used throughout; masked keys contribute exactly zero.

#include "device_common.h"
#include "griffin_internal.h"

namespace griffin {

template <int DH, int NW, bool RAGGED, bool PACK>
__global__ __launch_bounds__(64 * NW, 1) void tree_attention_kernel(AttnArgs a) {
  constexpr int CH = DH / 64;          // 64-dim chunks of Q/K per lane pair
  constexpr int DB = DH / 32;          // 32-dim blocks of the output
  constexpr int KP = CH * 4;           // 1 KB pieces of a K block
  constexpr int PIECES = KP + DB * 2;  // K and V pieces of one 32-key block
  constexpr int PPW = PIECES / NW;     // pieces each wave stages per block
  constexpr int D = ATTN_RING;         // ring slots
  static_assert(PIECES % NW == 0 && PPW * (D - 1) < 64 && (!PACK || NW == 1), "ring shape");
  __shared__ u32x4 ring[D][PIECES][64];

  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int col = lane & 31, hh = lane >> 5;
  // Work units: the step's key-split table holds, per unit j, a sequence b,
  // one of its key splits and that sequence's split count (sequences get
  // splits in proportion to their prefix lengths).  XCD-aware decode:
  // workgroups are dispatched round-robin over the 8 XCDs (id % 8), so every
  // workgroup of one (unit, KV head) gets the same id % 8 and the K/V blocks
  // it re-reads are shared through that XCD's L2.
  const int G = a.Hq / a.Hkv;
  const int tiles = PACK ? 1 : G * a.qblocks;  // row tiles of a KV head: tile qb * G + head
  const int per_unit = (tiles + NW - 1) / NW;
  const int id = blockIdx.x;
  const int rest = id >> 3;
  const int u_raw = (rest / per_unit) * 8 + (id & 7);
  // a workgroup past the last unit (the grid is rounded up) runs the
  // prologue's loads for unit 0 and leaves with the workgroups without live
  // rows: no branch before the loads, so the kernel arguments are fetched at
  // once
  const bool unit_live = u_raw < a.units * a.Hkv;  // uniform over the workgroup
  const int u = unit_live ? u_raw : 0;
  const int tile0 = rest % per_unit * NW;  // first row tile of the workgroup
  const int hk = u % a.Hkv;
  // RAGGED: the unit comes from the step's split table; else every sequence
  // has a.sp splits and unit j is split j % sp of sequence j / sp
  int4 ent;
  if constexpr (RAGGED) {
    ent = a.meta.split_tab[u / a.Hkv];
    if (ent.x < 0) return;  // a unit without work this step
  } else {
    ent = make_int4((u / a.Hkv / a.sp) | ((u / a.Hkv % a.sp) << 16), a.sp, 0, 0);
  }
  const int b = ent.x & 0xffff, split = ent.x >> 16, nsplit = ent.y;
  const bool tile_live = tile0 + w < tiles;  // wave-uniform
  const int tile_w = tile_live ? tile0 + w : tile0;
  const int qb = PACK ? 0 : tile_w / G;
  const int qrows = a.qblocks * 32;
  // row `col` of the tile: head gh of the group, node qi (PACK: the group's
  // heads one after the other, max_tree rows each)
  auto row_head = [&](int r) { return PACK ? r / a.max_tree : tile_w % G; };
  auto row_node = [&](int r) { return PACK ? r % a.max_tree : qb * 32 + r; };

  // Q^T operand (B): lane (col = query row, hh = k-group), 32 dims per chunk;
  // split bf16, so S = K (q_hi + q_lo).  Loaded before the per-sequence
  // metadata is known (rows past the tree hold stale values and are never
  // written out; the row index stays inside the sequence's max_tree rows).
  const int qr = b * a.max_tree + min(row_node(col), a.max_tree - 1);
  const int hq = hk * G + min(row_head(col), G - 1);
  u32x4 qf[2][CH][4];
  {
    const long long qo = ((long long)qr * a.Hq + hq) * DH + 32 * hh;
#pragma unroll
    for (int c = 0; c < CH; ++c)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        qf[0][c][j] = ld_u4(a.q + qo + 64 * c + 8 * j);
        qf[1][c][j] = ld_u4(a.q_lo + qo + 64 * c + 8 * j);
      }
  }

  const int P = RAGGED ? ent.z : a.meta.prefix_len[b];
  const int n_nodes = RAGGED ? ent.w : a.meta.n_nodes[b];

  // prefix key range of this split, in whole 32-key blocks
  const int nblk = (P + 31) >> 5;
  const int kb0 = (int)((long long)nblk * split / nsplit);
  const int kb1 = (int)((long long)nblk * (split + 1) / nsplit);
  const int nb = kb1 - kb0;

  const long long head = ((long long)b * a.Hkv + hk) * a.kv_cap * DH;
  const uint16_t* kbase = a.k_cache + head;
  const uint16_t* vbase = a.v_cache + head;
  // MFMA row -> key offset inside a 32-key block: row 8q + 4h + e holds key 16h + 4q + e
  const int krow = 16 * ((col >> 2) & 1) + 4 * (col >> 3) + (col & 3);
  // this lane's byte offset inside a block, for each piece this wave stages
  // (each DMA takes a wave-uniform block base plus this offset)
  const int wu = __builtin_amdgcn_readfirstlane(w);
  uint32_t goff[PPW];
#pragma unroll
  for (int p = 0; p < PPW; ++p) {
    const int pc = wu * PPW + p;
    if (pc < KP) {
      const int c = pc >> 2, j = pc & 3;
      goff[p] = 2u * (krow * DH + 64 * c + 32 * hh + 8 * j);
    } else {
      const int v = pc - KP, d = v >> 1, t = v & 1;
      goff[p] = 2u * ((32 * d + col) * 32 + 16 * hh + 8 * t);
    }
  }
  auto issue_piece = [&](int slot, int kb, int p) {
    const int pc = wu * PPW + p;
    const char* blk = reinterpret_cast<const char*>((pc < KP ? kbase : vbase) + (long long)kb * 32 * DH);
    __builtin_amdgcn_global_load_lds((const void*)(blk + goff[p]), (lds_void*)&ring[slot][pc][0], 16, 0, 0);
  };
  auto issue = [&](int slot, int kb) {
#pragma unroll
    for (int p = 0; p < PPW; ++p) issue_piece(slot, kb, p);
  };
  // The first D blocks go out as soon as the prefix length is known (the
  // longest latency of the prologue), before the check for live rows: a
  // workgroup without live rows lets them land and leaves.
  if (nb > 0) {
#pragma unroll
    for (int i = 0; i < D; ++i) issue(i, kb0 + min(i, nb - 1));
  }
  if (!unit_live || (!PACK && tile0 / G * 32 >= n_nodes)) {  // no unit, or no live query rows (uniform)
    wait_vmcnt_lds<0>();
    return;
  }

  // Softmax reference: each lane's row uses a fixed reference m_ref (log2
  // domain), the maximum of its scores in the split's first block, so the
  // output accumulators are never rescaled inside the block loop (a rescale
  // there would make the compiler shuttle them between register files every
  // block), and later blocks compute no maximum at all.  Later scores may
  // exceed m_ref: a row whose sum of p = 2^(s - m_ref) passes 2^64 (which
  // every row with a key more than 64 above its reference does) is flagged,
  // and the merge recomputes that split exactly.  So p needs no clamp: only
  // flagged rows can overflow, and a NaN score stays NaN (a clamp cost 0.8 us
  // per launch, the running maximum 10 us at 16384 keys per sequence).
  // l_run adds up the blocks, each block's 16 keys of the lane first as a tree
  // (sum_key): one chain over all keys of a split loses what is below half a unit
  // of its growing sum key by key (2.9 times the rms error at 1876 keys a split).
  // The two halves of a row meet once, after the loop.
  float m_ref = -INFINITY, l_run = 0.f;
  f32x16 oacc[DB];
#pragma unroll
  for (int d = 0; d < DB; ++d)
#pragma unroll
    for (int r = 0; r < 16; ++r) oacc[d][r] = 0.f;

  u32x4 kf[KP], vf[2][DB];
  auto read_k = [&](int slot) {
#pragma unroll
    for (int x = 0; x < KP; ++x) kf[x] = ring[slot][x][lane];
  };
  // S^T = K Q^T (rows: keys, cols: queries) in two chains, one per part of
  // q = q_hi + q_lo: a single chain of dependent MFMAs issues one every 52
  // clocks instead of 32
  struct Scores {
    f32x16 hi, lo;
  };
  auto qk = [&](Scores& s) {
#pragma unroll
    for (int r = 0; r < 16; ++r) s.hi[r] = s.lo[r] = 0.f;
#pragma unroll
    for (int x = 0; x < KP; ++x) {
      s.hi = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(kf[x]), as_bf16x8(qf[0][x / 4][x % 4]), s.hi, 0, 0, 0);
      s.lo = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(kf[x]), as_bf16x8(qf[1][x / 4][x % 4]), s.lo, 0, 0, 0);
    }
  };
  // P as split bf16 (p_hi + p_lo), the operand of O^T += V^T P^T, of keys 8 t ..
  // 8 t + 7 of the lane's 16, a part at a time: part u of n = 4 or 8 is a pair
  // of keys or one plane of a pair
  float p[16];
  auto pack_part = [&](u32x4 (&pf)[2], int t, int u, int n) {
    const int q = u * 4 / n;
    const float x = p[8 * t + 2 * q], y = p[8 * t + 2 * q + 1];
    if (n == 4 || u % 2 == 0) pf[0][q] = pack_bf16x2(x, y);
    if (n == 4 || u % 2 == 1)
      pf[1][q] = pack_bf16x2(x - __uint_as_float(pf[0][q] << 16), y - __uint_as_float(pf[0][q] & 0xffff0000u));
  };
  float part[4];  // sums of 1, 2, 4, 8 keys that wait for their neighbours
  auto sum_key = [&](int r) {
    float v = p[r];
    int level = 0;
#pragma unroll
    for (; r >> level & 1; ++level) v = part[level] + v;
    if (level == 4) l_run += v;
    else part[level] = v;
  };
  // One wave per SIMD: an MFMA leaves 28 of its 32 clocks to the wave's other
  // instructions (measured: up to 6 vector instructions, or 4 and an exp2,
  // between two MFMAs cost nothing, each further one 4 to 8 clocks), so step i
  // is written as a sequence of MFMAs with their share of everything else:
  // the score MFMAs of block i + 1 between the softmax of block i and its V
  // reads, then, past the barrier, the P V MFMAs of block i between the second
  // half of its packing, the K reads of block i + 2 and the DMA of block i + D.
  // sched_barrier holds that order; left alone the compiler moves each LDS read
  // next to its use and waits for it there.  The barrier (every wave's pieces of
  // block i + 2 have landed, and every wave holds its V of block i) publishes
  // slot i + 2 and frees slot i.  The split's last block, the only one that can be
  // partial, is handled after the loop.  Issues past the last block re-read it
  // into slots that are never consumed; every DMA has landed before the waves
  // leave.
  //
  // What bounds it: at 8 x 16384 keys the matrix cores' power.  The step takes
  // 1.48 kclk of 1.06 k (the MFMAs alone) but the shader clock falls to 1.6 GHz;
  // 64 rows a wave, which halves the LDS reads and the DMA per MFMA, measured 3 %
  // less.  Per launch, against two workgroups per CU with the reads beside their
  // uses, on one box: 253 -> 244 us there, 69 -> 64 us at 1 x 30011 keys.
  static_assert(D >= 3, "two blocks run ahead of the ring");
  if (nb > 0) {
    Scores sa, sb;
    wait_vmcnt_lds<(D - 1) * PPW>();
    __builtin_amdgcn_s_barrier();
    read_k(0);
    qk(sa);
    {
      float mx = -INFINITY;
#pragma unroll
      for (int r = 0; r < 16; ++r) mx = fmaxf(mx, kb0 * 32 + 16 * hh + r < P ? sa.hi[r] + sa.lo[r] : -INFINITY);
      m_ref = fmaxf(mx, __shfl_xor(mx, 32, 64)) * a.scale_log2;
    }
    wait_vmcnt_lds<(D - 2) * PPW>();
    __builtin_amdgcn_s_barrier();
    read_k(1);  // a single-block split reads a repeat of block 0 and leaves it
    int slot = 0;  // i % D
    auto step = [&](const Scores& s, Scores& sn, int i) {
      u32x4 pf[2][2];
      constexpr int S1 = 2 * KP, E = 16 / S1;  // score MFMAs; keys of the softmax per MFMA
#pragma unroll
      for (int r = 0; r < 16; ++r) sn.hi[r] = sn.lo[r] = 0.f;
#pragma unroll
      for (int g = 0; g < S1; ++g) {
        const int x = g >> 1;
        f32x16& c = g & 1 ? sn.lo : sn.hi;
        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(kf[x]), as_bf16x8(qf[g & 1][x / 4][x % 4]), c, 0, 0, 0);
        if (g < 2 * DB) vf[g / DB][g % DB] = ring[slot][KP + (g % DB) * 2 + g / DB][lane];
#pragma unroll
        for (int e = 0; e < E; ++e) {
          const int r = g * E + e;
          p[r] = __builtin_amdgcn_exp2f(fmaf(s.hi[r] + s.lo[r], a.scale_log2, -m_ref));
          sum_key(r);
        }
        if (g >= S1 / 2) pack_part(pf[0], 0, g - S1 / 2, S1 / 2);
        __builtin_amdgcn_sched_barrier(0);
      }
      wait_vmcnt_lds<(D - 3) * PPW>();
      __builtin_amdgcn_s_barrier();
      const int s1 = slot + 1 == D ? 0 : slot + 1, s2 = s1 + 1 == D ? 0 : s1 + 1;
      const int kb = kb0 + min(i + D, nb - 1);
      constexpr int S2 = 4 * DB, HALF = 2 * DB;  // P V MFMAs
      constexpr int PER = (PPW + S2 - KP - 1) / (S2 - KP);  // DMA pieces per MFMA behind the K reads
#pragma unroll
      for (int g = 0; g < S2; ++g) {
        const int t = g / HALF, h = g / DB % 2, d = g % DB;
        oacc[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(vf[t][d]), as_bf16x8(pf[t][h]), oacc[d], 0, 0, 0);
        if (g < KP) kf[g] = ring[s2][g][lane];
        if (g < HALF) pack_part(pf[1], 1, g, HALF);
        if (g >= KP) {
#pragma unroll
          for (int u = 0; u < PER; ++u)
            if ((g - KP) * PER + u < PPW) issue_piece(slot, kb, (g - KP) * PER + u);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      slot = s1;
    };
    int i = 0;
    for (; i + 2 < nb; i += 2) {
      step(sa, sb, i);
      step(sb, sa, i + 1);
    }
    if (i + 1 < nb) {  // uniform
      step(sa, sb, i);
      sa = sb;
      ++i;
    }
    // last block (i = nb - 1), full or partial: keys at or past P get
    // probability 0, and their V (tree or stale values) is zeroed
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float x = (kb0 + i) * 32 + 16 * hh + r < P ? sa.hi[r] + sa.lo[r] : -INFINITY;
      p[r] = __builtin_amdgcn_exp2f(fmaf(x, a.scale_log2, -m_ref));
      sum_key(r);
    }
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      u32x4 pf[2];
#pragma unroll
      for (int u = 0; u < 4; ++u) pack_part(pf, t, u, 4);
#pragma unroll
      for (int d = 0; d < DB; ++d) {
        u32x4 v = ring[slot][KP + d * 2 + t][lane];
#pragma unroll
        for (int q = 0; q < 4; ++q) {  // bf16 element 2q is the low half of dword q
          const int key = (kb0 + i) * 32 + 16 * hh + 8 * t + 2 * q;
          v[q] &= (key < P ? 0x0000ffffu : 0u) | (key + 1 < P ? 0xffff0000u : 0u);
        }
#pragma unroll
        for (int h = 0; h < 2; ++h)
          oacc[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(v), as_bf16x8(pf[h]), oacc[d], 0, 0, 0);
      }
    }
    wait_vmcnt_lds<0>();
    l_run += __shfl_xor(l_run, 32, 64);
  }
  // a row whose probabilities went past the cap marks its partial invalid
  // (l < 0); the merge recomputes that split exactly
  if (l_run > 0x1p64f) l_run = -1.f;

  // ---- partials, row-major [32 rows][DH].  The accumulators hold O^T (lane:
  // query col, dims 32 d + 8 (r/4) + 4 hh + r%4), so each wave transposes its
  // tile through its own part of the ring, which every wave has left after
  // this barrier: 16-byte chunk c of row `col` sits at chunk c ^ (col & 7)
  // (conflict-free writes and reads), and the global stores are contiguous.
  constexpr int CHUNKS = DH / 4;  // 16-byte chunks per row
  constexpr int RPI = 64 / CHUNKS;  // rows per wave-wide store
  static_assert(NW * 32 * DH * 4 <= (int)sizeof(ring), "transpose tiles fit in the ring");
  __builtin_amdgcn_s_barrier();
  if (!tile_live) return;
  float* tile = reinterpret_cast<float*>(&ring[0][0][0]) + w * 32 * DH;
#pragma unroll
  for (int d = 0; d < DB; ++d)
#pragma unroll
    for (int rg = 0; rg < 4; ++rg) {
      const int c = 8 * d + 2 * rg + hh;
      *reinterpret_cast<float4*>(tile + col * DH + 4 * (c ^ (col & 7))) =
          make_float4(oacc[d][4 * rg], oacc[d][4 * rg + 1], oacc[d][4 * rg + 2], oacc[d][4 * rg + 3]);
    }
  // rows of absent nodes are not stored (the merge reads live rows only)
  const long long head0 = (long long)b * a.Hq + hk * G;
  auto part_row = [&](int r, int s) { return ((head0 + row_head(r)) * a.sp + s) * qrows + row_node(r); };
  auto row_live = [&](int r) { return row_node(r) < n_nodes && row_head(r) < G; };
#pragma unroll
  for (int n = 0; n < 32 / RPI; ++n) {
    const int r = n * RPI + lane / CHUNKS, c = lane % CHUNKS;
    if (row_live(r))
      *reinterpret_cast<float4*>(a.part_o + part_row(r, split) * DH + 4 * c) =
          *reinterpret_cast<const float4*>(tile + r * DH + 4 * (c ^ (r & 7)));
  }
  if (hh == 0 && row_live(col)) {
    float* pml = a.part_ml + part_row(col, split) * 2;
    pml[0] = m_ref;
    pml[1] = l_run;
    // the sequence's last split marks its unused slots empty, so that the
    // merge reads all sp slots without knowing the split count
    if (RAGGED && split == nsplit - 1)
      for (int s2 = nsplit; s2 < a.sp; ++s2) {
        float* pe = a.part_ml + part_row(col, s2) * 2;
        pe[0] = -INFINITY;
        pe[1] = 0.f;
      }
  }
}

AttnShape attn_shape(int group, int max_tree) {
  AttnShape s;
  s.qblocks = (max_tree + 31) / 32;
  // a group's rows packed into one tile: the vector work and the MFMAs of a
  // short chain are those of one row tile instead of one per head
  s.pack = group * max_tree <= 32;
  s.tiles = s.pack ? 1 : group * s.qblocks;
  s.nw = s.tiles >= 4 ? 4 : s.tiles >= 2 ? 2 : 1;
  s.per_unit = (s.tiles + s.nw - 1) / s.nw;
  return s;
}

template <int DH, int NW, bool PACK>
static void launch_attn_nw(const AttnArgs& a, dim3 grid, hipStream_t s) {
  if (a.meta.split_tab) hipLaunchKernelGGL((tree_attention_kernel<DH, NW, true, PACK>), grid, dim3(64 * NW), 0, s, a);
  else hipLaunchKernelGGL((tree_attention_kernel<DH, NW, false, PACK>), grid, dim3(64 * NW), 0, s, a);
}

template <int DH>
static void launch_attn_dh(const AttnArgs& a, const AttnShape& sh, dim3 grid, hipStream_t s) {
  if (sh.pack) launch_attn_nw<DH, 1, true>(a, grid, s);
  else if (sh.nw == 4) launch_attn_nw<DH, 4, false>(a, grid, s);
  else if (sh.nw == 2) launch_attn_nw<DH, 2, false>(a, grid, s);
  else launch_attn_nw<DH, 1, false>(a, grid, s);
}

hipError_t launch_attention(const AttnArgs& a, int batch, hipStream_t s) {
  if (a.batch != batch) return hipErrorInvalidValue;
  const AttnShape sh = attn_shape(a.Hq / a.Hkv, a.max_tree);
  if (a.units < 1 || a.sp < 1 || a.sp > 16 || a.qblocks != sh.qblocks) return hipErrorInvalidValue;
  const int streams = a.units * a.Hkv;
  dim3 grid(((streams + 7) / 8) * 8 * sh.per_unit);
  if (a.dh == 128) launch_attn_dh<128>(a, sh, grid, s);
  else if (a.dh == 64) launch_attn_dh<64>(a, sh, grid, s);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

// Finish attention for every (row, head): merge the prefix splits and add the
// node's tree keys.  Prefix split s contributes (m_s, l_s, o_s) in the log2
// domain; the tree keys are the node's ancestors and itself (bits of anc),
// scored in fp32 from q = q_hi + q_lo and the fp32 tree K/V, with a running
// (m_t, l_t, o_t).  Then o = (sum_s 2^(m_s - M) o_s + 2^(m_t - M) o_t) /
// (sum_s 2^(m_s - M) l_s + 2^(m_t - M) l_t).  Absent rows get zeros.  One
// workgroup per row, one thread per (head, 4 dims); the dot products of a
// tree key reduce over the head's dh/4 threads with xor shuffles (a fixed
// order).  It reads the first MAXS of the sp partial slots of each (sequence,
// head): the step's largest split count rounded up, so that a batch whose
// sequences all hold the even share does not read the slots kept for
// uneven ones.  The merged rows are written fragment-packed split bf16 (o_ks K
// steps per tile) as the activation operand of the output projection.
template <int MAXS, bool RAGGED>
__global__ __launch_bounds__(256) void attn_combine_kernel(const float* __restrict__ part_o,
                                                           const float* __restrict__ part_ml, StepMeta meta,
                                                           int Hq, int Hkv, int dh, int sp, int qrows, int max_tree,
                                                           const uint16_t* __restrict__ q,
                                                           const uint16_t* __restrict__ q_lo, TreeKV32 tree,
                                                           PrefixKV prefix, float scale_log2,
                                                           uint16_t* __restrict__ o_out, int o_ks, int row0) {
  const int r = row0 + blockIdx.x;
  const int b = r / max_tree, i = r % max_tree;
  const int quads = dh / 4;
  const int t = blockIdx.y * blockDim.x + threadIdx.x;
  if (t >= Hq * quads) return;  // whole heads at a time (quads divides the block size)
  const int h = t / quads, d = (t % quads) * 4;
  // Every load that does not wait on another is issued first: the row's
  // metadata, its q and all split partials (row slots of absent nodes are
  // allocated, so these loads stay unconditional).
  const int n_nodes = meta.n_nodes[b];
  const int P = meta.prefix_len[b];
  const int ns = RAGGED ? meta.n_split[b] : MAXS;
  uint64_t anc = meta.anc[r];
  // the sequence's key splits fill the first of its sp slots and the
  // attention kernel marks the rest empty (m = -inf, l = 0), so the first
  // MAXS (at least the step's largest split count) hold every split
  const long long base = ((long long)b * Hq + h) * sp;
  float ms[MAXS], ls[MAXS];
  float4 os[MAXS];
#pragma unroll
  for (int s = 0; s < MAXS; ++s) {
    const long long row = (base + s) * qrows + i;
    ms[s] = part_ml[row * 2];
    ls[s] = part_ml[row * 2 + 1];
    os[s] = *reinterpret_cast<const float4*>(part_o + row * dh + d);
  }
  const long long qo = ((long long)r * Hq + h) * dh + d;
  const uint2 qh = *reinterpret_cast<const uint2*>(q + qo), ql = *reinterpret_cast<const uint2*>(q_lo + qo);
  float4 out = make_float4(0.f, 0.f, 0.f, 0.f);
  if (i < n_nodes) {  // uniform over the workgroup
    const int hk = h / (Hq / Hkv);
    const float q0 = bf16_to_f32(qh.x & 0xffff) + bf16_to_f32(ql.x & 0xffff);
    const float q1 = bf16_to_f32(qh.x >> 16) + bf16_to_f32(ql.x >> 16);
    const float q2 = bf16_to_f32(qh.y & 0xffff) + bf16_to_f32(ql.y & 0xffff);
    const float q3 = bf16_to_f32(qh.y >> 16) + bf16_to_f32(ql.y >> 16);
    // splits flagged by the attention kernel (their p = 2^(s - m_ref) summed
    // past 2^64, where p may have overflowed): recompute
    // (m, l, o) over the split's prefix keys in fp32 from the bf16 cache, with
    // an exact running maximum
    {
      const int nblk = (P + 31) >> 5;
      const uint16_t* kh = prefix.k + ((long long)b * Hkv + hk) * prefix.kv_cap * dh + d;
      const uint16_t* vh = prefix.v + ((long long)b * Hkv + hk) * prefix.kv_cap * dh;
#pragma unroll
      for (int s = 0; s < MAXS; ++s) {
        if (!(ls[s] < 0.f)) continue;  // uniform over the head's lanes
        const int k0 = 32 * (int)((long long)nblk * s / ns);
        const int k1 = min(P, 32 * (int)((long long)nblk * (s + 1) / ns));
        float m = -INFINITY, l = 0.f;
        float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
        for (int key = k0; key < k1; ++key) {
          const uint2 kk = *reinterpret_cast<const uint2*>(kh + (long long)key * dh);
          float dot = q0 * bf16_to_f32(kk.x & 0xffff) + q1 * bf16_to_f32(kk.x >> 16) +
                      q2 * bf16_to_f32(kk.y & 0xffff) + q3 * bf16_to_f32(kk.y >> 16);
          for (int o2 = quads >> 1; o2 > 0; o2 >>= 1) dot += __shfl_xor(dot, o2, 64);
          const float sj = dot * scale_log2;
          const float mn = fmaxf(m, sj);
          const float al = exp2f(m - mn), e = exp2f(sj - mn);
          // V tiles: element (key, dim) at ((key / 32) * dh + dim) * 32 + key % 32
          const uint16_t* vk = vh + ((long long)(key >> 5) * dh + d) * 32 + (key & 31);
          l = l * al + e;
          o = make_float4(o.x * al + e * bf16_to_f32(vk[0]), o.y * al + e * bf16_to_f32(vk[32]),
                          o.z * al + e * bf16_to_f32(vk[64]), o.w * al + e * bf16_to_f32(vk[96]));
          m = mn;
        }
        ms[s] = m;
        ls[s] = l;
        os[s] = o;
      }
    }
    // tree keys
    const float* tk = tree.k + ((long long)b * Hkv + hk) * max_tree * dh + d;
    const float* tv = tree.v + ((long long)b * Hkv + hk) * max_tree * dh + d;
    float mt = -INFINITY, lt = 0.f;
    float4 ot = make_float4(0.f, 0.f, 0.f, 0.f);
    constexpr int TB = 8;  // ancestors per batch: all their loads are issued before any is used
    while (anc) {          // uniform over the workgroup (one row)
      int js[TB];
      bool ok[TB];
#pragma unroll
      for (int u = 0; u < TB; ++u) {
        ok[u] = anc != 0;
        js[u] = ok[u] ? __builtin_ctzll(anc) : 0;
        anc &= anc - 1;
      }
      float4 k4[TB], v4[TB];
#pragma unroll
      for (int u = 0; u < TB; ++u) {
        k4[u] = *reinterpret_cast<const float4*>(tk + (long long)js[u] * dh);
        v4[u] = *reinterpret_cast<const float4*>(tv + (long long)js[u] * dh);
      }
      // the batch's scores side by side: TB independent dot products and
      // shuffle reductions, one maximum, then the exponentials (a chain of
      // dependent per-key updates measured 1.3 us slower per launch)
      float sc[TB];
#pragma unroll
      for (int u = 0; u < TB; ++u) sc[u] = q0 * k4[u].x + q1 * k4[u].y + q2 * k4[u].z + q3 * k4[u].w;
      for (int o = quads >> 1; o > 0; o >>= 1)
#pragma unroll
        for (int u = 0; u < TB; ++u) sc[u] += __shfl_xor(sc[u], o, 64);
      float mn = mt;
#pragma unroll
      for (int u = 0; u < TB; ++u) {
        sc[u] = ok[u] ? sc[u] * scale_log2 : -INFINITY;
        mn = fmaxf(mn, sc[u]);
      }
      const float al = exp2f(mt - mn);
      lt *= al;
      ot = make_float4(ot.x * al, ot.y * al, ot.z * al, ot.w * al);
#pragma unroll
      for (int u = 0; u < TB; ++u) {
        if (!ok[u]) break;  // uniform over the workgroup
        const float e = exp2f(sc[u] - mn);
        lt += e;
        ot = make_float4(ot.x + e * v4[u].x, ot.y + e * v4[u].y, ot.z + e * v4[u].z, ot.w + e * v4[u].w);
      }
      mt = mn;
    }
    float M = mt;
#pragma unroll
    for (int s = 0; s < MAXS; ++s) M = fmaxf(M, ms[s]);
    const float wt = exp2f(mt - M);
    float4 num = make_float4(wt * ot.x, wt * ot.y, wt * ot.z, wt * ot.w);
    float den = wt * lt;
#pragma unroll
    for (int s = 0; s < MAXS; ++s)
      if (ms[s] != -INFINITY) {
        const float w = exp2f(ms[s] - M);
        num.x += w * os[s].x; num.y += w * os[s].y; num.z += w * os[s].z; num.w += w * os[s].w;
        den += w * ls[s];
      }
    const float inv = 1.f / den;
    out = make_float4(num.x * inv, num.y * inv, num.z * inv, num.w * inv);
  }
  uint16_t* dst = o_out + xpack_off(r, h * dh + d, o_ks);
  const Hilo2 p0 = pack_hilo2(out.x, out.y), p1 = pack_hilo2(out.z, out.w);
  *reinterpret_cast<uint2*>(dst) = make_uint2(p0.hi, p1.hi);
  *reinterpret_cast<uint2*>(dst + XPACK_LO) = make_uint2(p0.lo, p1.lo);
}

hipError_t launch_attn_combine(const float* part_o, const float* part_ml, StepMeta meta, int Hq, int Hkv, int dh,
                               int slots, int sp, int qrows, int max_tree, int row0, int rows, const uint16_t* q,
                               const uint16_t* q_lo, TreeKV32 tree, PrefixKV prefix, float scale_log2,
                               uint16_t* o_out, int o_ks, hipStream_t s) {
  const int quads = dh / 4;
  if (256 % quads != 0 || slots < 1 || slots > sp) return hipErrorInvalidValue;
  const int items = Hq * quads;
  const dim3 grid(rows, (items + 255) / 256);
  switch (slots) {
#define GRIFFIN_COMB_CASE(n)                                                                                   \
  case n:                                                                                                     \
    if (meta.split_tab)                                                                                       \
      hipLaunchKernelGGL((attn_combine_kernel<n, true>), grid, dim3(256), 0, s, part_o, part_ml, meta, Hq, Hkv,   \
                         dh, sp, qrows, max_tree, q, q_lo, tree, prefix, scale_log2, o_out, o_ks, row0);          \
    else                                                                                                      \
      hipLaunchKernelGGL((attn_combine_kernel<n, false>), grid, dim3(256), 0, s, part_o, part_ml, meta, Hq, Hkv,  \
                         dh, sp, qrows, max_tree, q, q_lo, tree, prefix, scale_log2, o_out, o_ks, row0);          \
    break;
    GRIFFIN_COMB_CASE(1) GRIFFIN_COMB_CASE(2) GRIFFIN_COMB_CASE(3) GRIFFIN_COMB_CASE(4) GRIFFIN_COMB_CASE(5)
    GRIFFIN_COMB_CASE(6) GRIFFIN_COMB_CASE(7) GRIFFIN_COMB_CASE(8) GRIFFIN_COMB_CASE(9) GRIFFIN_COMB_CASE(10)
    GRIFFIN_COMB_CASE(11) GRIFFIN_COMB_CASE(12) GRIFFIN_COMB_CASE(13) GRIFFIN_COMB_CASE(14) GRIFFIN_COMB_CASE(15)
    GRIFFIN_COMB_CASE(16)
#undef GRIFFIN_COMB_CASE
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace griffin
