// Device code of the rotation of reused keys (Eq. 8, delta form) with the copy of their values: used by the
// kernels of ct_rerope_scatter.hip and, beside the projection of the selected rows, by ct_gemm.hip.
#pragma once

#include "ct_internal.h"

namespace ct {

// Streaming accesses.  Cached keys and values are read once: their loads do not allocate in the
// caches (measured cold: +3 % out of place).  A rotation in place also writes lines nobody reads
// soon, so its stores bypass the caches as well (+17 % at 64 MiB, 5.3 -> 6.0 TB/s at 256 MiB);
// rows written into a layer buffer are read by the attention kernel next and are stored normally.
template <bool NT>
__device__ __forceinline__ u32x4 ld16(const uint16_t* p) {
  if (NT) return __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
  return *reinterpret_cast<const u32x4*>(p);
}
template <bool NT>
__device__ __forceinline__ void st16(uint16_t* p, u32x4 v) {
  if (NT) __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(p));
  else *reinterpret_cast<u32x4*>(p) = v;
}

// Rotate (and optionally copy V for) one token's share owned by this thread.
// STYLE 0: pairs (j, j + D/2); STYLE 1: pairs (2j, 2j + 1).  HEADS > 0 fixes the head count
// at compile time (full unroll, all loads in flight before the first use).
// k_src/k_dst (and v_src/v_dst) may be the same row: a thread reads all it owns before it
// writes, and no two threads own the same bytes.
template <int D, int STYLE, int HEADS, bool NT_STORE = false>
__device__ __forceinline__ void rerope_token(const uint16_t* k_src, uint16_t* k_dst, const uint16_t* v_src,
                                             uint16_t* v_dst, int32_t delta, int jg, int n_heads_rt,
                                             const RopeTable& table) {
  const int n_heads = HEADS > 0 ? HEADS : n_heads_rt;
  float cs[8], sn[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) sincos_turns(delta, table.turns[jg * 8 + i], cs[i], sn[i]);

  // element offsets (in bf16) of the two 16-byte pieces this thread owns inside a head row
  const int off_a = STYLE == 0 ? jg * 8 : jg * 16;
  const int off_b = STYLE == 0 ? jg * 8 + D / 2 : jg * 16 + 8;

  auto rotate_head = [&](u32x4 a, u32x4 b, u32x4& ra, u32x4& rb) {
    if (STYLE == 0) {
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        float a0 = bf16_lo(a[w]), a1 = bf16_hi(a[w]);
        float b0 = bf16_lo(b[w]), b1 = bf16_hi(b[w]);
        float c0 = cs[2 * w], s0 = sn[2 * w], c1 = cs[2 * w + 1], s1 = sn[2 * w + 1];
        ra[w] = pack_bf16(a0 * c0 - b0 * s0, a1 * c1 - b1 * s1);
        rb[w] = pack_bf16(a0 * s0 + b0 * c0, a1 * s1 + b1 * c1);
      }
    } else {
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        float x = bf16_lo(a[w]), y = bf16_hi(a[w]);
        ra[w] = pack_bf16(x * cs[w] - y * sn[w], x * sn[w] + y * cs[w]);
        float x2 = bf16_lo(b[w]), y2 = bf16_hi(b[w]);
        rb[w] = pack_bf16(x2 * cs[4 + w] - y2 * sn[4 + w], x2 * sn[4 + w] + y2 * cs[4 + w]);
      }
    }
  };

  if (HEADS > 0) {
    u32x4 a[HEADS > 0 ? HEADS : 1], b[HEADS > 0 ? HEADS : 1];
#pragma unroll
    for (int h = 0; h < HEADS; ++h) {
      a[h] = ld16<true>(k_src + h * D + off_a);
      b[h] = ld16<true>(k_src + h * D + off_b);
    }
#pragma unroll
    for (int h = 0; h < HEADS; ++h) {
      u32x4 ra, rb;
      rotate_head(a[h], b[h], ra, rb);
      st16<NT_STORE>(k_dst + h * D + off_a, ra);
      st16<NT_STORE>(k_dst + h * D + off_b, rb);
    }
    if (v_src != nullptr) {
#pragma unroll
      for (int h = 0; h < HEADS; ++h) {
        a[h] = ld16<true>(v_src + h * D + off_a);
        b[h] = ld16<true>(v_src + h * D + off_b);
      }
#pragma unroll
      for (int h = 0; h < HEADS; ++h) {
        st16<NT_STORE>(v_dst + h * D + off_a, a[h]);
        st16<NT_STORE>(v_dst + h * D + off_b, b[h]);
      }
    }
  } else {
    for (int h = 0; h < n_heads; ++h) {
      u32x4 a = ld16<true>(k_src + h * D + off_a);
      u32x4 b = ld16<true>(k_src + h * D + off_b);
      u32x4 ra, rb;
      rotate_head(a, b, ra, rb);
      st16<NT_STORE>(k_dst + h * D + off_a, ra);
      st16<NT_STORE>(k_dst + h * D + off_b, rb);
      if (v_src != nullptr) {
        u32x4 va = ld16<true>(v_src + h * D + off_a);
        u32x4 vb = ld16<true>(v_src + h * D + off_b);
        st16<NT_STORE>(v_dst + h * D + off_a, va);
        st16<NT_STORE>(v_dst + h * D + off_b, vb);
      }
    }
  }
}

// Sorted skip lists (the recompute set: rows that are overwritten by the scatter and need not be
// moved).  count_below: number of listed rows < row, by binary search.
__device__ __forceinline__ int count_below(const int32_t* __restrict__ list, int n, int32_t row) {
  int lo = 0, hi = n;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (list[mid] < row) lo = mid + 1; else hi = mid;
  }
  return lo;
}
// The rows of one wave lie next to each other: the whole wave searches the list for its first row, 64 probes at a time
// (two or three rounds of loads instead of one per bit), and takes the entries from there on into a register each, where every lane
// compares its own row with them.  Rows far from the first one (a gap between chunks) search on their own.
// With one search by halves per workgroup and a walk over the entries in memory per thread, and a walk over the chunk table
// with a load per chunk, 6964 of 8192 rows (8 heads of 128, 8 chunks) took 15.7 us.
struct SkipWindow {
  int32_t first_row;
  int below, n_near;   // entries below first_row; entries in [first_row, first_row + rows)
  int32_t entry;       // this lane's entry: number `below + lane` of the list
};
// All lanes of the wave must come here with the same first_row.
__device__ __forceinline__ SkipWindow skip_window(const int32_t* __restrict__ list, int n, int32_t first_row, int rows) {
  const int lane = threadIdx.x & 63;
  int lo = 0, len = n;
  while (len > 0) {
    const int step = (len + 63) >> 6, at = lane * step + step - 1;   // the last entry of this lane's block
    const bool block_below = at < len && list[lo + at] < first_row;
    const int k = __popcll(__ballot(block_below));                   // the blocks 0 .. k - 1 lie below the row
    lo += k * step;
    len = min(step - 1, len - k * step);
  }
  SkipWindow w;
  w.first_row = first_row;
  w.below = lo;
  w.entry = lo + lane < n ? list[lo + lane] : 0x7fffffff;
  w.n_near = __popcll(__ballot(w.entry < first_row + rows));
  return w;
}
// Number of listed rows < row, and whether the row itself is listed.
__device__ __forceinline__ int find_near(const SkipWindow& w, const int32_t* __restrict__ list, int n, int32_t row, int rows, bool* listed) {
  int below = w.below;
  bool hit = false;
  for (int i = 0; i < w.n_near; ++i) {
    const int32_t e = __builtin_amdgcn_readlane(w.entry, i);
    below += e < row;
    hit |= e == row;
  }
  if (row < w.first_row || row - w.first_row >= rows) {
    below = count_below(list, n, row);
    hit = below < n && list[below] == row;
  }
  *listed = hit;
  return below;
}

// Chunk of token t: the same walk for all lanes, scalar loads that do not wait for one another.
// (Token numbers stay below 2^24, the limit of the layer buffers' rows.)
__device__ __forceinline__ int chunk_of(const ReropeChunks& chunks, int32_t t) {
  int c = 0;
#pragma unroll 4
  for (int i = 1; i < chunks.n; ++i) c += t >= (int32_t)chunks.tok_start[i];
  return c;
}

// Several chunks in one launch: buffer row -> chunk by search in the (small) table.  The work of workgroup
// `block` of `n_blocks`.
// NEAR: the grid covers every token once, so a wave's rows are neighbours and share one search
// of the skip list; otherwise (few workgroups striding over the tokens) every token searches.
template <int D, int STYLE, int HEADS, bool NEAR>
__device__ __forceinline__ void rerope_chunk_tokens(uint16_t* k_buf, uint16_t* v_buf, int32_t n_heads_rt,
                                                    const RopeTable& table, const ReropeChunks& chunks, int threads,
                                                    uint32_t block, uint32_t n_blocks) {
  constexpr int GROUPS = D / 16;
  constexpr int WAVE_ROWS = 64 / GROUPS;
  const int64_t gid = (int64_t)block * threads + threadIdx.x;
  const int jg = (int)(gid % GROUPS);
  const int64_t t_step = (int64_t)n_blocks * (threads / GROUPS);
  SkipWindow near = {};
  if (NEAR && chunks.skip_rows != nullptr) {
    const int32_t t0 = __builtin_amdgcn_readfirstlane((int32_t)(gid / GROUPS));   // the wave's first token
    const int c0 = __builtin_amdgcn_readfirstlane(chunk_of(chunks, t0));
    near = skip_window(chunks.skip_rows, chunks.n_skip, chunks.row_start[c0] + (t0 - (int32_t)chunks.tok_start[c0]), WAVE_ROWS);
  }
  for (int64_t t_all = gid / GROUPS; t_all < chunks.total_tokens; t_all += t_step) {   // ordinal among the listed tokens
    const int c = chunk_of(chunks, (int32_t)t_all);
    const int32_t t = (int32_t)(t_all - chunks.tok_start[c]);
    int32_t t_src = t;   // row inside the chunk's source
    if (chunks.skip_rows != nullptr) {   // is this buffer row in the sorted skip list?
      const int32_t row = chunks.row_start[c] + t;
      bool listed;
      int lo;
      if (NEAR) {
        lo = find_near(near, chunks.skip_rows, chunks.n_skip, row, WAVE_ROWS, &listed);
      } else {
        lo = count_below(chunks.skip_rows, chunks.n_skip, row);
        listed = lo < chunks.n_skip && chunks.skip_rows[lo] == row;
      }
      if (listed) continue;
      // a compact source holds only the rows that are kept: step over the skipped ones before this row
      if ((chunks.compact_mask >> c) & 1u) t_src = t - (lo - count_below(chunks.skip_rows, chunks.n_skip, chunks.row_start[c]));
    }
    const int64_t heads = HEADS > 0 ? HEADS : n_heads_rt;
    const int64_t src_row = (int64_t)t_src * heads * D;
    const int64_t dst_row = ((int64_t)chunks.row_start[c] + t) * heads * D;
    const uint16_t* ks = static_cast<const uint16_t*>(chunks.k_src[c]) + src_row;
    const uint16_t* vs = chunks.v_src[c] ? static_cast<const uint16_t*>(chunks.v_src[c]) + src_row : nullptr;
    const int32_t delta = chunks.delta0[c] + chunks.delta_step[c] * t;
    rerope_token<D, STYLE, HEADS>(ks, k_buf + dst_row, vs, v_buf + dst_row, delta, jg, n_heads_rt, table);
  }
}

}  // namespace ct
