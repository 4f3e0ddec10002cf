// Causal attention for the selected query rows over the fused layer KV (Sec. 4.2: the
// check / fusion layers compute attention for the selected tokens alone), GQA aware.
//
// Formulation.  Everything is computed transposed so that a lane owns a query column:
//   S^T = K Q^T            A = K tile rows (keys) from LDS,       B = Q^T kept in registers
//   O^T += V^T P^T         A = V^T (head_dim x keys) from LDS,    B = P^T taken straight from
//                                                                     the S^T accumulators
// In the 16x16 MFMA accumulator layout lane l holds column l%16 (one query) and 4 rows (keys) of each
// tile, so the row maximum and row sum of the softmax are in-lane reductions plus an exchange
// between the four rows of 16 lanes, the rescale factor of the online softmax is a per-lane
// scalar per column tile, and the probabilities need no trip through LDS: the accumulators of the
// 16-key tiles 2t and 2t+1 are exactly the B operand of PV step t (32 keys) once V^T is read in the
// same key order (lane row h takes keys 32t + 4h + 0..3 and 32t + 16 + 4h + 0..3).
// 16 x 16 x 32 and not 32 x 32 x 16: the chip is limited by power, and an accumulator tile that is
// read and written half as often per flop costs less of it (nothing but MFMAs on data-like operands:
// 2.10 PFLOP/s against 1.83).  32768 tokens, 32/8 heads of 128, all rows: 7.59 -> 7.07 ms, 4915 rows
// 1.258 -> 1.189 ms; where the clock is not held down by power (few workgroups) the twice as many
// instructions take back part of it.
//
// Work decomposition.  A workgroup (8 waves, two per SIMD) owns one KV head and a tile of 256
// query columns = (256 / G) selected tokens x the G query heads of that KV head; every wave
// owns 32 columns and all keys.  K and V tiles of 64 keys are staged once per workgroup in LDS
// by direct global->LDS loads (three stages each); V^T fragments come out of LDS with
// transposing reads.  The selected rows are sorted, so a tile needs keys [0, last position of
// the tile]; only key tiles that straddle a query position of the wave evaluate the causal mask.
// When (tile, head) pairs are too few to fill the chip, the key range is split and fp32
// partial (O, m, l) are merged by a second kernel; tiles whose keys fit one split write their
// result directly.
// Workgroup ids map KV head = id mod n_kv_heads, so with 8 KV heads every XCD streams the
// keys of one head through its own L2; tiles are issued heaviest first.
#include <math.h>
#include <stdlib.h>

#include <type_traits>

#include "ct_internal.h"

namespace ct {

namespace {

constexpr int BN = 64;                 // keys per LDS tile

struct AttnArgs {
  const uint16_t* q;
  const uint16_t* k;
  const uint16_t* v;
  const int32_t* sel_idx;
  uint16_t* out;
  float* lse;
  float* partial;     // workspace when n_splits > 1
  int32_t n_sel, n_ctx, Hq, Hkv, G, TM, tm_shift, cols;
  int32_t n_tiles, n_splits, split_keys;
  // state == NULL: only tiles whose visible key count lies in (key_after, key_upto] are computed by
  // this launch (the rest by other launches, each started when the rows it needs are in place).
  // state != NULL: this launch takes every tile that sees keys past key_after through the keys
  // [key_after, key_upto) and no further; a tile that needs later keys leaves its fp32
  // (O, m, l) in `state` ([tile][kv head][256 columns][D], then m[256], l[256]) and the launch
  // for the next key range resumes from there.
  int32_t key_after, key_upto;
  float* state;
  float scale_log2;   // softmax scale * log2(e)
};

// The keys one workgroup (tile, key-range split) of a launch works through: [k_lo, k_hi), or nothing.
// Shared by the kernel and by the host-side check of the rows a launch reads.
struct ItemRange {
  int k_lo, k_hi;
  bool active;
};
__host__ __device__ inline ItemRange item_range(int kmax, int split, int split_keys, bool resumable, int key_after,
                                                int key_upto) {
  ItemRange r = {0, 0, false};
  if (kmax <= key_after || (!resumable && kmax > key_upto)) return r;   // another launch's tile
  r.k_lo = resumable ? key_after : split * split_keys;
  if (r.k_lo >= kmax) return r;                                          // empty split
  r.k_hi = resumable ? (key_upto < kmax ? key_upto : kmax)
                     : (r.k_lo + split_keys < kmax ? r.k_lo + split_keys : kmax);
  r.active = true;
  return r;
}
// Row of the K (or V) buffer behind row `row_in_tile` of the LDS tile that starts at key k0: rows from
// k_hi on (the end of the item's key range) are replaced by row k_hi - 1.
__host__ __device__ inline int tile_load_row(int k0, int row_in_tile, int k_hi) {
  const int key = k0 + row_in_tile;
  return key < k_hi - 1 ? key : k_hi - 1;
}

// Reductions over the four 16-lane rows of a wave, of two values x and y at once.
// v_permlane32_swap exchanges the upper half of its first operand with the lower half of the second:
// combining its two results leaves x over (l, l ^ 32) in the lower half and y in the upper one.
// v_permlane16_swap exchanges the odd rows of the first with the even rows of the second, which adds the
// other row of each half, and a last v_permlane32_swap hands both results to all lanes.
template <typename Op>
__device__ __forceinline__ void reduce_rows(float& x, float& y, Op op) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
  uint32_t c = __float_as_uint(op(__uint_as_float(r[0]), __uint_as_float(r[1])));
  r = __builtin_amdgcn_permlane16_swap(c, c, false, false);
  c = __float_as_uint(op(__uint_as_float(r[0]), __uint_as_float(r[1])));
  r = __builtin_amdgcn_permlane32_swap(c, c, false, false);
  x = __uint_as_float(r[0]);
  y = __uint_as_float(r[1]);
}

typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((address_space(3))) void* lds_ptr_t;

// Swizzles of the 16-byte pieces inside a key row of the LDS tiles (rows are unpadded:
// direct global->LDS loads write 64 lanes x 16 bytes contiguously).  K rows are read one
// row per lane (ds_read_b128), V rows four rows per 16-lane block (ds_read_b64_tr_b16).
template <int D>
__device__ __forceinline__ int swz_k(int r) { return D == 128 ? (r & 15) : ((r >> 1) & 7); }
template <int D>
__device__ __forceinline__ int swz_v(int r) { return D == 128 ? (r & 7) << 1 : ((r >> 1) & 3) << 1; }

// A workgroup has 8 waves, two per SIMD; every wave owns 32 query columns (two MFMA column
// tiles) and all keys, so the workgroup owns 256 query columns.
//
// Ping-pong schedule.  The work of a wave on key tile i splits into a matrix-core part
//   M(i): O^T += V^T(i-1) P^T(i-1), then S^T(i) = K(i) Q^T            (64 MFMAs)
// and a vector-ALU part
//   V(i): causal mask, online softmax of S^T(i) into P^T(i), rescale of O^T.
// The loop runs in periods separated by one workgroup barrier.  Waves 0-3 (one per SIMD) run
// M(i) and then V(i) in period i; waves 4-7 run V(i-1) and then M(i).  The two parts take about
// the same time, so each SIMD has one wave feeding the matrix cores and one wave doing softmax
// arithmetic for most of the period without a barrier between the halves (a second barrier
// there makes every wave wait for the slowest of eight twice per period: measured 2 % slower).
// K(i) and V(i-1) are the tiles in use during period i; K(i+2) and V(i+1) are fetched during
// it with direct global->LDS loads into three K and three V stages.
// One loop for both groups, V(i) then M(i+1), with the barrier between the two for waves 0-3 and
// behind them for waves 4-7: written as two loops, the compiler kept the initial accumulators for both
// (253 registers and scratch reloads in the loop; 190 now).
template <int D>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void attn_kernel(AttnArgs a) {
  constexpr int NWAVES = 8;
  constexpr int COLS = 32 * NWAVES;            // query columns per workgroup
  constexpr int NST = 3;                       // LDS stages per tensor
  constexpr int ROWB = D * 2;                  // bytes per key row in LDS (no padding)
  constexpr int TILE_BYTES = BN * ROWB;        // one K (or V) tile
  constexpr int KS = D / 32;                   // MFMA k-steps over head_dim
  constexpr int MT = D / 16;                   // O^T row tiles
  constexpr int PCS = D / 8;                   // 16-byte pieces per key row
  constexpr int RPI = 64 / PCS;                // key rows covered by one wave-wide 16-byte load
  constexpr int INSTS = BN / RPI / NWAVES;     // such loads per wave, tile and tensor
  static_assert(INSTS >= 1 && (NWAVES * RPI) % 16 == 0, "tile / wave count mismatch");

  __shared__ __align__(1024) unsigned char lds[2 * NST * TILE_BYTES];     // stages of K, then of V
  constexpr int V_LDS = NST * TILE_BYTES;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, h = lane >> 4;
  const bool group_b = wave >= NWAVES / 2;

  // ---- work item ---------------------------------------------------------------------------
  const int g = blockIdx.x % a.Hkv;
  const int rest = blockIdx.x / a.Hkv;
  // split-major order: the workgroups resident on an XCD at one time work on neighbouring
  // tiles of the same key range and share its K/V lines in that XCD's L2
  const int split = rest / a.n_tiles;
  const int tile = a.n_tiles - 1 - rest % a.n_tiles;    // heaviest (latest) tiles first
  const int tok0 = tile * a.TM;
  const int last_tok = min(tok0 + a.TM, a.n_sel) - 1;
  const int kmax = a.sel_idx[last_tok] + 1;              // keys this tile can see
  const bool resumable = a.state != nullptr;
  const ItemRange item = item_range(kmax, split, a.split_keys, resumable, a.key_after, a.key_upto);
  if (!item.active) return;                              // uniform for the workgroup
  const int k_lo = item.k_lo, k_hi = item.k_hi;
  const int n_kt = (k_hi - k_lo + BN - 1) / BN;

  // ---- this lane's two query columns (16 apart) ----------------------------------------------------
  // row of q and out behind the lane's column n (of a token that is not there: the last one's)
  auto query_row = [&](int col, bool& valid, int& tokv) __attribute__((always_inline)) -> size_t {
    const int tok_raw = tok0 + (col & (a.TM - 1));
    valid = tok_raw < a.n_sel;
    tokv = valid ? tok_raw : a.n_sel - 1;
    return (size_t)tokv * a.Hq + g * a.G + (col >> a.tm_shift);
  };
  int pos[2];
  bf16x8 qf[2][KS];     // Q^T fragments: B operand, lane = column, 8 consecutive head_dim elements per k-step
#pragma unroll
  for (int n = 0; n < 2; ++n) {
    bool valid;
    int tokv;
    const uint16_t* qp = a.q + query_row(wave * 32 + l16 + 16 * n, valid, tokv) * D + h * 8;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) qf[n][ks] = *reinterpret_cast<const bf16x8*>(qp + ks * 32);
    // keys from k_hi on belong to a later launch (or to nobody): the causal mask is taken against
    // min(position, k_hi - 1), which cuts the last key tile of the range where the range ends
    pos[n] = min(a.sel_idx[tokv], k_hi - 1);
  }
  int wmin = min(pos[0], pos[1]);
#pragma unroll
  for (int off = 8; off >= 1; off >>= 1) wmin = min(wmin, __shfl_xor(wmin, off));
  wmin = __builtin_amdgcn_readfirstlane(wmin);

  // ---- global -> LDS staging (direct loads, no registers) ----------------------------------
  // load i of this wave fills LDS rows (NWAVES * i + wave) * RPI .. + RPI - 1 of a tile; this
  // lane supplies physical piece lane % PCS of row lane / PCS, i.e. logical piece
  // (that ^ swizzle); NWAVES * RPI is a multiple of 16 rows, so the swizzle is the same for all i
  const int ld_row = wave * RPI + lane / PCS;
  const int ld_pk = (lane % PCS) ^ swz_k<D>(ld_row);
  const int ld_pv = (lane % PCS) ^ swz_v<D>(ld_row);
  // byte offsets from the tensor bases fit 32 bits and row numbers 24 (checked on the host)
  const uint32_t kv_row_bytes = (uint32_t)a.Hkv * D * 2;
  const uint32_t k_lane_off = ((uint32_t)g * D + ld_pk * 8) * 2;
  const uint32_t v_lane_off = ((uint32_t)g * D + ld_pv * 8) * 2;
  // The loads are inline assembly (M0 = LDS base of the wave's 1 KiB slot, each lane lands at
  // +16 * lane): the compiler neither reorders them nor adds waits of its own; the pipeline
  // below orders them against the fragment reads with explicit vmcnt waits and barriers.
  const uint32_t lds_addr = (uint32_t)(uintptr_t)(lds_ptr_t)lds;
  const uint32_t lds_wave = __builtin_amdgcn_readfirstlane(lds_addr + wave * 1024);     // where this wave's first load of stage 0 goes
  // One wave-wide load: rows (NWAVES * idx + wave) * RPI .. of the tile that starts at key k0.
  // Rows from k_hi on (the end of this item's key range) are replaced by row k_hi - 1: they are
  // masked (their probabilities are zero), or belong to look-ahead tiles that are never consumed,
  // but what stands in those rows may not have been written yet - a later group of chunks still on
  // the host link - and a non-finite bit pattern there would turn 0 * v into NaN in the PV product.
  auto row_offset = [&](int k0, int idx) __attribute__((always_inline)) -> uint32_t {
    return __umul24(tile_load_row(k0, ld_row + NWAVES * RPI * idx, k_hi), kv_row_bytes);
  };
  // (`to`: LDS address of the wave's first load in a K stage, uniform; `at`: bytes from there)
  auto load16 = [&](const uint16_t* base, uint32_t byte_off, uint32_t to, int at) __attribute__((always_inline)) {
    asm volatile("s_add_u32 m0, %0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 : : "s"(to), "v"(byte_off), "s"(base), "i"(at) : "memory", "m0", "scc");
  };
  auto issue_rows = [&](const uint16_t* base, uint32_t lane_off, int k0, int at) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < INSTS; ++i) load16(base, row_offset(k0, i) + lane_off, lds_wave, at + i * NWAVES * 1024);
  };

  // ---- per-lane LDS read offsets ----------------------------------------------------------------
  // K fragment (16-key tile u, k-step ks): row 16u + l16, logical piece 4ks + h, i.e. byte offset
  //   l16 * ROWB + ((4ks + h) ^ swizzle) * 16 + u * 16 * ROWB  =  (k_a ^ (ks << 6)) + u * 16 * ROWB,
  // because the swizzle is an exclusive-or on bits the row term leaves clear: one register holds
  // k_a and every fragment address is that register exclusive-or a constant.
  const int k_a = l16 * ROWB + ((h ^ swz_k<D>(l16)) * 16);
  // V^T fragment (row tile m, 32-key step t, half a2): 16-lane block h reads 4 key rows x
  // 16 head_dim columns; lane j of the block addresses row j / 4, 8-byte chunk j % 4:
  //   r = 4h + j / 4 (+ 32t + 16 a2, which leave the swizzle unchanged), piece pc = 2m + j % 4 / 2,
  //   offset r * ROWB + (pc ^ swizzle(r)) * 16 + 8 (j % 2)  =  (v_a ^ (m << 5)) + (32t + 16 a2) * ROWB.
  const int v_r = 4 * h + (l16 >> 2);
  const int v_a = v_r * ROWB + ((((l16 & 3) >> 1) ^ swz_v<D>(v_r)) * 16) + 8 * (l16 & 1);

  // ---- state ---------------------------------------------------------------------------------------
  f32x4 o[MT][2];
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int n = 0; n < 2; ++n) o[m][n] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m_run[2] = {-INFINITY, -INFINITY};
  float l_run[2] = {0.f, 0.f};   // per-lane partial row sums; the four rows of lanes are added at the end
  if (resumable && k_lo > 0) {   // what the launch for the previous key range left
    const float* base = a.state + ((size_t)tile * a.Hkv + g) * (size_t)(COLS * (D + 2));
#pragma unroll
    for (int n = 0; n < 2; ++n) {
      const int col = wave * 32 + l16 + 16 * n;
      const float* op = base + (size_t)col * D + 4 * h;
#pragma unroll
      for (int m = 0; m < MT; ++m) o[m][n] = *reinterpret_cast<const f32x4*>(op + m * 16);
      m_run[n] = base[COLS * D + col];
      l_run[n] = h == 0 ? base[COLS * D + COLS + col] : 0.f;
    }
  }
  // scores above which the reference of the exponents moves: 2^8 above it
  const float limit_step = 8.0f / a.scale_log2;
  float m_limit[2];
#pragma unroll
  for (int n = 0; n < 2; ++n) m_limit[n] = m_run[n] == -INFINITY ? -INFINITY : m_run[n] / a.scale_log2 + limit_step;
  f32x4 s[4][2];       // S^T of the tile whose scores were computed last (four 16-key tiles)
  bf16x8 pf[2][2];     // P^T fragments (32-key step t, column tile n) of the tile whose softmax was done last

  typedef __attribute__((ext_vector_type(8))) short s16x8;

  // ---- M part: O^T += V^T P^T (previous tile), S^T = K Q^T (this tile) ----------------------------
  // One stream of NPV + NQK fragments, two MFMAs (one per column tile) each.  With one wave per SIMD in
  // this part nothing else hides the LDS latency, so the reads run PD fragments ahead of their MFMAs
  // through a ring of PD + 1, across the PV -> QK boundary as well, one LDS instruction per MFMA:
  // a wave issues in order, one LDS instruction per ~15 cycles, about the time of an MFMA (both reads
  // of a V^T fragment in a row: 3 % of the launch).  Distances of 2 to 4 measure the same within 0.5 %, 5 costs 1 to 2 %.
  // MFMAs, reads, tile loads and nothing else: a vector instruction between two MFMAs of a wave waits for the
  // first of them, so addresses are worked out behind the part and not where they are used.  The tile loads go out one
  // by one, every fourth fragment of the PV half: together ahead of the first MFMA they hold it up.
  // With those two, before / now: 32768 tokens, 4915 rows, 32/8 heads of 128 1093 / 1083 us, 8/2 heads of 64
  // 284 / 271; 2048 tokens, 307 rows, 32/8 heads of 128 48.8 / 48.1, 8/2 of 64 41.5 / 39.7.  Not kept: addresses in
  // the gaps of the QK half (heads of 128 5 to 10 % slower), loads there (up to 10 %) or ahead of the softmax of waves
  // 4-7 (10 to 20 %), a fourth stage per tensor with the loads a tile further ahead (+-0.5 %), the loop written out for the three stages, so
  // that no address changes (the accumulators then change registers from period to period, and spill).
  // The wave runs it at raised priority: its instruction stream is sparse and must not queue
  // behind the dense softmax stream of the other wave on the SIMD (without: 4 to 6 % of the launch).
  // The first M part has no previous tile and runs the QK half alone, the last one the PV half.
  constexpr int NPV = 2 * MT, NQK = 4 * KS;
#ifndef CT_ATTN_PD
#define CT_ATTN_PD 3
#endif
  constexpr int PD = CT_ATTN_PD;
  static_assert(8 * INSTS <= NPV, "tile loads lie in the PV half");
  // M part i reads V(i-1) and K(i) at `va` and `ka`, and sends for K(i+2) and V(i+1): rows at `off_k` and
  // `off_v`, into the stages of K(i-1) and V(i-2), which nobody reads any more.
  uint32_t va[MT], ka[KS], off_k[INSTS], off_v[INSTS];
  uint32_t st_p = lds_wave + 2 * TILE_BYTES, st_c = lds_wave, st_n = lds_wave + TILE_BYTES;     // stages of tiles i - 1, i, i + 1
  const uint32_t k_to_v = v_lane_off - k_lane_off;
  int next_row = k_lo + 3 * BN + ld_row;                                      // row of K(i+3) for this lane's first load
#pragma unroll
  for (int m = 0; m < MT; ++m) va[m] = lds_addr + V_LDS + 2 * TILE_BYTES + (v_a ^ (m << 5));
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) ka[ks] = lds_addr + (k_a ^ (ks << 6));
#pragma unroll
  for (int x = 0; x < INSTS; ++x) {
    off_k[x] = row_offset(k_lo + 2 * BN, x) + k_lane_off;
    off_v[x] = row_offset(k_lo + BN, x) + v_lane_off;
  }
  auto refill = [&](int x) __attribute__((always_inline)) {
    if (x < INSTS) load16(a.k, off_k[x], st_p, x * NWAVES * 1024);
    else load16(a.v, off_v[x - INSTS], st_n, V_LDS + (x - INSTS) * NWAVES * 1024);
  };
  // (the asm statements keep this here)
  auto next_addresses = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int x = 0; x < INSTS; ++x) {
      off_v[x] = off_k[x] + k_to_v;
      off_k[x] = __umul24(tile_load_row(next_row, NWAVES * RPI * x, k_hi), kv_row_bytes) + k_lane_off;
      asm volatile("" : "+v"(off_v[x]), "+v"(off_k[x]));
    }
    next_row += BN;
#pragma unroll
    for (int m = 0; m < MT; ++m) {
      va[m] += st_c - st_p;
      asm volatile("" : "+v"(va[m]));
    }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      ka[ks] += st_n - st_c;
      asm volatile("" : "+v"(ka[ks]));
    }
    const uint32_t p = st_p;
    st_p = st_c;
    st_c = st_n;
    st_n = p;
  };
  // V^T fragments take two LDS instructions (halves of their keys), K fragments one.
  s16x8 fr[PD + 1];
  typedef __attribute__((address_space(3))) const unsigned char* lds_bytes_t;
  auto load_first = [&](int j) __attribute__((always_inline)) {
    s16x8& f = fr[j % (PD + 1)];
    if (j < NPV) {
      const s16x4 x = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
          (__attribute__((address_space(3))) s16x4*)((lds_bytes_t)va[j % MT] + 32 * (j / MT) * ROWB));
      f = __builtin_shufflevector(x, x, 0, 1, 2, 3, -1, -1, -1, -1);
    } else {
      const int ks = (j - NPV) >> 2, u = (j - NPV) & 3;
      f = *(__attribute__((address_space(3))) const s16x8*)((lds_bytes_t)ka[ks] + u * 16 * ROWB);
    }
  };
  auto load_second = [&](int j) __attribute__((always_inline)) {
    if (j >= NPV) return;
    s16x8& f = fr[j % (PD + 1)];
    const s16x4 x = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (__attribute__((address_space(3))) s16x4*)((lds_bytes_t)va[j % MT] + (32 * (j / MT) + 16) * ROWB));
    f = __builtin_shufflevector(f, __builtin_shufflevector(x, x, 0, 1, 2, 3, -1, -1, -1, -1), 0, 1, 2, 3, 8, 9, 10, 11);
  };
  auto part_m = [&](auto first, auto end) __attribute__((always_inline)) {
    constexpr int J0 = decltype(first)::value, J1 = decltype(end)::value;
    __builtin_amdgcn_s_setprio(3);
#pragma unroll
    for (int j = J0; j < J0 + PD; ++j) {
      load_first(j);
      load_second(j);
    }
    if (J0 == NPV) {     // (no PV half to send them from)
#pragma unroll
      for (int x = 0; x < 2 * INSTS; ++x) refill(x);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = J0; j < J1; ++j) {
#pragma unroll
      for (int n = 0; n < 2; ++n) {
        if (j + PD < J1 && n == 0) load_first(j + PD);
        if (j + PD < J1 && n == 1) load_second(j + PD);
        if (J0 == 0 && J1 > NPV && n == 1 && j % 4 == 0 && j / 4 < 2 * INSTS) {
          refill(j / 4);
          __builtin_amdgcn_sched_barrier(0);
        }
        const bf16x8 f = *reinterpret_cast<const bf16x8*>(&fr[j % (PD + 1)]);
        if (j < NPV) {
          const int t = j / MT, m = j % MT;
          o[m][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f, pf[t][n], o[m][n], 0, 0, 0);
        } else {
          const int ks = (j - NPV) >> 2, u = (j - NPV) & 3;
          const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
          s[u][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f, qf[n][ks], ks == 0 ? zero : s[u][n], 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);   // keep the read-ahead distance as written
      }
    }
    __builtin_amdgcn_s_setprio(0);
    if (J1 > NPV) next_addresses();
  };

  // ---- V part: causal mask, online softmax, P^T fragments, rescale of O^T -------------------------
  auto part_v = [&](int k0) __attribute__((always_inline)) {
    if (k0 + BN - 1 > wmin) {   // only tiles that reach past the earliest query of this wave
#pragma unroll
      for (int n = 0; n < 2; ++n) {
        const int rel = pos[n] - k0 - 4 * h;   // key offsets 16u + i <= rel are visible
        // Four selections at once.  Element by element the compiler joins their conditions: 100 instructions and
        // 90 scalar registers, where few rows, far apart, mask nearly every tile (32/8 heads of 128, 100 rows of 2048
        // tokens 49.5 -> 48.6 us; 16/8 heads 55.8 -> 54.1).
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const f32x4 x = s[u][n];
          s[u][n] = f32x4{rel < 16 * u ? -INFINITY : x[0], rel < 16 * u + 1 ? -INFINITY : x[1],
                          rel < 16 * u + 2 ? -INFINITY : x[2], rel < 16 * u + 3 ? -INFINITY : x[3]};
        }
      }
    }
    // The reference of the exponents follows the running maximum lazily: it moves only when the
    // tile's maximum exceeds it by more than 2^8, so probabilities stay below 256 (bf16 keeps
    // their relative precision, the sums are fp32) and the rescale of O^T becomes rare.  A
    // rescale in one wave holds up the whole workgroup at the next barrier, and with the exact
    // maximum some wave of the eight has one in most periods.
    float mx[2];
#pragma unroll
    for (int n = 0; n < 2; ++n) {
      mx[n] = m_limit[n];
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int i = 0; i < 4; ++i) mx[n] = fmaxf(mx[n], s[u][n][i]);
    }
    reduce_rows(mx[0], mx[1], [](float x, float y) { return fmaxf(x, y); });
    if (__any(mx[0] > m_limit[0] || mx[1] > m_limit[1])) {
#pragma unroll
      for (int n = 0; n < 2; ++n) {
        if (mx[n] > m_limit[n]) {
          const float m_new = mx[n] * a.scale_log2;
          const float alpha = __builtin_amdgcn_exp2f(m_run[n] - m_new);   // (0 from the first reference on)
          m_run[n] = m_new;
          m_limit[n] = mx[n] + limit_step;
          l_run[n] *= alpha;
#pragma unroll
          for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int i = 0; i < 4; ++i) o[m][n][i] *= alpha;
        }
      }
    }
#pragma unroll
    for (int n = 0; n < 2; ++n) {
      const float m_use = m_run[n] == -INFINITY ? 0.f : m_run[n];
      float rs0 = 0.f, rs1 = 0.f;   // of this tile alone: added to the running sum once, not probability by probability
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int i = 0; i < 4; i += 2) {
          const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[u][n][i], a.scale_log2, -m_use));
          const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[u][n][i + 1], a.scale_log2, -m_use));
          s[u][n][i] = p0;
          s[u][n][i + 1] = p1;
          rs0 = u + i == 0 ? p0 : rs0 + p0;
          rs1 = u + i == 0 ? p1 : rs1 + p1;
        }
      l_run[n] += rs0 + rs1;
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        u32x4 w;
#pragma unroll
        for (int e = 0; e < 4; ++e) w[e] = pack_bf16(s[2 * t + (e >> 1)][n][2 * (e & 1)], s[2 * t + (e >> 1)][n][2 * (e & 1) + 1]);
        asm volatile("" : "+v"(w));   // (as below)
        pf[t][n] = *reinterpret_cast<bf16x8*>(&w);
      }
      // done here, ahead of the barrier: left alone, the compiler moves the sums behind the matrix part and the
      // exponentials behind the barrier
      asm volatile("" : "+v"(l_run[n]));
    }
  };

  // ---- the period loop -----------------------------------------------------------------------------
  // Loads past the last tile are still issued (row index clamped) so that the number of loads
  // outstanding at the wait, and with it the wait itself, is the same in every period.
  constexpr int LPP = 2 * INSTS;                                              // loads per wave and period
  constexpr int WAIT_OLDER = (LPP & 15) | ((LPP >> 4) << 14) | 0x0f70;        // s_waitcnt vmcnt(LPP)
  // Every ordinary global load so far (indices, Q fragments) is waited for here, once: the
  // compiler would otherwise guard their first use inside the loop with vmcnt waits that also
  // wait for the look-ahead tile loads.
  __builtin_amdgcn_s_waitcnt(0x0f70);
  issue_rows(a.k, k_lane_off, k_lo, 0);                                    // K(0)
  issue_rows(a.k, k_lane_off, k_lo + BN, TILE_BYTES);                      // K(1)
  issue_rows(a.v, v_lane_off, k_lo, V_LDS);                                // V(0)
  __builtin_amdgcn_s_waitcnt(WAIT_OLDER);                                  // K(0) has landed
  __syncthreads();
  auto end_of_period = [&]() __attribute__((always_inline)) {
    __builtin_amdgcn_s_waitcnt(WAIT_OLDER);     // this wave's loads of the previous period have landed
    __syncthreads();                            // everybody's have; everybody is done with K(i), V(i-1)
  };
  // Period i uses K(i) and V(i-1).  Nothing but the place of the barrier differs between the two groups: both read
  // the same tiles for the whole period.
  using J0 = std::integral_constant<int, 0>;
  using JQK = std::integral_constant<int, NPV>;
  using JEND = std::integral_constant<int, NPV + NQK>;
  part_m(JQK{}, JEND{});
  if (group_b) end_of_period();
  for (int i = 0; i + 1 < n_kt; ++i) {
    part_v(k_lo + i * BN);
    if (!group_b) end_of_period();
    part_m(J0{}, JEND{});
    if (group_b) end_of_period();
  }
  part_v(k_lo + (n_kt - 1) * BN);
  if (!group_b) end_of_period();
  part_m(J0{}, JQK{});
  __builtin_amdgcn_s_waitcnt(0x0f70);           // drain the look-ahead loads before the LDS is released

  // ---- epilogue -------------------------------------------------------------------------------
  float l_tot[2] = {l_run[0], l_run[1]};
  reduce_rows(l_tot[0], l_tot[1], [](float x, float y) { return x + y; });
  int tid_e = threadIdx.x;
  asm("" : "+v"(tid_e));   // places of the results are worked out again here: nothing of them stays in registers during the loop
  const int col_e = (tid_e >> 6) * 32 + (tid_e & 15), h_e = (tid_e >> 4) & 3;
  if (resumable ? k_hi == kmax : kmax <= a.split_keys) {   // the tile's key range ends here: final result
#pragma unroll
    for (int n = 0; n < 2; ++n) {
      bool valid;
      int tokv;
      const size_t row = query_row(col_e + 16 * n, valid, tokv);
      if (!valid) continue;
      const float inv = 1.0f / l_tot[n];
      uint16_t* op = a.out + row * D + 4 * h_e;
#pragma unroll
      for (int m = 0; m < MT; ++m) {
        u32x2 w;
        w[0] = pack_bf16(o[m][n][0] * inv, o[m][n][1] * inv);
        w[1] = pack_bf16(o[m][n][2] * inv, o[m][n][3] * inv);
        *reinterpret_cast<u32x2*>(op + m * 16) = w;
      }
      if (a.lse != nullptr && h_e == 0) a.lse[row] = (m_run[n] + __builtin_log2f(l_tot[n])) * 0.69314718055994531f;
    }
  } else {
    // partial results: [item][COLS columns][D] fp32, then m[COLS], l[COLS]
    const size_t item = ((size_t)tile * a.Hkv + g) * a.n_splits + split;
    float* base = (resumable ? a.state : a.partial) + item * (size_t)(COLS * (D + 2));
#pragma unroll
    for (int n = 0; n < 2; ++n) {
      const int col = col_e + 16 * n;
      float* op = base + (size_t)col * D + 4 * h_e;
#pragma unroll
      for (int m = 0; m < MT; ++m) *reinterpret_cast<f32x4*>(op + m * 16) = o[m][n];
      if (h_e == 0) {
        base[COLS * D + col] = m_run[n];
        base[COLS * D + COLS + col] = l_tot[n];
      }
    }
  }
}

// Merge of the key-range splits: out = sum_i w_i O_i / sum_i w_i l_i, w_i = 2^(m_i - max m).
// One thread owns 4 head_dim elements of one (token, query head).
template <int D>
__global__ __launch_bounds__(256) void attn_merge_kernel(AttnArgs a) {
  constexpr int TPR = D / 4;                       // threads per (token, head) row
  const int64_t gid = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t rowid = gid / TPR;
  const int d4 = (int)(gid % TPR) * 4;
  if (rowid >= (int64_t)a.n_sel * a.Hq) return;
  const int tok = (int)(rowid / a.Hq), h = (int)(rowid % a.Hq);
  const int g = h / a.G, hg = h % a.G;
  const int tile = tok / a.TM;
  const int col = hg * a.TM + (tok - tile * a.TM);
  const int last_tok = min(tile * a.TM + a.TM, a.n_sel) - 1;
  const int kmax = a.sel_idx[last_tok] + 1;
  const int ns = min(a.n_splits, (kmax + a.split_keys - 1) / a.split_keys);
  if (ns == 1) return;                             // written by the attention kernel itself
  const size_t item0 = ((size_t)tile * a.Hkv + g) * a.n_splits;
  const int C = a.cols;
  const size_t istride = (size_t)C * (D + 2);
  float mx = -INFINITY;
  for (int i = 0; i < ns; ++i) mx = fmaxf(mx, a.partial[(item0 + i) * istride + (size_t)C * D + col]);
  float L = 0.f;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  for (int i = 0; i < ns; ++i) {
    const float* base = a.partial + (item0 + i) * istride;
    const float mi = base[(size_t)C * D + col];
    const float w = __builtin_amdgcn_exp2f(mi - mx);     // 0 for a split with nothing visible (m = -inf)
    L += w * base[(size_t)C * D + C + col];
    const f32x4 oi = *reinterpret_cast<const f32x4*>(base + (size_t)col * D + d4);
    if (w > 0.f) acc += w * oi;
  }
  const float inv = 1.0f / L;
  u32x2 w2;
  w2[0] = pack_bf16(acc[0] * inv, acc[1] * inv);
  w2[1] = pack_bf16(acc[2] * inv, acc[3] * inv);
  *reinterpret_cast<u32x2*>(a.out + ((size_t)tok * a.Hq + h) * D + d4) = w2;
  if (a.lse != nullptr && d4 == 0)
    a.lse[(size_t)tok * a.Hq + h] = (mx + __builtin_log2f(L)) * 0.69314718055994531f;
}

}  // namespace

ct_status launch_attention(const ct_layer_cfg* cfg, const AttnPlan& p, const void* q_sel, const void* k_buf, const void* v_buf,
                           int32_t n_ctx, const int32_t* sel_idx, int32_t n_sel, void* out, float* lse,
                           void* workspace, hipStream_t s, int32_t key_after, int32_t key_upto, float* state) {
  if (n_sel == 0) return CT_OK;
  AttnArgs a;
  a.q = static_cast<const uint16_t*>(q_sel);
  a.k = static_cast<const uint16_t*>(k_buf);
  a.v = static_cast<const uint16_t*>(v_buf);
  a.sel_idx = sel_idx;
  a.out = static_cast<uint16_t*>(out);
  a.lse = lse;
  a.partial = static_cast<float*>(workspace);
  a.n_sel = n_sel;
  a.n_ctx = n_ctx;
  a.Hq = cfg->n_q_heads;
  a.Hkv = cfg->n_kv_heads;
  a.G = cfg->n_q_heads / cfg->n_kv_heads;
  a.TM = p.tile_tokens;
  a.cols = 256;
  a.tm_shift = 0;
  while ((1 << a.tm_shift) < a.TM) ++a.tm_shift;
  a.n_tiles = p.n_tiles;
  a.n_splits = p.n_splits;
  a.split_keys = p.split_keys;
  a.key_after = key_after;
  a.key_upto = key_upto;
  a.state = state;
  const float scale = cfg->softmax_scale > 0.f ? cfg->softmax_scale : 1.0f / sqrtf((float)cfg->head_dim);
  a.scale_log2 = scale * 1.4426950408889634f;

  const int D = cfg->head_dim;
  dim3 grid((unsigned)((size_t)p.n_tiles * cfg->n_kv_heads * p.n_splits));
  hipError_t e;
  if (D == 128)
    launch_kernel(KC_ATTN, attn_kernel<128>, grid, dim3(512), 0, s, a);
  else
    launch_kernel(KC_ATTN, attn_kernel<64>, grid, dim3(512), 0, s, a);
  e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, "attention kernel launch");
  if (p.n_splits > 1) {
    const int64_t threads = (int64_t)n_sel * cfg->n_q_heads * (D / 4);
    dim3 mgrid((unsigned)((threads + 255) / 256)), block(256);
    if (D == 128)
      launch_kernel(KC_MERGE, attn_merge_kernel<128>, mgrid, block, 0, s, a);
    else
      launch_kernel(KC_MERGE, attn_merge_kernel<64>, mgrid, block, 0, s, a);
    e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "attention merge kernel launch");
  }
  return CT_OK;
}

// Host-side replay of the key rows one launch reads (same item and row functions as the kernel, same
// tile loads: the prologue's K(0), K(1) and V(0), then K(i + 2) and V(i + 1) in period i < n_kt).
ct_status attention_rows_read(const ct_layer_cfg* cfg, const int32_t* sel_idx_host, int32_t n_sel, int32_t n_ctx,
                              int32_t key_after, int32_t key_upto, bool resumable, int32_t* first_row,
                              int32_t* last_row) {
  const AttnPlan p = plan_attention(cfg, n_ctx, n_sel);
  int lo = 0x7fffffff, hi = -1;
  for (int tile = 0; tile < p.n_tiles; ++tile) {
    const int last_tok = (tile * p.tile_tokens + p.tile_tokens < n_sel ? tile * p.tile_tokens + p.tile_tokens : n_sel) - 1;
    const int kmax = sel_idx_host[last_tok] + 1;
    for (int split = 0; split < p.n_splits; ++split) {
      const ItemRange it = item_range(kmax, split, p.split_keys, resumable, key_after, key_upto);
      if (!it.active) continue;
      const int n_kt = (it.k_hi - it.k_lo + BN - 1) / BN;
      for (int t = 0; t <= n_kt + 1; ++t)          // tiles 0 .. n_kt + 1 of the item are loaded
        for (int r = 0; r < BN; r += BN - 1) {     // first and last row of a tile bound the others
          const int row = tile_load_row(it.k_lo + t * BN, r, it.k_hi);
          lo = row < lo ? row : lo;
          hi = row > hi ? row : hi;
        }
    }
  }
  *first_row = hi < 0 ? -1 : lo;
  *last_row = hi;
  return CT_OK;
}

}  // namespace ct
