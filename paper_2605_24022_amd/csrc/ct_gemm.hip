// The bf16 MFMA GEMM of the selected rows with fused epilogues:
//   - selective recompute of Q, K, V (Eq. 1) with RoPE at the rows' true positions
//     (Sec. 4.2, last paragraph);
//   - the other linear maps a transformer layer applies to the selected rows only
//     (Sec. 4.2: every layer after the check layer works on the selected tokens): output
//     projection and FFN down projection with the residual added, and the SwiGLU gate/up pair.
//
// The kernel computes the transposed product  C^T[f, t] = sum_e W[f, e] * X[row(t), e]
// (features in the MFMA M dimension, tokens in N) so that, in the 16x16 accumulator layout,
// a lane holds one token (column) and four consecutive features (rows) of every tile:
//   - both elements of every RoPE pair of a token sit in the same lane (no cross-lane
//     traffic in the epilogue), and the token's position is a per-lane scalar;
//   - results leave as 16-byte stores of eight consecutive bf16 features (odd and even rows of lanes swap halves of
//     two neighbouring tiles).
// Both operands are K-contiguous in memory (W is out-features major, X is token major).
// Tiles go from global memory straight into LDS (global_load_lds_dwordx4, no register
// staging): a wave-wide load fills 8 rows of 128 bytes, the 16-byte pieces of a row are
// XOR-swizzled so that the 128-bit fragment reads of 16 consecutive rows hit distinct banks.
//
// Workgroup: 512 threads = 8 waves, two to a SIMD; tile 256 features x 256 (or 128) tokens x 64 (K step),
// 16 x 16 x 32 MFMAs: a launch over the whole chip is limited by power, and an accumulator tile of 16 x 16 x 32 is read
// and written half as often per flop as one of 32 x 32 x 16 (linear 8192 x 8192 x 8192 802 -> 761 us with the old order of
// the loop; where few units work nothing changes).  Wave tiles are 64 x 64 on 128 tokens, 128 x 64 on 256 tokens.
// LDS holds three weight tiles and two (of 128 tokens: three) token tiles, and the loads of two K steps are in flight.
// On 256 tokens the slot of a step's token tile becomes free in the middle of the step, behind a barrier of its
// own, once all waves have its fragments in registers: with the token tile one step ahead instead (and no second
// barrier) 8192 x 8192 x 8192 and QKV of 4915 rows take 2 to 3 % longer.  Each barrier has MFMAs of the
// same wave ahead of it and behind it, so it passes while the matrix core is busy.  Fragment reads and tile loads
// go out one by one behind the MFMAs (in bursts ahead of each group of 16: 2 % longer as well).
// Before, with 32 x 32 x 16 MFMAs / now: QKV 1228 rows 57 / 53 us, 2458 rows 102 / 92, 4915 rows 200 / 183, 32768 rows
// 1235 / 1145; gate/up of 4915 rows 909 / 856; down projection of 4915 rows (K = 14336) 471 / 433.
// Not kept: on 128 tokens two wave groups that take one k-step each, with wave tiles of 128 x 64 and the halves added
// through LDS (a quarter fewer fragment reads; gate/up of 1228 rows 280 -> 288 us: reads from LDS are not the limit,
// at 128 tokens a step's tiles are 48 bytes per cycle and unit out of L2).
// Workgroups are numbered so that the ones resident on one XCD (ids congruent mod 8) cover a
// patch of neighbouring tiles and share their W and X tiles in that XCD's L2.
#include <string.h>

#include <type_traits>

#include "ct_internal.h"
#include "ct_rerope.h"

namespace ct {

namespace {

constexpr int kGemmThreads = 512;
constexpr int BF = 256;           // features per workgroup
// tokens per workgroup: 128 * NB (template parameter; 2 unless the grid would otherwise end in a mostly empty last
// round of workgroups)
constexpr int BK = 64;            // reduction elements per stage
constexpr int ROWB = BK * 2;      // LDS row in bytes (unpadded, swizzled)
constexpr int A_BYTES = BF * ROWB;
constexpr int A_SLOTS = 3;        // LDS slots of weight tiles
// LDS slots of token tiles of 128 * nb rows
constexpr int b_slots(int nb) { return nb == 1 ? 3 : 2; }
constexpr int gemm_lds_bytes(int nb) { return A_SLOTS * A_BYTES + b_slots(nb) * 128 * nb * ROWB; }

enum Epilogue { EPI_QKV_ROPE = 0, EPI_LINEAR = 1, EPI_SWIGLU = 2, EPI_PARTIAL = 3 };

struct GemmArgs {
  const uint16_t* hidden;        // B operand X [*, E], token major
  const int32_t* hidden_rows;    // optional row gather
  const uint16_t* wqkv;          // A operand W [O, E], feature major (SwiGLU: the gate matrix)
  const uint16_t* w_up;          // SwiGLU only: the up matrix [O, E]
  int32_t n_sel, E, O;           // tokens, reduction length, features (rows of W)
  int32_t nF, nT;                // tiles
  // this launch covers tiles v_begin .. v_begin + v_count - 1 (in the patch order below), each by
  // k_parts workgroups that take consecutive parts of the reduction (k_parts > 1: EPI_PARTIAL)
  int32_t v_begin, v_count, k_parts;
  float* partial;                // EPI_PARTIAL: fp32 [v_count * k_parts][256 tokens][256 features]
  // EPI_QKV_ROPE
  const int32_t* sel_pos;
  const int32_t* sel_idx;
  const uint16_t* bias;
  uint16_t* q_out;
  uint16_t* k_out;
  uint16_t* v_out;
  // optional: row of k_out / v_out that takes the keys and values of selected row t (the layer
  // buffers with kv_rows = sel_idx: the scatter of the recomputed rows done by the epilogue)
  const int32_t* kv_rows;
  int32_t Hq, Hkv;
  // EPI_LINEAR / EPI_SWIGLU: out[t, f] (+ residual[t, f]), row length O
  const uint16_t* residual;
  uint16_t* out;
};
typedef GemmArgs QkvArgs;

// Buffer rows -> new positions.  The walk over the chunks is the same for all lanes, so the table comes in scalar
// loads that do not wait for one another (a walk per lane, one dependent load per chunk and token, held every epilogue up).
template <int N>
__device__ __forceinline__ void rows_to_positions(const ChunkTable& tab, int32_t (&r)[N]) {
  int32_t shift[N];
#pragma unroll
  for (int n = 0; n < N; ++n) shift[n] = tab.new_start[0] - tab.row_start[0];
#pragma unroll 4
  for (int c = 1; c < tab.n; ++c) {
    const int32_t start = tab.row_start[c], by = tab.new_start[c] - start;
#pragma unroll
    for (int n = 0; n < N; ++n) shift[n] = r[n] >= start ? by : shift[n];
  }
#pragma unroll
  for (int n = 0; n < N; ++n) r[n] += shift[n];
}

// swizzle of the 16-byte pieces of LDS row r (rows are 128 bytes: two rows per 256-byte bank span)
__device__ __forceinline__ int swz(int r) { return (r >> 1) & 7; }

// Tile number -> (feature tile, token tile): tiles are numbered patch by patch (4 feature tiles x
// 8 token tiles), so that the workgroups resident on one XCD cover neighbouring tiles.
__device__ __forceinline__ void tile_of(int v, int nF, int nT, int* f_tile, int* t_tile) {
  constexpr int PF = 4, PT = 8;
  const int tp = v / (PT * nF);
  const int rem = v - tp * PT * nF;
  const int th = min(PT, nT - tp * PT);
  const int fp = rem / (PF * th);
  const int r2 = rem - fp * PF * th;
  const int fw = min(PF, nF - fp * PF);
  *f_tile = fp * PF + r2 % fw;
  *t_tile = tp * PT + r2 / fw;
}

// EPI_SWIGLU: 128 A rows are 64 gate rows followed by the 64 up rows of the same
// output features, and a wave owns both, so gate and up of one (feature, token) land in the same lane and register
// index of accumulator tiles 64 rows apart - the same pairing the half-split RoPE uses.
template <int EPI, int D, int STYLE, int NB>
__device__ __forceinline__ void gemm_workgroup(const GemmArgs& a, const RopeTable& rope, const ChunkTable& chunks,
                                               unsigned char* lds) {
  constexpr int NWAVES = kGemmThreads / 64;  // two per SIMD
  constexpr int A_LOADS = BF / 8 / NWAVES;   // wave-wide loads (8 rows each) per wave and stage
  constexpr int BT = 128 * NB;
  constexpr int WF = NB == 1 ? 4 : 2, WT = NWAVES / WF;   // waves along features and tokens
  constexpr int FM = BF / 16 / WF, TW = BT / 16 / WT;   // 16 x 16 MFMA tiles per wave
  // rows of a wave's feature tiles: 256 tokens 128 consecutive rows; 128 tokens 64 rows or,
  // where the epilogue pairs rows 64 apart (gate with up, halves of a 128-wide head), 32 and the 32 that go with them
  constexpr bool PAIR64 = EPI == EPI_SWIGLU || (EPI == EPI_QKV_ROPE && D == 128);
  constexpr int B_BYTES = BT * ROWB;
  constexpr int B_LOADS = BT / 8 / NWAVES;
  constexpr int B_SLOTS = b_slots(NB);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, h = lane >> 4;

  // ---- workgroup -> tile, XCD aware (consecutive ids go to different XCDs) ----------------
  const int items = a.v_count * a.k_parts;
  const int per_xcd = (items + kNumXCDs - 1) / kNumXCDs;
  const int item = (blockIdx.x % kNumXCDs) * per_xcd + blockIdx.x / kNumXCDs;
  if (item >= items) return;
  const int kp = item % a.k_parts;
  int f_tile, t_tile;
  tile_of(a.v_begin + item / a.k_parts, a.nF, a.nT, &f_tile, &t_tile);
  const int f_blk = f_tile * (EPI == EPI_SWIGLU ? BF / 2 : BF);   // first output feature
  const int t_blk = t_tile * BT;

  // ---- global -> LDS loads -------------------------------------------------------------------
  // load j of this wave fills LDS rows (NWAVES * j + wave) * 8 .. + 7 of the A (or B) tile; this
  // lane supplies physical piece lane % 8 of row lane / 8, i.e. logical piece (that ^ swizzle).
  // Byte offsets from the tensor bases fit 32 bits (the entry points check the extents of the
  // weights and of compact token matrices; gathered rows are the caller's contract); the K step advances
  // the scalar base, so the per-lane offsets are loop invariant.
  uint32_t a_off[A_LOADS], b_off[B_LOADS];
#pragma unroll
  for (int j = 0; j < A_LOADS; ++j) {
    const int row = (NWAVES * j + wave) * 8 + (lane >> 3);
    // SwiGLU: tile row -> (wave half, gate | up, feature within the wave's 64)
    const int frow = EPI == EPI_SWIGLU ? f_blk + (row >> 7) * 64 + (row & 63) : f_blk + row;
    const int f = min(frow, a.O - 1);
    a_off[j] = ((uint32_t)f * a.E + (((lane & 7) ^ swz(row)) * 8)) * 2;
  }
#pragma unroll
  for (int j = 0; j < B_LOADS; ++j) {
    const int row = (NWAVES * j + wave) * 8 + (lane >> 3);
    const int t = min(t_blk + row, a.n_sel - 1);
    const uint32_t xr = a.hidden_rows ? (uint32_t)a.hidden_rows[t] : (uint32_t)t;
    b_off[j] = (xr * a.E + (((lane & 7) ^ swz(row)) * 8)) * 2;
  }
  const int wf = wave % WF, wt = wave / WF;
  const int t0 = wt * 16 * TW + l16;      // the lane's first token of the tile (of TW, 16 apart)
  // what the rotation in the epilogue needs to know of the lane's tokens, fetched with the row indices
  [[maybe_unused]] int32_t pos[TW], kv_row[TW];
  if constexpr (EPI == EPI_QKV_ROPE) {
#pragma unroll
    for (int n = 0; n < TW; ++n) {
      const int t = min(t_blk + t0 + 16 * n, a.n_sel - 1);
      pos[n] = a.sel_pos ? a.sel_pos[t] : a.sel_idx[t];
      kv_row[n] = a.kv_rows ? a.kv_rows[t] : t;
    }
  }
  typedef __attribute__((address_space(3))) void* lds_ptr_t;
  const uint32_t lds_addr0 = (uint32_t)(uintptr_t)(lds_ptr_t)lds;
  auto dma16 = [&](const uint16_t* base, uint32_t byte_off, uint32_t lds_addr) __attribute__((always_inline)) {
    const uint32_t m0 = __builtin_amdgcn_readfirstlane(lds_addr);
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(m0), "v"(byte_off), "s"(base) : "memory", "m0");
  };
  // A (weight) tiles cycle through A_SLOTS LDS slots, B (token) tiles through B_SLOTS; j is one of a tile's loads.
  auto issue_a1 = [&](int k0, int slot, int j) __attribute__((always_inline)) {
    // scalar bases advanced to the K step; a wave-wide load covers 8 consecutive tile rows: all gate or all up
    const bool up = EPI == EPI_SWIGLU && ((((NWAVES * j + wave) * 8) >> 6) & 1);
    dma16((up ? a.w_up : a.wqkv) + k0, a_off[j], lds_addr0 + slot * A_BYTES + (NWAVES * j + wave) * 1024);
  };
  auto issue_b1 = [&](int k0, int slot, int j) __attribute__((always_inline)) {
    dma16(a.hidden + k0, b_off[j], lds_addr0 + A_SLOTS * A_BYTES + slot * B_BYTES + (NWAVES * j + wave) * 1024);
  };
  auto issue_a = [&](int k0, int slot) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < A_LOADS; ++j) issue_a1(k0, slot, j);
  };
  auto issue_b = [&](int k0, int slot) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < B_LOADS; ++j) issue_b1(k0, slot, j);
  };

  constexpr bool SPLIT = NB == 1 && PAIR64;
  const int row0 = NB == 2 ? wf * 128 : SPLIT ? (wf >> 1) * 128 + (wf & 1) * 32 : wf * 64;
  auto m_row = [](int m) __attribute__((always_inline)) { return SPLIT ? (m >> 1) * 64 + (m & 1) * 16 : m * 16; };
  // fragment read offsets inside a stage (bytes): row base + swizzled piece; the second k-step's piece is 4 further,
  // which is an exclusive-or on bits the row term leaves clear
  const int a_frag = (row0 + l16) * ROWB + ((h ^ swz(l16)) * 16);
  const int b_frag = (wt * 16 * TW + l16) * ROWB + ((h ^ swz(l16)) * 16);

  f32x4 acc[FM][TW];
#pragma unroll
  for (int m = 0; m < FM; ++m)
#pragma unroll
    for (int n = 0; n < TW; ++n) acc[m][n] = f32x4{0.f, 0.f, 0.f, 0.f};

  // Pipeline.  The tiles of K step kt + 2 are sent for while step kt is multiplied, so the loads of one step may stay in
  // flight at its end.  Past the end the last step is loaded again into the free slots, which keeps the number of
  // loads in flight, and the wait, uniform.
  // The workgroup barrier of a step sits ahead of its last MFMA group, not after it: a wave waits
  // for its loads of the next step, meets the others, and the first fragment reads of the
  // next step go out between the MFMAs of that group, so the barrier and the
  // LDS latency that follows it pass while the matrix core still has work.  (All waves of
  // a workgroup stand at the barrier together, so the other wave of the SIMD cannot cover it.)
  // this workgroup's part of the reduction: K steps kbeg .. kbeg + nk - 1
  const int nk_all = a.E / BK;
  const int kbeg = (int)((long)kp * nk_all / a.k_parts);
  const int nk = (int)((long)(kp + 1) * nk_all / a.k_parts) - kbeg;
  const int kbase = kbeg * BK;
  constexpr int AHEAD = A_LOADS + B_LOADS;                            // loads of a step that may stay in flight at its end
  constexpr int WAIT_STEP = AHEAD | 0x0f70;                           // s_waitcnt vmcnt(AHEAD)
  static_assert(AHEAD < 16, "vmcnt field");
  __builtin_amdgcn_s_waitcnt(0x0f70);   // ordinary loads so far (row indices) are complete
  const int k1 = kbase + min(1, nk - 1) * BK;
  issue_a(kbase, 0);
  issue_b(kbase, 0);
  issue_a(k1, 1);
  issue_b(k1, 1);
  if constexpr (EPI == EPI_QKV_ROPE) {
    if (a.sel_pos == nullptr) rows_to_positions(chunks, pos);   // while the first tiles are on their way
  }
  // Fragments: two register sets of four feature tiles each, two of the four token tiles.
  bf16x8 fa[2][4], fb[2][TW];
  auto read_a = [&](const unsigned char* a_base, int ks, int m, int set) __attribute__((always_inline)) {
    fa[set][m & 3] = *reinterpret_cast<const bf16x8*>(a_base + (a_frag ^ (ks << 6)) + m_row(m) * ROWB);
  };
  auto read_b = [&](const unsigned char* b_base, int ks, int n, int set) __attribute__((always_inline)) {
    fb[set][n] = *reinterpret_cast<const bf16x8*>(b_base + (b_frag ^ (ks << 6)) + n * 16 * ROWB);
  };
  // MFMA i of the 16 on feature tiles m0 .. m0 + 3 of k-step ks; these are in set `aset`, the token tiles in set ks
  auto mfma = [&](int aset, int ks, int m0, int i) __attribute__((always_inline)) {
    const int m = m0 + (i >> 2), n = i & 3;
    acc[m][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[aset][i >> 2], fb[ks][n], acc[m][n], 0, 0, 0);
  };
  const unsigned char* const b_lds = lds + A_SLOTS * A_BYTES;
  // vmcnt(AHEAD): this wave's loads of the step after this one have landed; lgkmcnt(0): its fragment reads of this step are done
  constexpr int WAIT_END = WAIT_STEP & ~0x0f00;
  __builtin_amdgcn_s_waitcnt(WAIT_STEP);   // this wave's loads of step 0 have landed
  __syncthreads();                         // everybody's have
  // (in the order of the loops: the compiler's count of reads in flight at a loop's start is then exact)
#pragma unroll
  for (int r = 0; r < 4; ++r) read_b(b_lds, 0, r, 0);
#pragma unroll
  for (int r = 0; r < 4; ++r) read_a(lds, 0, r, 0);
  if constexpr (NB == 2) {
    int sa = 0, sb = 0;
    for (int kt = 0; kt < nk; ++kt) {
      const int sa_free = sa == 0 ? A_SLOTS - 1 : sa - 1;   // slot of step kt - 1
      const int sa_next = sa == A_SLOTS - 1 ? 0 : sa + 1, sb_next = sb ^ 1;
      const unsigned char *a_base = lds + sa * A_BYTES, *a_next = lds + sa_next * A_BYTES;
      const unsigned char *b_base = b_lds + sb * B_BYTES, *b_next = b_lds + sb_next * B_BYTES;
      const int k2 = kbase + min(kt + 2, nk - 1) * BK;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        mfma(0, 0, 0, i);
        if (i < 4) read_a(a_base, 0, 4 + i, 1);
        else if (i < 8) read_b(b_base, 1, i - 4, 1);
        else if (i % 2 == 0) issue_a1(k2, sa_free, (i - 8) / 2);
        __builtin_amdgcn_sched_barrier(0);
      }
      __builtin_amdgcn_s_waitcnt(0xc07f);      // lgkmcnt(0): this wave has read all of the token tile
      __syncthreads();                         // everybody has: its slot is free for step kt + 2
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        mfma(1, 0, 4, i);
        if (i < 4) read_a(a_base, 1, i, 0);
        else if (i == 4 || i == 8) issue_b1(k2, sb, (i - 4) / 4);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        mfma(0, 1, 0, i);
        if (i < 4) read_a(a_base, 1, 4 + i, 1);
        else if (i == 4 || i == 8) issue_b1(k2, sb, 2 + (i - 4) / 4);
        __builtin_amdgcn_sched_barrier(0);
      }
      __builtin_amdgcn_s_waitcnt(WAIT_END);
      __syncthreads();                         // everybody's loads have landed; everybody is done reading step kt
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        mfma(1, 1, 4, i);
        if (i < 4) read_b(b_next, 0, i, 0);
        else if (i < 8) read_a(a_next, 0, i - 4, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
      sa = sa_next;
      sb = sb_next;
    }
  } else {
    // Few 128-token tiles leave units idle and the clock high: the MFMAs of a step, 1024 cycles of a SIMD's two waves, have to go out
    // one after the other.  So between two MFMAs of a wave stand at most one read or one load (three instructions), never
    // both; the scalars of the next step are worked out in its second half, where nothing waits for them (at the start
    // of a step, where all waves stand, the matrix cores waited with them).  QKV of 153 rows, K = 4096 40.3 -> 38.4 us,
    // gate/up of 300 rows of 4096 x 4096 39.8 -> 38.0; all loads behind the reads, or half of them a step earlier: no gain.
    uint32_t lds_a = lds_addr0 + 2 * A_BYTES + wave * 1024;      // where this wave's loads of step kt + 2 go
    uint32_t lds_b = lds_addr0 + A_SLOTS * A_BYTES + 2 * B_BYTES + wave * 1024;
    uint32_t at_a = 0, at_b = 0, next_a = A_BYTES, next_b = B_BYTES;     // slots of steps kt and kt + 1
    const int k2 = kbase + min(2, nk - 1) * BK;
    const uint16_t *from_a = a.wqkv + k2, *from_up = EPI == EPI_SWIGLU ? a.w_up + k2 : nullptr, *from_b = a.hidden + k2;
    static_assert(B_SLOTS == 3 && A_SLOTS == 3 && A_LOADS == 4 && B_LOADS == 2 && FM == 4, "the order of reads and loads below");
    auto load = [&](const uint16_t* base, uint32_t byte_off, uint32_t lds_addr, int j) __attribute__((always_inline)) {
      asm volatile("s_add_u32 m0, %0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                   : : "s"(lds_addr), "v"(byte_off), "s"(base), "i"(j * NWAVES * 1024) : "memory", "m0", "scc");
    };
    for (int kt = 0; kt < nk; ++kt) {
      const unsigned char *a_base = lds + at_a, *b_base = b_lds + at_b;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        mfma(0, 0, 0, i);
        constexpr int READ[16] = {0, -1, 1, -1, 2, 3, -1, 4, 5, -1, 6, 7, -1, -1, -1, -1};
        constexpr int LOAD[16] = {-1, 0, -1, 1, -1, -1, 2, -1, -1, 3, -1, -1, -1, 4, -1, 5};
        const int r = READ[i], j = LOAD[i];
        if (r >= 0 && r < 4) read_b(b_base, 1, r, 1);
        if (r >= 4) read_a(a_base, 1, r - 4, 1);
        if (j >= 0 && j < 2) load(from_b, b_off[j & 1], lds_b, j);
        if (j >= 2) load(EPI == EPI_SWIGLU && (j & 1) ? from_up : from_a, a_off[(j - 2) & 3], lds_a, j - 2);   // (load 1 and 3 of a tile: up rows)
        __builtin_amdgcn_sched_barrier(0);
      }
      __builtin_amdgcn_s_waitcnt(WAIT_END);
      __syncthreads();                         // everybody's loads have landed; everybody is done reading step kt
      const unsigned char *a_next = lds + next_a, *b_next = b_lds + next_b;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        mfma(1, 1, 0, i);
        if (i < 4) read_b(b_next, 0, i, 0);
        else if (i < 8) read_a(a_next, 0, i - 4, 0);
        if (i == 9) {      // the slots of this step are free; the asm statements keep these here
          lds_a = lds_addr0 + at_a + wave * 1024;
          lds_b = lds_addr0 + A_SLOTS * A_BYTES + at_b + wave * 1024;
          asm volatile("" : "+s"(lds_a), "+s"(lds_b));
        }
        if (i == 11) {
          at_a = next_a;
          at_b = next_b;
          next_a = next_a == 2 * A_BYTES ? 0 : next_a + A_BYTES;
          next_b = next_b == 2 * B_BYTES ? 0 : next_b + B_BYTES;
          asm volatile("" : "+s"(at_a), "+s"(at_b), "+s"(next_a), "+s"(next_b));
        }
        if (i == 13) {
          const int by = kt + 3 < nk ? BK : 0;
          from_a += by;
          from_b += by;
          if (EPI == EPI_SWIGLU) from_up += by;
          asm volatile("" : "+s"(from_a), "+s"(from_b), "+s"(from_up));
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  __builtin_amdgcn_s_waitcnt(0x0f70);   // the repeated loads of the last steps have landed before the LDS is released

  // ---- epilogues ---------------------------------------------------------------------------------
  // accumulator element i of tile (m, n): feature m_row(m) + 4 h + i, token l16 (h: the lane's row of 16 lanes).
  // The packed results of tiles m and m + 1 (features 0 .. 31 of a run of 32) are exchanged between odd and even rows of
  // lanes (v_permlane16_swap), which gives each lane eight features of its token from feature
  // 16 (h & 1) + 8 (h >> 1) of the run on: one 16-byte store for two tiles.  `p` points at the token's row at the run's
  // first feature.  Every lane of the wave must come here; `ok` gates the store alone.
  const int f8 = 16 * (h & 1) + 8 * (h >> 1);
  auto store_run = [&](uint16_t* p, const f32x4& x, const f32x4& y, bool ok) __attribute__((always_inline)) {
    const auto w0 = __builtin_amdgcn_permlane16_swap(pack_bf16(x[0], x[1]), pack_bf16(y[0], y[1]), false, false);
    const auto w1 = __builtin_amdgcn_permlane16_swap(pack_bf16(x[2], x[3]), pack_bf16(y[2], y[3]), false, false);
    const u32x4 out16 = {w0[0], w1[0], w0[1], w1[1]};
    if (ok) *reinterpret_cast<u32x4*>(p + f8) = out16;
  };
  if constexpr (EPI == EPI_PARTIAL) {
    // fp32 partial sums of this part of the reduction, token major inside the tile, 16-byte stores
    float* dst = a.partial + (size_t)item * (BT * BF);
#pragma unroll
    for (int n = 0; n < TW; ++n)
#pragma unroll
      for (int m = 0; m < FM; ++m)
        *reinterpret_cast<f32x4*>(dst + (size_t)(t0 + 16 * n) * BF + row0 + m_row(m) + 4 * h) = acc[m][n];
    return;
  } else if constexpr (EPI == EPI_LINEAR) {
    const int f0 = f_blk + row0;
    // Residuals arrive the same way, as 16-byte loads of the lane's eight features, and are swapped
    // back into the accumulator layout.  All residual values of the wave's tile are fetched before
    // the first result is stored: `out` may be the residual buffer itself, so the compiler cannot
    // move these loads above stores on its own, and with few loads in flight per lane the epilogue
    // is bound by memory latency.
    u32x4 res[TW][FM / 2];
    if (a.residual != nullptr) {
#pragma unroll
      for (int n = 0; n < TW; ++n) {
        const int t = min(t_blk + t0 + 16 * n, a.n_sel - 1);
#pragma unroll
        for (int m = 0; m < FM; m += 2) {
          const int fm = min(f0 + m_row(m), a.O - 32);
          res[n][m / 2] = *reinterpret_cast<const u32x4*>(a.residual + (size_t)t * a.O + fm + f8);
        }
      }
    }
#pragma unroll
    for (int n = 0; n < TW; ++n) {
      const int t = t_blk + t0 + 16 * n;
      const bool t_ok = t < a.n_sel;
#pragma unroll
      for (int m = 0; m < FM; m += 2) {
        const int fm = f0 + m_row(m);
        if (fm >= a.O) continue;            // uniform for the wave
        if (a.residual != nullptr) {
          const u32x4 r = res[n][m / 2];
          const auto d0 = __builtin_amdgcn_permlane16_swap(r[0], r[2], false, false);   // dword 0 of tiles m, m + 1
          const auto d1 = __builtin_amdgcn_permlane16_swap(r[1], r[3], false, false);   // dword 1
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            acc[m + e][n][0] += bf16_lo(d0[e]);
            acc[m + e][n][1] += bf16_hi(d0[e]);
            acc[m + e][n][2] += bf16_lo(d1[e]);
            acc[m + e][n][3] += bf16_hi(d1[e]);
          }
        }
        store_run(a.out + (size_t)(t_ok ? t : 0) * a.O + fm, acc[m][n], acc[m + 1][n], t_ok);
      }
    }
    return;
  } else if constexpr (EPI == EPI_SWIGLU) {
    const int f0 = f_blk + (row0 >> 7) * 64 + (row0 & 63);   // first output feature of this wave
#pragma unroll
    for (int n = 0; n < TW; ++n) {
      const int t = t_blk + t0 + 16 * n;
      const bool t_ok = t < a.n_sel;
#pragma unroll
      for (int m = 0; m < FM / 2; m += 2) {     // gate tile m, up tile m + FM / 2
        const int fm = f0 + m * 16;
        if (fm >= a.O) continue;             // uniform for the wave
        f32x4 y[2];
#pragma unroll
        for (int e = 0; e < 2; ++e)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float gate = acc[m + e][n][i], up = acc[m + e + FM / 2][n][i];
            y[e][i] = gate / (1.0f + __builtin_amdgcn_exp2f(-gate * 1.4426950408889634f)) * up;   // silu(gate) * up
          }
        store_run(a.out + (size_t)(t_ok ? t : 0) * a.O + fm, y[0], y[1], t_ok);
      }
    }
    return;
  } else {
    const int f0 = f_blk + row0;
    const int rope_end = (a.Hq + a.Hkv) * D;   // features below this are q or k heads
    const int q_end = a.Hq * D;
    constexpr int STEP = STYLE != 0 ? 0 : SPLIT ? 2 : D / 32;   // tile distance between the halves of a pair (j, j + D/2)
    // the lane's frequencies, ahead of the first store: loaded where they are used, they came in a chain of two loads per token
    constexpr int PAIRS = STYLE == 0 ? 4 : 2;                   // per tile of "a" halves, or of neighbouring pairs
    double turns[FM][PAIRS];
  #pragma unroll
    for (int m = 0; m < FM; ++m) {
      if (m & STEP) continue;
      const int j0 = (f0 + m_row(m)) % D + 4 * h;
  #pragma unroll
      for (int i = 0; i < PAIRS; ++i) turns[m][i] = rope.turns[STYLE == 0 ? j0 + i : (j0 >> 1) + i];
    }
  #pragma unroll
    for (int n = 0; n < TW; ++n) {
      const int t = t_blk + t0 + 16 * n;
      const bool t_ok = t < a.n_sel;
      const int tc = t_ok ? t : a.n_sel - 1;
      if (a.bias != nullptr) {
  #pragma unroll
        for (int m = 0; m < FM; ++m)
  #pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int f = min(f0 + m_row(m) + 4 * h + i, a.O - 1);
            acc[m][n][i] += bf16_lo((uint32_t)a.bias[f]);
          }
      }

      if (STYLE == 0) {
        // pairs (j, j + D/2), D/2 rows apart
  #pragma unroll
        for (int m = 0; m < FM; ++m) {
          if (m & STEP) continue;
          if (f0 + m_row(m) >= rope_end) continue;      // v heads are not rotated
  #pragma unroll
          for (int i = 0; i < 4; ++i) {
            float c, s;
            sincos_turns(pos[n], turns[m][i], c, s);
            const float x = acc[m][n][i], y = acc[m + STEP][n][i];
            acc[m][n][i] = x * c - y * s;
            acc[m + STEP][n][i] = x * s + y * c;
          }
        }
      } else {
  #pragma unroll
        for (int m = 0; m < FM; ++m) {
          if (f0 + m_row(m) >= rope_end) continue;
  #pragma unroll
          for (int i = 0; i < 4; i += 2) {
            float c, s;
            sincos_turns(pos[n], turns[m][i >> 1], c, s);
            const float x = acc[m][n][i], y = acc[m][n][i + 1];
            acc[m][n][i] = x * c - y * s;
            acc[m][n][i + 1] = x * s + y * c;
          }
        }
      }

  #pragma unroll
      for (int m = 0; m < FM; m += 2) {
        const int fm = f0 + m_row(m);
        if (fm >= a.O) continue;             // uniform for the wave
        uint16_t* dst;
        if (fm < q_end)
          dst = a.q_out + (size_t)tc * q_end + fm;
        else if (fm < rope_end)
          dst = a.k_out + (size_t)kv_row[n] * (a.Hkv * D) + (fm - q_end);
        else
          dst = a.v_out + (size_t)kv_row[n] * (a.Hkv * D) + (fm - rope_end);
        store_run(dst, acc[m][n], acc[m + 1][n], t_ok);
      }
    }
  }
}

template <int EPI, int D, int STYLE, int NB>
__global__ __launch_bounds__(kGemmThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void gemm_kernel(
    GemmArgs a, RopeTable rope, ChunkTable chunks) {
  __shared__ __align__(1024) unsigned char lds[gemm_lds_bytes(NB)];
  gemm_workgroup<EPI, D, STYLE, NB>(a, rope, chunks, lds);
}

// The projection with the rotation of the device-resident chunks in the same launch: workgroups from
// move_after on bring reused rows into the layer buffers.  The two touch different rows (the recompute set
// is what `move` skips) and different limits (matrix cores, memory), and the rotation runs on the compute units that
// the projection's last round leaves idle instead of in a launch of its own before it.  Few tokens per workgroup:
// with four times as many, fetched all heads at once, one waits for the last of them (8192 tokens, 1228 rows 208 -> 215 us).
template <int D, int STYLE, int NB>
__global__ __launch_bounds__(kGemmThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void qkv_move_kernel(
    GemmArgs a, RopeTable rope, ChunkTable chunks, ReropeChunks move, uint16_t* k_buf, uint16_t* v_buf, int32_t move_after) {
  __shared__ __align__(1024) unsigned char lds[gemm_lds_bytes(NB)];
  if ((int)blockIdx.x >= move_after) {
    const uint32_t block = blockIdx.x - move_after, blocks = gridDim.x - move_after;
    if (a.Hkv == 8) rerope_chunk_tokens<D, STYLE, 8, true>(k_buf, v_buf, 8, rope, move, kGemmThreads, block, blocks);
    else if (a.Hkv == 2) rerope_chunk_tokens<D, STYLE, 2, true>(k_buf, v_buf, 2, rope, move, kGemmThreads, block, blocks);
    else rerope_chunk_tokens<D, STYLE, 0, true>(k_buf, v_buf, a.Hkv, rope, move, kGemmThreads, block, blocks);
    return;
  }
  gemm_workgroup<EPI_QKV_ROPE, D, STYLE, NB>(a, rope, chunks, lds);
}

// Sum of the k_parts partial tiles of EPI_PARTIAL (+ residual), rounded to bf16 and written to
// out[t, f].  One thread per token and four consecutive features; a workgroup covers 4 tokens.
__global__ __launch_bounds__(256) void gemm_reduce_kernel(GemmArgs a) {
  const int tile_local = blockIdx.x >> 6;                 // 64 workgroups per 256 x 256 tile
  const int tl = ((blockIdx.x & 63) << 2) + (threadIdx.x >> 6);
  const int fl = (threadIdx.x & 63) << 2;
  int f_tile, t_tile;
  tile_of(a.v_begin + tile_local, a.nF, a.nT, &f_tile, &t_tile);
  const int t = t_tile * 256 + tl, f = f_tile * BF + fl;
  if (t >= a.n_sel || f >= a.O) return;
  const float* src = a.partial + ((size_t)tile_local * a.k_parts * 256 + tl) * BF + fl;
  f32x4 sum = *reinterpret_cast<const f32x4*>(src);
  for (int kp = 1; kp < a.k_parts; ++kp) {
    const f32x4 p = *reinterpret_cast<const f32x4*>(src + (size_t)kp * (256 * BF));
    sum += p;
  }
  const size_t o = (size_t)t * a.O + f;
  if (a.residual != nullptr) {
    const u32x2 r = *reinterpret_cast<const u32x2*>(a.residual + o);
    sum[0] += bf16_lo(r[0]); sum[1] += bf16_hi(r[0]); sum[2] += bf16_lo(r[1]); sum[3] += bf16_hi(r[1]);
  }
  u32x2 w;
  w[0] = pack_bf16(sum[0], sum[1]);
  w[1] = pack_bf16(sum[2], sum[3]);
  *reinterpret_cast<u32x2*>(a.out + o) = w;
}

}  // namespace

static void fill_tiles(GemmArgs* a, bool swiglu, int nb) {
  a->nF = (a->O + (swiglu ? BF / 2 : BF) - 1) / (swiglu ? BF / 2 : BF);
  a->nT = (a->n_sel + 128 * nb - 1) / (128 * nb);
  a->v_begin = 0;
  a->v_count = a->nF * a->nT;
  a->k_parts = 1;
}

// Token tile width for a launch: 256 tokens per workgroup unless the workgroups then fill the last
// round over the 256 compute units so badly that 128-token tiles (about 0.56 of the time of a
// 256-token tile each) finish earlier.  Measured, a full round of 128-token tiles against one of 256: linear with residual
// K = 512 0.59, 2048 and 4096 0.56, 14336 0.54, gate/up 0.54 to 0.56.  Whole launches at the chosen height / the other:
// QKV 4096 -> 6144 614 rows 41 / 70 us, 1228 56 / 77, 1638 85 / 94, 2458 97 / 106, 3276 152 / 170, 4915 189 / 207;
// gate/up 4096 -> 14336 819 rows 178 / 189, 1228 246 / 258, 1638 303 / 350, 4915 829 / 897.
static int pick_nb(const GemmArgs& a, bool swiglu) {
  GemmArgs t = a;
  double cost[3] = {0, 0, 0};
  for (int nb = 1; nb <= 2; ++nb) {
    fill_tiles(&t, swiglu, nb);
    const long wgs = (long)t.nF * t.nT;
    cost[nb] = (double)((wgs + kNumCUs - 1) / kNumCUs) * (nb == 2 ? 1.0 : 0.56);
  }
  return cost[1] < cost[2] ? 1 : 2;
}

template <typename Kernel>
static ct_status launch_gemm(Kernel kernel, const GemmArgs& a, const RopeTable& rope, const ChunkTable& tab,
                             KernelClass kc, hipStream_t s) {
  const int items = a.v_count * a.k_parts;
  const int per_xcd = (items + kNumXCDs - 1) / kNumXCDs;
  dim3 grid(per_xcd * kNumXCDs), block(kGemmThreads);
  launch_kernel(kc, kernel, grid, block, 0, s, a, rope, tab);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, "gemm kernel launch");
  return CT_OK;
}

template <int EPI, int D, int STYLE, int NB>
static ct_status launch_variant(const GemmArgs& a, const RopeTable& rope, const ChunkTable& tab, KernelClass kc,
                                hipStream_t s) {
  return launch_gemm(gemm_kernel<EPI, D, STYLE, NB>, a, rope, tab, kc, s);
}

template <int D, int STYLE, int NB>
static ct_status launch_qkv_variant(const GemmArgs& a, const RopeTable& rope, const ChunkTable& tab, const ReropeChunks* move,
                                    void* k_buf, void* v_buf, hipStream_t s) {
  if (move == nullptr) return launch_variant<EPI_QKV_ROPE, D, STYLE, NB>(a, rope, tab, KC_QKV, s);
  const int gemm_blocks = (a.v_count + kNumXCDs - 1) / kNumXCDs * kNumXCDs;
  const int64_t move_blocks = (move->total_tokens * (D / 16) + kGemmThreads - 1) / kGemmThreads;
  launch_kernel(KC_QKV, qkv_move_kernel<D, STYLE, NB>, dim3((unsigned)(gemm_blocks + move_blocks)), dim3(kGemmThreads), 0, s, a,
                rope, tab, *move, static_cast<uint16_t*>(k_buf), static_cast<uint16_t*>(v_buf), gemm_blocks);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, "projection kernel launch");
  return CT_OK;
}

// The rotation beside the projection costs it some of its memory bandwidth, which pays as long as idle compute
// units take most of the work.  Llama-3-8B layer, fused / in a launch of its own before: 2048 tokens,
// 307 rows 67 / 77 us, 8192 tokens, 983 rows 146 / 159, 32768 tokens, 1638 rows 518 / 538, 131072 tokens, 1310 rows 2133 / 2193;
// with 240 tiles on 256 units 200 / 199 (8192 tokens, 1228 rows) and 511 / 517 (16384 tokens, 2457 rows): within what runs differ by.
// A unit holds one such workgroup (it claims the LDS of a tile).  With the loads of eight heads in flight that still
// reads at speed, with two or with the loop over any number it does not, and what the idle units have not moved when the
// projection ends takes longer than in a launch of its own: at most 3 MB for each.  Fused / apart: 16/16 heads of 64,
// 32768 tokens, 9830 rows (6.1 MB) 1024 / 1021 us, 1638 rows (2.7 MB) 359 / 360, 327 rows (1.2 MB) 194 / 199; with inputs from memory
// (earlier forms of the kernels) 1093 / 1074, 381 / 384, 214 / 218, and 32/2 heads of 128, 131072 tokens, 1310 rows (4.6 MB) 1844 / 1812.
bool projection_leaves_units(const ct_layer_cfg* cfg, int32_t n_sel, int64_t move_tokens) {
  GemmArgs a;
  memset(&a, 0, sizeof(a));
  a.n_sel = n_sel;
  a.O = (cfg->n_q_heads + 2 * cfg->n_kv_heads) * cfg->head_dim;
  fill_tiles(&a, false, pick_nb(a, false));
  const int last = a.v_count % kNumCUs, idle = kNumCUs - last;
  if (last == 0 || idle < kNumCUs / 8) return false;
  const int64_t moved = move_tokens * cfg->n_kv_heads * cfg->head_dim * 2 * 4;   // keys and values, read and written
  return cfg->n_kv_heads == 8 || moved <= (int64_t)idle * 3000000;
}

ct_status launch_qkv(const ct_layer_cfg* cfg, const void* hidden, const int32_t* hidden_rows, const int32_t* sel_pos,
                     const int32_t* sel_idx, const ChunkTable* chunks, int32_t n_sel, const void* wqkv,
                     const void* bias, void* q_out, void* k_out, void* v_out, hipStream_t s,
                     const int32_t* kv_rows, const ReropeChunks* move, void* k_buf, void* v_buf) {
  if (n_sel == 0) return CT_OK;
  GemmArgs a;
  memset(&a, 0, sizeof(a));
  a.hidden = static_cast<const uint16_t*>(hidden);
  a.hidden_rows = hidden_rows;
  a.kv_rows = kv_rows;
  a.sel_pos = sel_pos;
  a.sel_idx = sel_idx;
  a.wqkv = static_cast<const uint16_t*>(wqkv);
  a.bias = static_cast<const uint16_t*>(bias);
  a.q_out = static_cast<uint16_t*>(q_out);
  a.k_out = static_cast<uint16_t*>(k_out);
  a.v_out = static_cast<uint16_t*>(v_out);
  a.n_sel = n_sel;
  a.E = cfg->hidden;
  a.Hq = cfg->n_q_heads;
  a.Hkv = cfg->n_kv_heads;
  a.O = (cfg->n_q_heads + 2 * cfg->n_kv_heads) * cfg->head_dim;
  const int nb = pick_nb(a, false);
  fill_tiles(&a, false, nb);
  RopeTable rope;
  fill_rope_table(cfg, &rope);
  ChunkTable tab;
  if (chunks != nullptr) {
    tab = *chunks;
  } else {
    tab.n = 1;
    tab.row_start[0] = 0;
    tab.row_start[1] = 0x7fffffff;
    tab.new_start[0] = 0;
  }
  auto launch = [&](auto d, auto style) -> ct_status {
    constexpr int D = decltype(d)::value, STYLE = decltype(style)::value;
    return nb == 2 ? launch_qkv_variant<D, STYLE, 2>(a, rope, tab, move, k_buf, v_buf, s)
                   : launch_qkv_variant<D, STYLE, 1>(a, rope, tab, move, k_buf, v_buf, s);
  };
  using C0 = std::integral_constant<int, 0>;
  using C1 = std::integral_constant<int, 1>;
  using C64 = std::integral_constant<int, 64>;
  using C128 = std::integral_constant<int, 128>;
  if (cfg->head_dim == 128) return cfg->rope_style == 0 ? launch(C128{}, C0{}) : launch(C128{}, C1{});
  return cfg->rope_style == 0 ? launch(C64{}, C0{}) : launch(C64{}, C1{});
}

// The last round of 256-token tiles of a linear launch, when it would leave most compute units
// idle, is run with the reduction of each tile split over several workgroups (fp32 partial tiles
// in `ws`, then a small kernel that adds them, and the residual, and rounds).  Returns the number
// of parts, or 1 when splitting is not worth it or `ws` is too small.
static int split_plan(const GemmArgs& a256, size_t ws_bytes, double cost_unsplit, int n_cu, int* full_tiles) {
  const int tiles = a256.nF * a256.nT;
  const int rem = tiles % n_cu;
  const int nk = a256.E / BK;
  *full_tiles = tiles - rem;
  if (rem == 0 || rem > n_cu / 2) return 1;
  int parts = n_cu / rem;
  if (parts > 8) parts = 8;
  if (parts > nk / 8) parts = nk / 8;
  if (parts < 2) return 1;
  if (ws_bytes < (size_t)rem * parts * 256 * BF * sizeof(float)) return 1;
  // in units of one round of 256-token tiles: the split round, plus the partial tiles' trip
  // through memory and the two extra launches (measured: 0.45 of a round for 256 partial tiles at
  // K = 4096, where a round takes 100 us; in proportion less for longer reductions).  4096 features with residual, split /
  // whole: K = 14336 153 rows 46 / 121 us, 614 85 / 121, 1228 125 / 141, 1638 167 / 157, 4915 434 / 503; K = 4096 153 rows
  // 27 / 39, 300 38 / 39, 614 43 / 40, 1638 67 / 51: chosen right but for 300 rows, 4 % behind
  const double cost = (double)(*full_tiles / n_cu) + 1.05 / parts + 0.45 * (64.0 / nk) * (rem * parts / 256.0);
  return cost < cost_unsplit ? parts : 1;
}

size_t linear_workspace_bytes(int32_t n_tok, int32_t k_len, int32_t n_out) {
  GemmArgs a;
  memset(&a, 0, sizeof(a));
  a.n_sel = n_tok;
  a.E = k_len;
  a.O = n_out;
  fill_tiles(&a, false, 2);
  // at most one partial tile per compute unit, whatever share of the chip the launch is planned for
  const int tiles = a.nF * a.nT;
  return (size_t)(tiles < kNumCUs ? tiles * 8 < kNumCUs ? tiles * 8 : kNumCUs : kNumCUs) * 256 * BF * sizeof(float);
}

ct_status launch_linear(const void* x, int32_t n_tok, int32_t k_len, const void* w, int32_t n_out, const void* residual,
                        void* out, void* ws, size_t ws_bytes, int n_cu, hipStream_t s) {
  if (n_tok == 0) return CT_OK;
  GemmArgs a;
  memset(&a, 0, sizeof(a));
  a.hidden = static_cast<const uint16_t*>(x);
  a.wqkv = static_cast<const uint16_t*>(w);
  a.residual = static_cast<const uint16_t*>(residual);
  a.out = static_cast<uint16_t*>(out);
  a.n_sel = n_tok;
  a.E = k_len;
  a.O = n_out;
  RopeTable rope;
  memset(&rope, 0, sizeof(rope));
  ChunkTable tab;
  memset(&tab, 0, sizeof(tab));
  const int nb = pick_nb(a, false);
  if (ws != nullptr) {
    GemmArgs t2 = a, t1 = a;
    fill_tiles(&t2, false, 2);
    fill_tiles(&t1, false, 1);
    if (n_cu <= 0 || n_cu > kNumCUs) n_cu = kNumCUs;
    const double c2 = (double)((t2.nF * t2.nT + n_cu - 1) / n_cu), c1 = 0.56 * (double)((t1.nF * t1.nT + n_cu - 1) / n_cu);
    int full = 0;
    const int parts = split_plan(t2, ws_bytes, c1 < c2 ? c1 : c2, n_cu, &full);
    if (parts > 1) {
      ct_status st = CT_OK;
      a = t2;
      if (full > 0) {
        a.v_count = full;
        if ((st = launch_variant<EPI_LINEAR, 128, 0, 2>(a, rope, tab, KC_LINEAR, s)) != CT_OK) return st;
      }
      a.v_begin = full;
      a.v_count = t2.nF * t2.nT - full;
      a.k_parts = parts;
      a.partial = static_cast<float*>(ws);
      if ((st = launch_variant<EPI_PARTIAL, 128, 0, 2>(a, rope, tab, KC_LINEAR, s)) != CT_OK) return st;
      launch_kernel(KC_LINEAR, gemm_reduce_kernel, dim3(a.v_count * 64), dim3(256), 0, s, a);
      hipError_t e = hipGetLastError();
      if (e != hipSuccess) return hip_fail(e, "gemm reduce launch");
      return CT_OK;
    }
  }
  fill_tiles(&a, false, nb);
  return nb == 2 ? launch_variant<EPI_LINEAR, 128, 0, 2>(a, rope, tab, KC_LINEAR, s)
                 : launch_variant<EPI_LINEAR, 128, 0, 1>(a, rope, tab, KC_LINEAR, s);
}

ct_status launch_swiglu(const void* x, int32_t n_tok, int32_t k_len, const void* w_gate, const void* w_up, int32_t n_out,
                        void* out, hipStream_t s) {
  if (n_tok == 0) return CT_OK;
  GemmArgs a;
  memset(&a, 0, sizeof(a));
  a.hidden = static_cast<const uint16_t*>(x);
  a.wqkv = static_cast<const uint16_t*>(w_gate);
  a.w_up = static_cast<const uint16_t*>(w_up);
  a.out = static_cast<uint16_t*>(out);
  a.n_sel = n_tok;
  a.E = k_len;
  a.O = n_out;
  const int nb = pick_nb(a, true);
  fill_tiles(&a, true, nb);
  RopeTable rope;
  memset(&rope, 0, sizeof(rope));
  ChunkTable tab;
  memset(&tab, 0, sizeof(tab));
  return nb == 2 ? launch_variant<EPI_SWIGLU, 128, 0, 2>(a, rope, tab, KC_LINEAR, s)
                 : launch_variant<EPI_SWIGLU, 128, 0, 1>(a, rope, tab, KC_LINEAR, s);
}

}  // namespace ct
