// Bandwidth-bound steps of the partial-prefill layer: deferred RoPE recovery of reused keys
// (Eq. 8, delta form) and scatter fusion of recomputed K/V rows (Sec. 4.2).
//
// Both kernels move every byte exactly once with 128-bit accesses.  Key rows are
// [n_kv_heads, head_dim] bf16; a thread owns 8 rotation pairs of one token and walks over
// all KV heads, so the 8 sin/cos values (angle reduced in fp64) are computed once per
// token and pair and reused for every head.
#include "ct_internal.h"
#include "ct_rerope.h"

namespace ct {

namespace {

constexpr int kReropeThreads = 256;

// Per-token positions, or one arithmetic progression of deltas (delta0 + delta_step * t).
template <int D, int STYLE, int HEADS, bool NT_STORE>
__global__ __launch_bounds__(kReropeThreads) void rerope_kernel(
    const uint16_t* k_src, uint16_t* k_dst, const uint16_t* v_src, uint16_t* v_dst,
    const int32_t* __restrict__ old_pos, const int32_t* __restrict__ new_pos, int32_t delta0, int32_t delta_step,
    int32_t n_tokens, int32_t n_heads_rt, RopeTable table, const int32_t* __restrict__ skip_rows, int32_t n_skip) {
  constexpr int GROUPS = D / 16;  // threads per token: each owns 8 pairs = 16 elements per head
  const int64_t gid = (int64_t)blockIdx.x * kReropeThreads + threadIdx.x;
  const int64_t token = gid / GROUPS;
  const int jg = (int)(gid % GROUPS);
  bool listed = false;
  if (skip_rows != nullptr) {
    constexpr int WAVE_ROWS = 64 / GROUPS;
    const int32_t first = __builtin_amdgcn_readfirstlane((int32_t)token);
    const SkipWindow near = skip_window(skip_rows, n_skip, first, WAVE_ROWS);
    find_near(near, skip_rows, n_skip, (int32_t)token, WAVE_ROWS, &listed);
  }
  if (token >= n_tokens || listed) return;
  int32_t delta;
  if (new_pos != nullptr) {
    delta = new_pos[token] - (old_pos != nullptr ? old_pos[token] : 0);
  } else {
    delta = delta0 + delta_step * (int32_t)token;
  }
  const int64_t row = token * (int64_t)(HEADS > 0 ? HEADS : n_heads_rt) * D;
  rerope_token<D, STYLE, HEADS, NT_STORE>(k_src + row, k_dst + row, v_src ? v_src + row : nullptr,
                                v_dst ? v_dst + row : nullptr, delta, jg, n_heads_rt, table);
}

template <int D, int STYLE, int HEADS>
__global__ __launch_bounds__(kReropeThreads) void rerope_chunks_kernel(uint16_t* k_buf, uint16_t* v_buf,
                                                                      int32_t n_heads_rt, RopeTable table,
                                                                      ReropeChunks chunks) {
  rerope_chunk_tokens<D, STYLE, HEADS, true>(k_buf, v_buf, n_heads_rt, table, chunks, kReropeThreads, blockIdx.x, gridDim.x);
}

// The same work for chunks in pinned host memory, read over the host link by a few resident
// workgroups that stride over the tokens (Sec. 4.2: RoPE recovery overlapped with the transfer).
// What it is shaped by, measured on MI355X:
//  - a load from host memory takes microseconds, and while it is pending it holds a slot in the
//    memory pipeline of its compute unit and in the L2 channel's queue to the fabric; waves of
//    other kernels on the same compute unit, and L2 misses of any kernel in the same XCD, wait
//    behind it.  So a thread keeps only one head's two 16-byte loads in flight (about 128 KiB
//    over the whole grid already keeps the link at 45-50 GB/s; more only lengthens the queues);
//  - the launch asks for 80 KiB of (dynamic) LDS that the kernel does not use: they keep the
//    workgroups of the GEMM and attention kernels, which need 96-160 KiB, off the few compute units
//    this kernel sits on, where they would run at the speed of the host link.
constexpr int kStreamInThreads = 1024;
template <int D, int STYLE>
__global__ __launch_bounds__(kStreamInThreads) void stream_in_kernel(uint16_t* k_buf, uint16_t* v_buf, int32_t n_heads_rt,
                                                                    RopeTable table, ReropeChunks chunks) {
  rerope_chunk_tokens<D, STYLE, 0, false>(k_buf, v_buf, n_heads_rt, table, chunks, kStreamInThreads, blockIdx.x,
                                             gridDim.x);
}

// One 16-byte piece per thread and loop step; a selected row's K and V are `row_vec`
// pieces each.  Pieces of consecutive threads are consecutive in memory.
// The launch asks for kKeepOutLdsBytes of dynamic LDS that the kernel does not use (see there).
__global__ __launch_bounds__(1024) void scatter_kernel(u32x4* __restrict__ k_buf, u32x4* __restrict__ v_buf,
                                                      const u32x4* __restrict__ k_sel,
                                                      const u32x4* __restrict__ v_sel,
                                                      const int32_t* __restrict__ sel_idx, int32_t n_sel,
                                                      int32_t row_vec) {
  const int64_t total = (int64_t)n_sel * row_vec;
  for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < total; p += (int64_t)gridDim.x * blockDim.x) {
    const int64_t s = p / row_vec;
    const int c = (int)(p - s * row_vec);
    const int64_t dst = (int64_t)sel_idx[s] * row_vec + c;
    u32x4 kv = k_sel[p];
    u32x4 vv = v_sel[p];
    k_buf[dst] = kv;
    v_buf[dst] = vv;
  }
}

// Arguments of the per-token form, bundled for the dispatch over (head_dim, style, head count).
struct ReropeLaunch {
  const uint16_t* ks; uint16_t* kd; const uint16_t* vs; uint16_t* vd;
  const int32_t* old_pos; const int32_t* new_pos; int32_t delta0, delta_step, n_tokens;
  const int32_t* skip_rows; int32_t n_skip;
};

template <int D, int STYLE, int HEADS>
void launch_rerope_one(dim3 grid, hipStream_t s, const ReropeLaunch& r, int H, const RopeTable& t,
                       const ReropeChunks* chunks, bool big_blocks) {
  if (chunks != nullptr) {
    if (big_blocks)
      launch_kernel(KC_REROPE, stream_in_kernel<D, STYLE>, grid, dim3(kStreamInThreads), kStreamInLdsBytes, s, r.kd, r.vd,
                    H, t, *chunks);
    else
      launch_kernel(KC_REROPE, rerope_chunks_kernel<D, STYLE, HEADS>, grid, dim3(kReropeThreads), 0, s, r.kd, r.vd, H, t,
                    *chunks);
  } else {
    if (r.ks == r.kd)   // in place
      launch_kernel(KC_REROPE, rerope_kernel<D, STYLE, HEADS, true>, grid, dim3(kReropeThreads), 0, s, r.ks, r.kd, r.vs,
                    r.vd, r.old_pos, r.new_pos, r.delta0, r.delta_step, r.n_tokens, H, t, r.skip_rows, r.n_skip);
    else
      launch_kernel(KC_REROPE, rerope_kernel<D, STYLE, HEADS, false>, grid, dim3(kReropeThreads), 0, s, r.ks, r.kd, r.vs,
                    r.vd, r.old_pos, r.new_pos, r.delta0, r.delta_step, r.n_tokens, H, t, r.skip_rows, r.n_skip);
  }
}

template <int D, int STYLE>
void launch_rerope_heads(int H, dim3 grid, hipStream_t s, const ReropeLaunch& r, const RopeTable& t,
                         const ReropeChunks* chunks, bool big_blocks) {
  if (H == 8)
    launch_rerope_one<D, STYLE, 8>(grid, s, r, H, t, chunks, big_blocks);
  else if (H == 2)
    launch_rerope_one<D, STYLE, 2>(grid, s, r, H, t, chunks, big_blocks);
  else
    launch_rerope_one<D, STYLE, 0>(grid, s, r, H, t, chunks, big_blocks);
}

// The stream-in and scatter kernels are launched with more dynamic LDS than the default limit
// of a kernel: raise the limit once per kernel.
template <typename Kernel>
hipError_t allow_dynamic_lds(Kernel kernel, unsigned bytes) {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

ct_status launch_rerope_any(const ct_layer_cfg* cfg, const ReropeLaunch& r, int64_t n_tokens, const ReropeChunks* chunks,
                            int max_blocks, hipStream_t s) {
  if (n_tokens == 0) return CT_OK;
  RopeTable table;
  fill_rope_table(cfg, &table);
  const int D = cfg->head_dim, H = cfg->n_kv_heads;
  const int64_t threads = n_tokens * (D / 16);
  const bool big_blocks = chunks != nullptr && max_blocks > 0;   // sources in pinned host memory
  const int per_block = big_blocks ? kStreamInThreads : kReropeThreads;
  int64_t blocks = (threads + per_block - 1) / per_block;
  if (big_blocks && blocks > max_blocks) blocks = max_blocks;
  dim3 grid((unsigned)blocks);
  if (big_blocks) {
    static const hipError_t allowed = []() {
      hipError_t e = allow_dynamic_lds(stream_in_kernel<128, 0>, kStreamInLdsBytes);
      if (e == hipSuccess) e = allow_dynamic_lds(stream_in_kernel<128, 1>, kStreamInLdsBytes);
      if (e == hipSuccess) e = allow_dynamic_lds(stream_in_kernel<64, 0>, kStreamInLdsBytes);
      if (e == hipSuccess) e = allow_dynamic_lds(stream_in_kernel<64, 1>, kStreamInLdsBytes);
      return e;
    }();
    if (allowed != hipSuccess) return hip_fail(allowed, "hipFuncSetAttribute (stream-in kernel LDS)");
  }
  if (D == 128) {
    if (cfg->rope_style == 0)
      launch_rerope_heads<128, 0>(H, grid, s, r, table, chunks, big_blocks);
    else
      launch_rerope_heads<128, 1>(H, grid, s, r, table, chunks, big_blocks);
  } else {
    if (cfg->rope_style == 0)
      launch_rerope_heads<64, 0>(H, grid, s, r, table, chunks, big_blocks);
    else
      launch_rerope_heads<64, 1>(H, grid, s, r, table, chunks, big_blocks);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, "re-RoPE kernel launch");
  return CT_OK;
}

}  // namespace

ct_status launch_rerope(const ct_layer_cfg* cfg, const void* k_src, void* k_dst, const void* v_src, void* v_dst,
                        const int32_t* old_pos, const int32_t* new_pos, int32_t delta0, int32_t delta_step,
                        int32_t n_tokens, hipStream_t s, const int32_t* skip_rows, int32_t n_skip) {
  ReropeLaunch r = {static_cast<const uint16_t*>(k_src), static_cast<uint16_t*>(k_dst), static_cast<const uint16_t*>(v_src),
                    static_cast<uint16_t*>(v_dst), old_pos, new_pos, delta0, delta_step, n_tokens,
                    n_skip > 0 ? skip_rows : nullptr, n_skip};
  return launch_rerope_any(cfg, r, n_tokens, nullptr, 0, s);
}

ct_status launch_rerope_chunks(const ct_layer_cfg* cfg, void* k_buf, void* v_buf, const ReropeChunks* chunks,
                               int max_blocks, hipStream_t s) {
  ReropeLaunch r = {nullptr, static_cast<uint16_t*>(k_buf), nullptr, static_cast<uint16_t*>(v_buf), nullptr, nullptr, 0, 0, 0,
                    nullptr, 0};
  return launch_rerope_any(cfg, r, chunks->total_tokens, chunks, max_blocks, s);
}

ct_status launch_scatter(const ct_layer_cfg* cfg, void* k_buf, void* v_buf, const void* k_sel, const void* v_sel,
                         const int32_t* sel_idx, int32_t n_sel, hipStream_t s) {
  if (n_sel == 0) return CT_OK;
  static const hipError_t allowed = allow_dynamic_lds(scatter_kernel, kKeepOutLdsBytes);
  if (allowed != hipSuccess) return hip_fail(allowed, "hipFuncSetAttribute (scatter kernel LDS)");
  const int row_vec = cfg->n_kv_heads * cfg->head_dim / 8;  // 16-byte pieces per row
  const int64_t total = (int64_t)n_sel * row_vec;
  int64_t blocks = (total + 1023) / 1024;
  if (blocks > 2048) blocks = 2048;
  launch_kernel(KC_SCATTER, scatter_kernel, dim3((unsigned)blocks), dim3(1024), kKeepOutLdsBytes, s,
                static_cast<u32x4*>(k_buf), static_cast<u32x4*>(v_buf), static_cast<const u32x4*>(k_sel),
                static_cast<const u32x4*>(v_sel), sel_idx, n_sel, row_vec);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, "scatter kernel launch");
  return CT_OK;
}

}  // namespace ct
