// Offline frequency-guided choice of the tokens to recompute (Sec. 4.1, Eq. 2-7).
//
// Scores.  The low-pass reconstruction of Eq. 2-4 is a forward FFT along the sequence, a mask
// and an inverse FFT, for every (head, dim) column of K and of V.  One workgroup takes a strip
// of 2*CP adjacent columns and all N tokens: two real columns ride as the real and imaginary
// part of one complex sequence (the mask is symmetric in +-frequency, so it commutes with that
// packing), which leaves CP complex sequences of length N.  They live in LDS for the whole
// transform, in place (see below).  After the inverse passes the squared magnitudes of a
// token's row are summed over the strip (Eq. 5 needs the norm over all heads and dims);
// a second small kernel adds the strips'
// partial sums in a fixed order, so the scores are reproducible bit for bit.
//
// Sequences longer than kFreqMaxTokens do not fit one workgroup's LDS: their transform is split as
// N = N1 N2 (token n = n1 N2 + n2, bin k = k1 + N1 k2) into length-N1 transforms over n1, a twiddle
// exp(-+2 pi i n2 k1 / N), and length-N2 transforms over n2, each done in LDS by the same passes,
// with one complex fp32 array of N x (row_elems / 2) per tensor in HBM between them:
//   A  (n2, strip):  x[n1 N2 + n2] -> FFT over n1 -> * twiddle -> Y[k1 N2 + n2]
//   B  (k1, strip):  Y[k1 N2 + .]  -> FFT over n2 -> mask bins k1 + N1 k2 -> inverse FFT over k2
//                    -> * conj twiddle -> Z[k1 N2 + n2]        (in place, contiguous rows)
//   C  (n2, strip):  Z[. N2 + n2]  -> inverse FFT over k1 -> squares summed per token.
//
// TopK (Eq. 7).  One workgroup per sequence: a 4 x 8-bit radix select over the order-preserving
// integer image of the scores finds the threshold value and how many of the tokens that tie with
// it still fit (lower index first); an ordered sweep then writes the chosen indices ascending.
#include <type_traits>

#include "ct_internal.h"

namespace ct {

// One workgroup of 1024 threads per compute unit (two of 512 with half the columns each read the rows in 16-byte
// pieces: 32 x 2048 x 1024 285 us against 205 with the kernel of then).
constexpr int kFreqThreads = 1024;
constexpr int kFreqMaxElems = 16384;   // complex values of a strip held in LDS (16 per thread)
constexpr int kFreqMaxTokens = 4096;

__device__ __forceinline__ float2 cmul(float2 a, float2 b) {
  return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
// a * conj(b)
__device__ __forceinline__ float2 cmul_conj(float2 a, float2 b) {
  return make_float2(a.x * b.x + a.y * b.y, a.y * b.x - a.x * b.y);
}
__device__ __forceinline__ float2 cadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 csub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
// a * (sgn * i)
__device__ __forceinline__ float2 mul_si(float2 a, float sgn) { return make_float2(-sgn * a.y, sgn * a.x); }

// exp(sgn * 2 pi i m / 16), m constant after unrolling
__device__ __forceinline__ float2 w16(int m, float sgn) {
  constexpr float c[16] = {1.f, 0.9238795325112867f, 0.7071067811865476f, 0.3826834323650898f, 0.f,
                           -0.3826834323650898f, -0.7071067811865476f, -0.9238795325112867f, -1.f,
                           -0.9238795325112867f, -0.7071067811865476f, -0.3826834323650898f, 0.f,
                           0.3826834323650898f, 0.7071067811865476f, 0.9238795325112867f};
  return make_float2(c[m & 15], sgn * c[(m + 12) & 15]);   // sin(x) = cos(x - pi/2)
}

// In-register DFTs of length R: v[k] <- sum_n v[n] exp(sgn 2 pi i n k / R).
template <int R>
__device__ __forceinline__ void dft(float2 (&v)[R], float sgn);

template <>
__device__ __forceinline__ void dft<2>(float2 (&v)[2], float) {
  const float2 a = v[0], b = v[1];
  v[0] = cadd(a, b);
  v[1] = csub(a, b);
}
template <>
__device__ __forceinline__ void dft<4>(float2 (&v)[4], float sgn) {
  const float2 t0 = cadd(v[0], v[2]), t1 = csub(v[0], v[2]);
  const float2 t2 = cadd(v[1], v[3]), t3 = mul_si(csub(v[1], v[3]), sgn);
  v[0] = cadd(t0, t2);
  v[2] = csub(t0, t2);
  v[1] = cadd(t1, t3);
  v[3] = csub(t1, t3);
}
template <>
__device__ __forceinline__ void dft<3>(float2 (&v)[3], float sgn) {
  const float2 s = cadd(v[1], v[2]), d = csub(v[1], v[2]);
  const float2 m = make_float2(v[0].x - 0.5f * s.x, v[0].y - 0.5f * s.y);
  const float2 q = mul_si(make_float2(0.8660254037844386f * d.x, 0.8660254037844386f * d.y), sgn);
  v[0] = cadd(v[0], s);
  v[1] = cadd(m, q);
  v[2] = csub(m, q);
}
template <>
__device__ __forceinline__ void dft<5>(float2 (&v)[5], float sgn) {
  // pairs (1,4) and (2,3): sums feed the cosines, differences the sines
  const float c1 = 0.30901699437494745f, c2 = -0.8090169943749473f;
  const float s1 = 0.9510565162951535f, s2 = 0.5877852522924731f;
  const float2 a1 = cadd(v[1], v[4]), b1 = csub(v[1], v[4]);
  const float2 a2 = cadd(v[2], v[3]), b2 = csub(v[2], v[3]);
  const float2 x0 = v[0];
  const float2 p1 = make_float2(x0.x + c1 * a1.x + c2 * a2.x, x0.y + c1 * a1.y + c2 * a2.y);
  const float2 p2 = make_float2(x0.x + c2 * a1.x + c1 * a2.x, x0.y + c2 * a1.y + c1 * a2.y);
  const float2 q1 = mul_si(make_float2(s1 * b1.x + s2 * b2.x, s1 * b1.y + s2 * b2.y), sgn);
  const float2 q2 = mul_si(make_float2(s2 * b1.x - s1 * b2.x, s2 * b1.y - s1 * b2.y), sgn);
  v[0] = cadd(x0, cadd(a1, a2));
  v[1] = cadd(p1, q1);
  v[4] = csub(p1, q1);
  v[2] = cadd(p2, q2);
  v[3] = csub(p2, q2);
}
// R = R1 * 4 by one Cooley-Tukey split: input n = 4 n1 + n2, output k = k1 + R1 k2.
template <int R1>
__device__ __forceinline__ void dft_by4(float2 (&v)[R1 * 4], float sgn) {
  constexpr int R = R1 * 4;
  float2 y[R1][4];
#pragma unroll
  for (int n2 = 0; n2 < 4; ++n2) {
    float2 col[R1];
#pragma unroll
    for (int n1 = 0; n1 < R1; ++n1) col[n1] = v[4 * n1 + n2];
    dft<R1>(col, sgn);
#pragma unroll
    for (int k1 = 0; k1 < R1; ++k1) y[k1][n2] = (n2 * k1 == 0) ? col[k1] : cmul(col[k1], w16(n2 * k1 * (16 / R), sgn));
  }
#pragma unroll
  for (int k1 = 0; k1 < R1; ++k1) {
    dft<4>(y[k1], sgn);
#pragma unroll
    for (int k2 = 0; k2 < 4; ++k2) v[k1 + R1 * k2] = y[k1][k2];
  }
}
template <>
__device__ __forceinline__ void dft<8>(float2 (&v)[8], float sgn) { dft_by4<2>(v, sgn); }
template <>
__device__ __forceinline__ void dft<16>(float2 (&v)[16], float sgn) { dft_by4<4>(v, sgn); }

// ---- power-of-two lengths 256 ... 4096: plan compiled in ----------------------------------------
// A forward transform by decimation in frequency leaves its bins in digit-reversed order, and an
// inverse by decimation in time takes them in that order, so nothing is ever reordered: every pass
// reads and writes the same places, each owned by one thread, and the last forward pass, the mask of
// Eq. 3 and the first inverse pass are one step in registers, as are the global load with the first
// pass and the squares with the last.
// N = 16 x 16 x MID (N = 256: 16 x 16), 16 elements per thread and pass, bin = k0 + 16 k1 + 256 k2 in row
// k0 N/16 + k1 MID + k2.  The N/16 rows of one k0 are what one wave owns in all passes but the first and the
// last, so only those two need a barrier.
// A thread's first twiddles do not depend on the strip: they are taken once from a table of rounded values and
// stay in 30 registers, the second ones in a small LDS table (rows of 17 against bank conflicts).
// The next strip's values are fetched into registers meanwhile, a quarter at a time: a wave that issues all 16 loads at once
// stands behind those of the others until most have arrived (32 x 2048 x 1024 with an earlier form of the passes 195 us against 161).
// No cache hint on the loads: with the streaming one, neighbouring strips find less of a shared line (the
// loads alone 122 us against 71).
// With all loads at once, the hint and a barrier per pass / now, 1024 columns of K and V: 32 sequences of 2048 212 / 150 us,
// 16 of 4096 315 / 182, 32 of 1024 84 / 69, 32 of 512 43 / 39; one sequence of 4096 20 / 20.  Without the loads the passes of 32 x 2048
// take 130 us and of 16 x 4096 138: bound by vector instructions and LDS accesses, which overlap in part.
// Not kept: all twiddles as (tan, cos) ahead of a butterfly, whose sums absorb the cosine.  Fewer instructions (1054 per
// wave and strip), but their sets take more LDS reads and a longer start: 32 x 2048 161 us, 16 x 4096 235, one sequence
// of 4096 25, only 32 x 512 and 32 x 1024 2 to 3 % less; and a quarter turn has no tangent, so that large bins overflow.

// a (1 + sgn i t), a + f b and a + sgn i f b
__device__ __forceinline__ float2 lean(float2 a, float t, float sgn) {
  return make_float2(fmaf(-sgn * t, a.y, a.x), fmaf(sgn * t, a.x, a.y));
}
__device__ __forceinline__ float2 axpy(float2 a, float f, float2 b) { return make_float2(fmaf(f, b.x, a.x), fmaf(f, b.y, a.y)); }
__device__ __forceinline__ float2 axpy_i(float2 a, float f, float2 b, float sgn) {
  return make_float2(fmaf(-sgn * f, b.y, a.x), fmaf(sgn * f, b.x, a.y));
}
// dft<4> of v[0], v[1] e^(sgn i x), v[2] e^(2 sgn i x) and v[3] e^(3 sgn i x), x = pi K / 8.  A rotation is taken as its tangent, two
// fused multiply-adds, and its cosine goes into the sums behind it (twiddles folded into fused multiply-adds: Linzer and
// Feig, "Implementation of efficient FFT algorithms on fused multiply-add architectures", IEEE Trans. Signal Process. 41, 1993).
template <int K>
__device__ __forceinline__ void dft4_by16(float2 (&v)[4], float sgn) {
  constexpr float h = 0.7071067811865476f, lo = 0.4142135623730950f, hi = 2.414213562373095f;     // cos pi/4, tan pi/8, tan 3 pi/8
  if constexpr (K == 0) {
    dft<4>(v, sgn);
  } else if constexpr (K == 2) {          // (its square is a quarter turn, which has no tangent)
    const float2 u1 = lean(v[1], 1.f, sgn), u3 = lean(v[3], -1.f, sgn);
    const float2 s0 = cadd(v[0], mul_si(v[2], sgn)), s1 = csub(v[0], mul_si(v[2], sgn));
    const float2 p = csub(u1, u3), q = cadd(u1, u3);
    v[0] = axpy(s0, h, p);
    v[2] = axpy(s0, -h, p);
    v[1] = axpy_i(s1, h, q, sgn);
    v[3] = axpy_i(s1, -h, q, sgn);
  } else {
    constexpr float c1 = K == 1 ? 0.9238795325112867f : 0.3826834323650898f, c2 = K == 1 ? h : -h;
    constexpr float t1 = K == 1 ? lo : hi, t2 = K == 1 ? 1.f : -1.f, t3 = K == 1 ? hi : lo, r = K == 1 ? lo : -hi;      // r = cos 3x / cos x
    const float2 u1 = lean(v[1], t1, sgn), u2 = lean(v[2], t2, sgn), u3 = lean(v[3], t3, sgn);
    const float2 s0 = axpy(v[0], c2, u2), s1 = axpy(v[0], -c2, u2);
    const float2 p = axpy(u1, r, u3), q = axpy(u1, -r, u3);
    v[0] = axpy(s0, c1, p);
    v[2] = axpy(s0, -c1, p);
    v[1] = axpy_i(s1, c1, q, sgn);
    v[3] = axpy_i(s1, -c1, q, sgn);
  }
}
// dft<16> that way; dft<R> otherwise.  OUTER (R = 4): of a forward transform (sgn < 0) results 0 and 3 alone, of an inverse one inputs 0 and 3.
template <int R, bool OUTER>
__device__ __forceinline__ void dft_fixed(float2 (&v)[R], float sgn) {
  if constexpr (R == 16) {
    float2 y[4][4];
#pragma unroll
    for (int n2 = 0; n2 < 4; ++n2) {
      float2 col[4] = {v[n2], v[4 + n2], v[8 + n2], v[12 + n2]};
      dft<4>(col, sgn);
#pragma unroll
      for (int k1 = 0; k1 < 4; ++k1) y[k1][n2] = col[k1];
    }
    dft4_by16<0>(y[0], sgn);
    dft4_by16<1>(y[1], sgn);
    dft4_by16<2>(y[2], sgn);
    dft4_by16<3>(y[3], sgn);
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = y[k & 3][k >> 2];
  } else if constexpr (OUTER) {
    static_assert(R == 4, "the other lengths gain nothing or spill");
    if (sgn < 0) {
      const float2 t2 = cadd(v[1], v[3]), t3 = mul_si(csub(v[1], v[3]), sgn), t1 = csub(v[0], v[2]);
      v[0] = cadd(cadd(v[0], v[2]), t2);
      v[3] = csub(t1, t3);
    } else {
      const float2 a = v[0], b = v[3], ib = mul_si(v[3], sgn);
      v[0] = cadd(a, b);
      v[1] = csub(a, ib);
      v[2] = csub(a, b);
      v[3] = cadd(a, ib);
    }
  } else {
    dft<R>(v, sgn);
  }
}

// x + (x of the lane that the DPP control names)
template <int CTRL>
__device__ __forceinline__ float add_dpp(float keep, float send) {
  return keep + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(send), CTRL, 0xf, 0xf, true));
}
// One step of a reduce-scatter over lane groups: e[0 .. 2 H) -> e[0 .. H); a lane of the upper half of
// its group keeps the upper half of the values.
template <int CTRL, int H>
__device__ __forceinline__ void halve(float* e, bool upper) {
#pragma unroll
  for (int i = 0; i < H; ++i) {
    const float keep = upper ? e[i + H] : e[i], send = upper ? e[i] : e[i + H];
    e[i] = add_dpp<CTRL>(keep, send);
  }
}
constexpr int kDppXor1 = 0xb1, kDppXor2 = 0x4e, kDppHalfMirror = 0x141, kDppMirror = 0x140;   // lanes i and i ^ 1, i ^ 2, 7 - i, 15 - i
// Sums of 16 values over the CP adjacent lanes of a group; lane `c` of the group ends up with the sums
// of values first .. first + max(1, 16 / CP) - 1 in e[0 ..].
template <int CP>
__device__ __forceinline__ int reduce_scatter16(float (&e)[16], int c) {
  int first = 0;
  if constexpr (CP >= 64) {
#pragma unroll
    for (int i = 0; i < 16; ++i) e[i] += __shfl_xor(e[i], 32);
  }
  if constexpr (CP >= 32) {
#pragma unroll
    for (int i = 0; i < 16; ++i) e[i] += __shfl_xor(e[i], 16);
  }
  if constexpr (CP >= 16) {
    halve<kDppMirror, 8>(e, c & 8);
    first += c & 8 ? 8 : 0;
    halve<kDppHalfMirror, 4>(e, c & 4);
    first += c & 4 ? 4 : 0;
    halve<kDppXor2, 2>(e, c & 2);
    first += c & 2 ? 2 : 0;
    halve<kDppXor1, 1>(e, c & 1);
    first += c & 1 ? 1 : 0;
  } else if constexpr (CP == 8) {
    halve<kDppHalfMirror, 8>(e, c & 4);
    halve<kDppXor2, 4>(e, c & 2);
    halve<kDppXor1, 2>(e, c & 1);
    first = (c & 4 ? 8 : 0) + (c & 2 ? 4 : 0) + (c & 1 ? 2 : 0);
  } else {
    static_assert(CP == 4, "sequences per strip");
    halve<kDppXor2, 8>(e, c & 2);
    halve<kDppXor1, 4>(e, c & 1);
    first = (c & 2 ? 8 : 0) + (c & 1 ? 4 : 0);
  }
  return first;
}

template <int N>
struct FixedPlan {
  static constexpr int CP = kFreqMaxElems / N;            // complex sequences per strip
  static constexpr int MID = N == 256 ? 16 : N / 256;
  static constexpr int M0 = N / 16;                       // distance of the elements of a first-pass butterfly
  static constexpr int M1 = MID;                          // and of a second-pass one
  // one spare row per 8 (16 when the middle pass owns 16 rows): the middle pass's accesses, MID rows
  // apart, then fall on distinct banks (N = 1024: with the order of rows that its lanes take)
  static constexpr int PAD = MID == 16 ? 4 : 3;
  static constexpr int ROWS = N + (N >> PAD);
  static constexpr __host__ __device__ int row(int n) { return n + (n >> PAD); }
  static constexpr size_t LDS_BYTES = ((size_t)ROWS * CP + (N == 256 ? 0 : MID * 17)) * sizeof(float2);
  static_assert(LDS_BYTES <= 160 * 1024, "LDS");
};

// partial[tensor * groups * n + g * n + token] = sum over strip g of |N x~|^2
template <int N>
__global__ __launch_bounds__(kFreqThreads) void freq_fixed_kernel(const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
                                                                  int64_t batch_stride, int32_t row_elems, int32_t n_work,
                                                                  int32_t groups, int32_t cutoff, float* __restrict__ partial) {
  using P = FixedPlan<N>;
  constexpr int CP = P::CP, MID = P::MID, M0 = P::M0, M1 = P::M1, T = kFreqThreads;
  extern __shared__ float2 data[];
  float2* const tab1 = data + P::ROWS * CP;      // [u % M1][j]
  const int tid = threadIdx.x, c = tid % CP, u = tid / CP;
  // first (and last) pass: rows u + j M0; second: rows k0 M0 + j M1 + u % M1; middle: rows k0 M0 + k1 MID + j; k0 = u / M1 is the wave
  const int k0 = u / M1;
  float2* const d0 = data + P::row(u) * CP + c;
  float2* const d1 = data + P::row(N == 256 ? 0 : k0 * M0 + u % M1) * CP + c;
  // twiddles exp(-2 pi i u j / N) and exp(-2 pi i (u % M1) j / M0), from a table that the strips then overwrite
  for (int t = tid; t < N; t += T) {
    float s, co;
    sincospif(-2.f * ((float)t / (float)N), &s, &co);
    data[t] = make_float2(co, s);
  }
  __syncthreads();
  float2 w0[16];
#pragma unroll
  for (int j = 1; j < 16; ++j) w0[j] = data[(u * j) % N];
  if (N > 256 && tid < M1 * 16) tab1[(tid >> 4) * 17 + (tid & 15)] = data[((tid >> 4) * (tid & 15) * 16) % N];
  __syncthreads();
  const float2* const w1 = tab1 + (u % M1) * 17;

  const int gone_first = cutoff, gone_last = cutoff == 0 ? N - 1 : N - cutoff;   // Eq. 3: these bins go
  const uint32_t gone = gone_last >= gone_first ? gone_last - gone_first + 1 : 0;
  // workgroups that share 128-byte lines of the rows (adjacent strips) are given ids that differ
  // by 8, which puts them on the same XCD (and its L2) at the same time.  An XCD that has whole tensors takes every
  // second line of one first and then the others, so that what it reads at a time comes through all channels of
  // its L2 (one column of lines for an XCD: 16 x 4096 x 1024 250 us against 237, 32 x 2048 166 against 161; with wider
  // strips the other way round, 32 x 1024 79 against 83).
  constexpr int per_line = CP >= 32 ? 1 : 32 / CP;
  const bool swizzled = n_work % (8 * per_line) == 0 && groups % per_line == 0 && gridDim.x % 8 == 0;
  const bool whole = CP <= 8 && n_work % (8 * groups) == 0 && groups % (2 * per_line) == 0;

  // strip number `it` of this launch -> tensor (batch * 2 + kv) and strip of it
  auto strip_of = [&](int it, int& strip) __attribute__((always_inline)) -> int {
    int w = it;
    if (swizzled) {
      const int xcd = w & 7, slot = w >> 3;
      if (whole) {
        const int t = slot / groups, r = slot % groups, line = r / per_line, half = groups / per_line / 2;
        w = (xcd * (n_work / 8 / groups) + t) * groups + (line < half ? 2 * line : 2 * (line - half) + 1) * per_line + r % per_line;
      } else {
        w = (slot / per_line) * (8 * per_line) + xcd * per_line + slot % per_line;
      }
    }
    const int tensor = w / groups;
    strip = w - tensor * groups;
    return tensor;
  };
  // a tensor is below 2 GiB here: offsets in 32 bits, a strip's first value as base
  const int lane_off = u * row_elems * 2 + 4 * c, step = M0 * row_elems * 2;
  uint32_t next[16];
  auto source = [&](int it) __attribute__((always_inline)) {
    int strip;
    const int tensor = strip_of(it, strip);
    const uint16_t* base = ((tensor & 1) ? v : k) + (int64_t)(tensor >> 1) * batch_stride + strip * (2 * CP);
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(base), 0, N * row_elems * 2 - strip * (4 * CP), 0x00020000);
  };
  auto fetch = [&](__amdgpu_buffer_rsrc_t src, int first, int last) __attribute__((always_inline)) {
#pragma unroll
    for (int j = first; j < last; ++j) next[j] = __builtin_amdgcn_raw_buffer_load_b32(src, lane_off, j * step, 0);
  };
  // rows that only this wave reads and writes: its LDS accesses run in order
  auto own_rows = [&]() __attribute__((always_inline)) {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
  // the last forward pass, the mask and the first inverse pass: MID neighbouring rows.  Up to half of the spectrum kept
  // (alpha <= 0.5), results 1 and 2 of a butterfly of four go whole and are neither computed nor transformed back (32 x 1024 x 1024 1 %).
  auto middle = [&](auto is_outer) __attribute__((always_inline)) {
    constexpr bool OUTER = decltype(is_outer)::value;
#pragma unroll
    for (int i = 0; i < 16 / MID; ++i) {
      const int k1 = N == 256 ? 0 : i * MID + (N == 1024 ? (u & 1) << 1 | (u >> 1 & 1) : u % MID);
      const int q = N == 256 ? u : k0 * 16 + k1;
      float2* const dm = data + P::row(q * MID) * CP + c;
      float2 y[MID];
#pragma unroll
      for (int j = 0; j < MID; ++j) y[j] = dm[P::row(j) * CP];
      dft_fixed<MID, OUTER>(y, -1.f);
      const int bin0 = N == 256 ? u : k0 + 16 * k1;
      constexpr int BSTEP = N == 256 ? 16 : 256;
#pragma unroll
      for (int j = 0; j < MID; ++j)
        if ((!OUTER || j == 0 || j == 3) && (uint32_t)(bin0 + BSTEP * j - gone_first) < gone) y[j] = make_float2(0.f, 0.f);
      dft_fixed<MID, OUTER>(y, 1.f);
#pragma unroll
      for (int j = 0; j < MID; ++j) dm[P::row(j) * CP] = y[j];
    }
  };
  fetch(source(blockIdx.x), 0, 16);
  for (int it = blockIdx.x; it < n_work; it += gridDim.x) {
    float2 x[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) x[j] = make_float2(bf16_lo(next[j]), bf16_hi(next[j]));
    const bool more = it + (int)gridDim.x < n_work;
    const __amdgpu_buffer_rsrc_t src = source(more ? it + gridDim.x : it);
    auto ahead = [&](int part) __attribute__((always_inline)) {
      if (more) fetch(src, 4 * part, 4 * part + 4);
    };
    ahead(0);
    dft_fixed<16, false>(x, -1.f);
#pragma unroll
    for (int j = 0; j < 16; ++j) d0[P::row(j * M0) * CP] = j == 0 ? x[0] : cmul(x[j], w0[j]);
    __syncthreads();
    ahead(1);
    if constexpr (N > 256) {
#pragma unroll
      for (int j = 0; j < 16; ++j) x[j] = d1[P::row(j * M1) * CP];
      dft_fixed<16, false>(x, -1.f);
#pragma unroll
      for (int j = 0; j < 16; ++j) d1[P::row(j * M1) * CP] = j == 0 ? x[0] : cmul(x[j], w1[j]);
      own_rows();
    }
    ahead(2);
    if (MID == 4 && cutoff <= N / 4) middle(std::integral_constant<bool, MID == 4>{});
    else middle(std::false_type{});
    if (N == 256) __syncthreads();
    ahead(3);
    if constexpr (N > 256) {
      own_rows();
#pragma unroll
      for (int j = 0; j < 16; ++j) x[j] = j == 0 ? d1[0] : cmul_conj(d1[P::row(j * M1) * CP], w1[j]);
      dft_fixed<16, false>(x, 1.f);
#pragma unroll
      for (int j = 0; j < 16; ++j) d1[P::row(j * M1) * CP] = x[j];
      __syncthreads();
    }
#pragma unroll
    for (int j = 0; j < 16; ++j) x[j] = j == 0 ? d0[0] : cmul_conj(d0[P::row(j * M0) * CP], w0[j]);
    dft_fixed<16, false>(x, 1.f);
    // Eq. 5: squares summed over the strip's sequences, which sit in CP adjacent lanes.  (The next strip's
    // first pass writes the places that this thread has just read: no barrier.)
    float e[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) e[j] = fmaf(x[j].x, x[j].x, x[j].y * x[j].y);
    const int first = reduce_scatter16<CP>(e, c);
    int strip;
    const int tensor = strip_of(it, strip);
    char* const out = reinterpret_cast<char*>(partial + ((int64_t)tensor * groups + strip) * N);
    if (CP <= 16 || c < 16) {
#pragma unroll
      for (int j = 0; j < (CP >= 16 ? 1 : 16 / CP); ++j)
        *reinterpret_cast<float*>(out + (uint32_t)(((first + j) * M0 + u) * sizeof(float))) = e[j];
    }
  }
}

// ---- other lengths: the same in-place transforms with the plan taken at run time -----------------
// N = R0 R1 R2 with radices up to 27, which reaches every 2^a 3^b 5^c up to 4096; bin = k0 + R0 k1 + R0 R1 k2
// in row (k0 R1 + k1) R2 + k2.  Blocks of R2 rows are `pitch` apart (one spare row when R2 is even and
// sequences are few), so that the middle pass's accesses fall on distinct banks.
struct MixPlan {
  int32_t n, lg_cp, r0, r1, r2, pitch;
  uint32_t mg1, mg2;       // floor(2^32 / r1) + 1 and the same of r2: quotients by multiplication
  int32_t cutoff;
  __host__ __device__ int rows() const { return r0 * r1 * pitch; }
  __host__ __device__ int tables() const { return 5 * (r1 * r2 + r2); }      // twiddles of the first two stages, powers 1, 2, 4, 8, 16
  size_t lds_bytes(int extra) const { return (((size_t)rows() << lg_cp) + tables() + extra) * sizeof(float2); }
};

// R = R1 R2 with coprime factors (Good-Thomas: index maps instead of twiddles): input
// n = (R2 n1 + R1 n2) mod R, output k with k = k1 mod R1 and k = k2 mod R2.
template <int R1, int R2>
__device__ __forceinline__ void dft_coprime(float2 (&v)[R1 * R2], float sgn) {
  constexpr int R = R1 * R2;
  float2 y[R1][R2];
#pragma unroll
  for (int n2 = 0; n2 < R2; ++n2) {
    float2 col[R1];
#pragma unroll
    for (int n1 = 0; n1 < R1; ++n1) col[n1] = v[(R2 * n1 + R1 * n2) % R];
    dft<R1>(col, sgn);
#pragma unroll
    for (int k1 = 0; k1 < R1; ++k1) y[k1][n2] = col[k1];
  }
  // with n = R2 n1 + R1 n2 the kernel is exp(i 2 pi (n1 k1 / R1 + n2 k2 / R2)), k1 = k mod R1, k2 = k mod R2
#pragma unroll
  for (int k1 = 0; k1 < R1; ++k1) dft<R2>(y[k1], sgn);
#pragma unroll
  for (int k = 0; k < R; ++k) v[k] = y[k % R1][k % R2];
}
template <> __device__ __forceinline__ void dft<6>(float2 (&v)[6], float sgn) { dft_coprime<2, 3>(v, sgn); }
template <> __device__ __forceinline__ void dft<10>(float2 (&v)[10], float sgn) { dft_coprime<2, 5>(v, sgn); }
template <> __device__ __forceinline__ void dft<12>(float2 (&v)[12], float sgn) { dft_coprime<4, 3>(v, sgn); }
template <> __device__ __forceinline__ void dft<15>(float2 (&v)[15], float sgn) { dft_coprime<3, 5>(v, sgn); }
// exp(2 pi i m / R), m constant after unrolling
template <int R>
__device__ __forceinline__ float2 root(int m, float sgn);
template <>
__device__ __forceinline__ float2 root<9>(int m, float sgn) {
  constexpr float co[9] = {1.f, 0.766044443f, 0.173648178f, -0.5f, -0.939692621f, -0.939692621f, -0.5f, 0.173648178f, 0.766044443f};
  constexpr float si[9] = {0.f, 0.64278761f, 0.984807753f, 0.866025404f, 0.342020143f, -0.342020143f, -0.866025404f, -0.984807753f,
      -0.64278761f};
  return make_float2(co[m], sgn * si[m]);
}
template <>
__device__ __forceinline__ float2 root<25>(int m, float sgn) {
  constexpr float co[25] = {1.f, 0.968583161f, 0.87630668f, 0.728968627f, 0.535826795f, 0.309016994f, 0.0627905195f, -0.187381315f,
      -0.425779292f, -0.63742399f, -0.809016994f, -0.929776486f, -0.992114701f, -0.992114701f, -0.929776486f,
      -0.809016994f, -0.63742399f, -0.425779292f, -0.187381315f, 0.0627905195f, 0.309016994f, 0.535826795f,
      0.728968627f, 0.87630668f, 0.968583161f};
  constexpr float si[25] = {0.f, 0.248689887f, 0.481753674f, 0.684547106f, 0.844327926f, 0.951056516f, 0.998026728f, 0.982287251f,
      0.904827052f, 0.770513243f, 0.587785252f, 0.368124553f, 0.125333234f, -0.125333234f, -0.368124553f,
      -0.587785252f, -0.770513243f, -0.904827052f, -0.982287251f, -0.998026728f, -0.951056516f, -0.844327926f,
      -0.684547106f, -0.481753674f, -0.248689887f};
  return make_float2(co[m], sgn * si[m]);
}
template <>
__device__ __forceinline__ float2 root<27>(int m, float sgn) {
  constexpr float co[27] = {1.f, 0.973044871f, 0.89363264f, 0.766044443f, 0.597158592f, 0.396079766f, 0.173648178f, -0.0581448289f,
      -0.286803233f, -0.5f, -0.686241638f, -0.835487811f, -0.939692621f, -0.993238358f, -0.993238358f,
      -0.939692621f, -0.835487811f, -0.686241638f, -0.5f, -0.286803233f, -0.0581448289f, 0.173648178f, 0.396079766f,
      0.597158592f, 0.766044443f, 0.89363264f, 0.973044871f};
  constexpr float si[27] = {0.f, 0.230615871f, 0.44879918f, 0.64278761f, 0.802123193f, 0.918216107f, 0.984807753f, 0.998308158f,
      0.957989512f, 0.866025404f, 0.727373642f, 0.549508978f, 0.342020143f, 0.116092914f, -0.116092914f,
      -0.342020143f, -0.549508978f, -0.727373642f, -0.866025404f, -0.957989512f, -0.998308158f, -0.984807753f,
      -0.918216107f, -0.802123193f, -0.64278761f, -0.44879918f, -0.230615871f};
  return make_float2(co[m], sgn * si[m]);
}
// R = R1 R2, input n = R2 n1 + n2, output k = k1 + R1 k2, twiddles exp(sgn 2 pi i n2 k1 / R)
template <int R1, int R2>
__device__ __forceinline__ void dft_split(float2 (&v)[R1 * R2], float sgn) {
  float2 y[R1][R2];
#pragma unroll
  for (int n2 = 0; n2 < R2; ++n2) {
    float2 col[R1];
#pragma unroll
    for (int n1 = 0; n1 < R1; ++n1) col[n1] = v[R2 * n1 + n2];
    dft<R1>(col, sgn);
#pragma unroll
    for (int k1 = 0; k1 < R1; ++k1) y[k1][n2] = n2 * k1 == 0 ? col[k1] : cmul(col[k1], root<R1 * R2>(n2 * k1, sgn));
  }
#pragma unroll
  for (int k1 = 0; k1 < R1; ++k1) {
    dft<R2>(y[k1], sgn);
#pragma unroll
    for (int k2 = 0; k2 < R2; ++k2) v[k1 + R1 * k2] = y[k1][k2];
  }
}
template <> __device__ __forceinline__ void dft<1>(float2 (&)[1], float) {}
template <> __device__ __forceinline__ void dft<9>(float2 (&v)[9], float sgn) { dft_split<3, 3>(v, sgn); }
template <> __device__ __forceinline__ void dft<18>(float2 (&v)[18], float sgn) { dft_coprime<2, 9>(v, sgn); }
template <> __device__ __forceinline__ void dft<25>(float2 (&v)[25], float sgn) { dft_split<5, 5>(v, sgn); }
template <> __device__ __forceinline__ void dft<27>(float2 (&v)[27], float sgn) { dft_split<3, 9>(v, sgn); }

template <int R> struct Radix { static constexpr int value = R; };
template <class F>
__device__ __forceinline__ void by_radix(int r, F&& f) {
  switch (r) {
    case 27: f(Radix<27>{}); break;
    case 25: f(Radix<25>{}); break;
    case 18: f(Radix<18>{}); break;
    case 16: f(Radix<16>{}); break;
    case 15: f(Radix<15>{}); break;
    case 12: f(Radix<12>{}); break;
    case 10: f(Radix<10>{}); break;
    case 9: f(Radix<9>{}); break;
    case 8: f(Radix<8>{}); break;
    case 6: f(Radix<6>{}); break;
    case 5: f(Radix<5>{}); break;
    case 4: f(Radix<4>{}); break;
    case 3: f(Radix<3>{}); break;
    case 2: f(Radix<2>{}); break;
    default: f(Radix<1>{}); break;
  }
}
// The thread's number, opaque: what a pass derives from it is computed there instead of being hoisted out of the
// loop over the strips, together for every radix of every pass (which overflows the registers).
__device__ __forceinline__ int pass_thread() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}
__device__ __forceinline__ int quotient(int x, int d, uint32_t magic) { return d == 1 ? x : (int)__umulhi((uint32_t)x, magic); }

// v[r] *= w^r (conjugated: SGN = -1), the powers 1, 2, 4, 8 and 16 of w from a table, `stride` apart, the others as
// products of at most five of those: a power taken by repeated products of w alone carries r times the rounding
// of w (scores of 4 x 1500 x 1024 were off by 4.4e-7 that way, 2-norm; so: 0.9e-7).
template <int R, int SGN>
__device__ __forceinline__ void times_powers(float2 (&v)[R], const float2* w, int stride) {
  auto base = [&](int k) __attribute__((always_inline)) {
    const float2 x = w[k * stride];
    return make_float2(x.x, SGN * x.y);
  };
  // pre[k]: product of the bits of r from bit k on
  float2 b[5], pre[5];
#pragma unroll
  for (int k = 0; k < 5; ++k)
    if ((1 << k) < R) b[k] = base(k);
#pragma unroll
  for (int r = 1; r < R; ++r) {
#pragma unroll
    for (int k = 4; k >= 0; --k) {
      if ((r & ((1 << k) - 1)) != 0 && k > 0) continue;     // pre[k] stands since r last was a multiple of 2^k
      const bool above = (r >> (k + 1)) != 0, bit = (r >> k) & 1;
      if (bit) pre[k] = above ? cmul(pre[k + 1], b[k]) : b[k];
      else if (above) pre[k] = pre[k + 1];
    }
    v[r] = cmul(v[r], pre[0]);
  }
}

// exp(-2 pi i u 2^k / n) for u < R1 R2 at tw[k R1 R2 + u], and behind them exp(-2 pi i u 2^k / (R1 R2)) for
// u < R2 at [k R2 + u], k < 5
__device__ __forceinline__ void mix_tables(float2* tw, const MixPlan& p, int threads) {
  const int m0 = p.r1 * p.r2;
  for (int t = threadIdx.x; t < 5 * (m0 + p.r2); t += threads) {
    const bool second = t >= 5 * m0;
    const int x = second ? t - 5 * m0 : t, m = second ? p.r2 : m0, len = second ? m0 : p.n;
    const int k = x / m, u = x - k * m;
    double s, c;
    sincospi(-2.0 * (double)((u << k) % len) / (double)len, &s, &c);
    tw[t] = make_float2((float)c, (float)s);
  }
}

// The passes.  A butterfly is (place, sequence c); `fn` bodies see registers only.
// First stage: rows u + i R1 R2 (i < R0), u = b1 R2 + r2, in LDS at ((i R1 + b1) pitch + r2).
template <int R, int T, class Load>
__device__ __forceinline__ void mix_first(float2* data, const float2* tw, const MixPlan& p, Load&& load) {
  const int m0 = p.r1 * p.r2, nb = m0 << p.lg_cp, step = (p.r1 * p.pitch) << p.lg_cp;
  constexpr int ITER = (kFreqMaxElems / kFreqThreads + R - 1) / R;   // 16 elements per thread at most
  const int tid = pass_thread();
#pragma unroll
  for (int it = 0; it < ITER; ++it) {
    const int b = tid + it * T;
    if (b < nb) {
      const int u = b >> p.lg_cp, c = b & ((1 << p.lg_cp) - 1);
      float2 v[R];
#pragma unroll
      for (int i = 0; i < R; ++i) v[i] = load(it * R + i, u + i * m0, c);
      dft<R>(v, -1.f);
      times_powers<R, 1>(v, tw + u, m0);
      const int b1 = quotient(u, p.r2, p.mg2);
      float2* d = data + ((b1 * p.pitch + u - b1 * p.r2) << p.lg_cp) + c;
#pragma unroll
      for (int i = 0; i < R; ++i) d[i * step] = v[i];
    }
  }
}
// Its inverse: `done(v, u, m0, c)` takes the results, v[i] being row u + i m0 of sequence c.
template <int R, int T, class Done>
__device__ __forceinline__ void mix_last(const float2* data, const float2* tw, const MixPlan& p, Done&& done) {
  const int m0 = p.r1 * p.r2, nb = m0 << p.lg_cp, step = (p.r1 * p.pitch) << p.lg_cp;
  for (int b = pass_thread(); b < nb; b += T) {
    const int u = b >> p.lg_cp, c = b & ((1 << p.lg_cp) - 1);
    const int b1 = quotient(u, p.r2, p.mg2);
    const float2* d = data + ((b1 * p.pitch + u - b1 * p.r2) << p.lg_cp) + c;
    float2 v[R];
#pragma unroll
    for (int i = 0; i < R; ++i) v[i] = d[i * step];
    times_powers<R, -1>(v, tw + u, m0);
    dft<R>(v, 1.f);
    done(v, u, m0, c);
  }
}
// Second stage and its inverse, in place: rows (a R1 + i) R2 + r2 (i < R1).
template <int R, int T, bool INV>
__device__ __forceinline__ void mix_second(float2* data, const float2* tw1, const MixPlan& p) {
  const int nb = (p.r0 * p.r2) << p.lg_cp, step = p.pitch << p.lg_cp;
  for (int b = pass_thread(); b < nb; b += T) {
    const int j = b >> p.lg_cp, c = b & ((1 << p.lg_cp) - 1);
    const int a = quotient(j, p.r2, p.mg2), r = j - a * p.r2;
    float2* d = data + ((a * R * p.pitch + r) << p.lg_cp) + c;
    float2 v[R];
#pragma unroll
    for (int i = 0; i < R; ++i) v[i] = d[i * step];
    if (INV) {
      times_powers<R, -1>(v, tw1 + r, p.r2);
      dft<R>(v, 1.f);
    } else {
      dft<R>(v, -1.f);
      times_powers<R, 1>(v, tw1 + r, p.r2);
    }
#pragma unroll
    for (int i = 0; i < R; ++i) d[i * step] = v[i];
  }
}
// Third stage: rows j R2 + i (i < R2), j = k0 R1 + k1, bins bin0 + i R0 R1 with bin0 = k0 + R0 k1.
// `mid(v, bin0, bin_step, c)` does what belongs between the two transforms, from and to registers;
// LOAD / STORE: the values come from, and go back to, LDS.
template <int R, int T, bool LOAD, bool STORE, class Mid>
__device__ __forceinline__ void mix_third(float2* data, const MixPlan& p, Mid&& mid) {
  const int nb = (p.r0 * p.r1) << p.lg_cp;
  for (int b = pass_thread(); b < nb; b += T) {
    const int j = b >> p.lg_cp, c = b & ((1 << p.lg_cp) - 1);
    const int k0 = quotient(j, p.r1, p.mg1), k1 = j - k0 * p.r1;
    float2* d = data + ((j * p.pitch) << p.lg_cp) + c;
    float2 v[R];
    if (LOAD) {
#pragma unroll
      for (int i = 0; i < R; ++i) v[i] = d[i << p.lg_cp];
      dft<R>(v, -1.f);
    }
    mid(v, k0 + p.r0 * k1, p.r0 * p.r1, c);
    if (STORE) {
      dft<R>(v, 1.f);
#pragma unroll
      for (int i = 0; i < R; ++i) d[i << p.lg_cp] = v[i];
    }
  }
}

// x + (x of the other lanes of its group of 2^lg adjacent lanes); every lane gets the sum
__device__ __forceinline__ float group_sum(float x, int lg) {
  if (lg > 0) x = add_dpp<kDppXor1>(x, x);
  if (lg > 1) x = add_dpp<kDppXor2>(x, x);
  if (lg > 2) x = add_dpp<kDppHalfMirror>(x, x);
  if (lg > 3) x = add_dpp<kDppMirror>(x, x);
  if (lg > 4) x += __shfl_xor(x, 16);
  if (lg > 5) x += __shfl_xor(x, 32);
  return x;
}
// Eq. 5 for the rows of a last-stage butterfly: squares summed over the strip's sequences, written (or added) once per row.
template <int R>
__device__ __forceinline__ void write_energy(const float2 (&v)[R], int lg, int c, float* out, int64_t step, bool add) {
  const int cmask = (1 << lg) - 1;
#pragma unroll
  for (int i = 0; i < R; ++i) {
    const float e = group_sum(fmaf(v[i].x, v[i].x, v[i].y * v[i].y), lg);
    if (c == (i & cmask)) out[i * step] = add ? out[i * step] + e : e;
  }
}

// Sequences that fit: as freq_fixed_kernel, a persistent workgroup per compute unit.  Bound by vector instructions
// and LDS accesses.  K and V, against sorting Stockham passes (one per radix up to 16, two barriers each):
// 4 x 1500 x 1024 75 -> 35 us, 4 x 3072 x 1024 158 -> 80 us, 4 x 4050 x 1000 303 -> 144 us; errors are smaller.
// (One token per sequence, which needs no transform, takes a microsecond longer: 8.3 -> 9.4 us with the finishing
// launch.)  The passes of all radices in one body hold more scalar values than there are registers: 111 of them
// here, 100 in freq_long_c_kernel, are kept in lanes of vector registers; none goes to memory.
__global__ __launch_bounds__(kFreqThreads) void freq_mixed_kernel(const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
                                                                  int64_t batch_stride, int32_t row_elems, int32_t n_work,
                                                                  int32_t groups, MixPlan p, float* __restrict__ partial) {
  constexpr int T = kFreqThreads;
  extern __shared__ float2 data[];
  float2* const tw = data + ((size_t)p.rows() << p.lg_cp);
  const float2* const tw1 = tw + 5 * p.r1 * p.r2;   // (no restrict: written by mix_tables below)
  mix_tables(tw, p, T);
  __syncthreads();
  const int cp = 1 << p.lg_cp, width = row_elems / 2, n = p.n;
  const int gone_first = p.cutoff, gone_last = p.cutoff == 0 ? n - 1 : n - p.cutoff;   // Eq. 3: these bins go
  const uint32_t gone = gone_last >= gone_first ? gone_last - gone_first + 1 : 0;
  const int per_line = cp >= 32 ? 1 : 32 / cp;      // strips that share 128-byte lines: see freq_fixed_kernel
  const bool swizzled = n_work % (8 * per_line) == 0 && groups % per_line == 0 && gridDim.x % 8 == 0;
  auto strip_of = [&](int it, int& strip) __attribute__((always_inline)) -> int {
    int w = it;
    if (swizzled) {
      const int xcd = w & 7, slot = w >> 3;
      w = (slot / per_line) * (8 * per_line) + xcd * per_line + slot % per_line;
    }
    const int tensor = w / groups;
    strip = w - tensor * groups;
    return tensor;
  };
  for (int it = blockIdx.x; it < n_work; it += gridDim.x) {
    int strip;
    const int tensor = strip_of(it, strip);
    const uint32_t* src = reinterpret_cast<const uint32_t*>(((tensor & 1) ? v : k) + (int64_t)(tensor >> 1) * batch_stride) + ((int64_t)strip << p.lg_cp);
    by_radix(p.r0, [&](auto r) __attribute__((always_inline)) {
      mix_first<decltype(r)::value, T>(data, tw, p, [&](int, int row, int c) __attribute__((always_inline)) {
        const uint32_t pair = src[(int64_t)row * width + c];
        return make_float2(bf16_lo(pair), bf16_hi(pair));
      });
    });
    __syncthreads();
    if (p.r1 > 1) {
      by_radix(p.r1, [&](auto r) __attribute__((always_inline)) { mix_second<decltype(r)::value, T, false>(data, tw1, p); });
      __syncthreads();
    }
    by_radix(p.r2, [&](auto r) __attribute__((always_inline)) {
      constexpr int R = decltype(r)::value;
      mix_third<R, T, true, true>(data, p, [&](float2 (&y)[R], int bin0, int step, int) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < R; ++i)
          if ((uint32_t)(bin0 + step * i - gone_first) < gone) y[i] = make_float2(0.f, 0.f);
      });
    });
    __syncthreads();
    if (p.r1 > 1) {
      by_radix(p.r1, [&](auto r) __attribute__((always_inline)) { mix_second<decltype(r)::value, T, true>(data, tw1, p); });
      __syncthreads();
    }
    float* out = partial + ((int64_t)tensor * groups + strip) * n;
    by_radix(p.r0, [&](auto r) __attribute__((always_inline)) {
      constexpr int R = decltype(r)::value;
      mix_last<R, T>(data, tw, p, [&](float2 (&y)[R], int u, int m0, int c) __attribute__((always_inline)) {
        write_energy<R>(y, p.lg_cp, c, out + u, m0, false);
      });
    });
    // (the next strip's first stage writes the places that this thread has just read: no barrier)
  }
}

// ---- sequences beyond kFreqMaxTokens: N = N1 N2 through HBM -----------------------------------
// Workgroups of 512 threads on 8192 complex values: two share a compute unit, so that one loads or
// stores while the other transforms.
// The array crosses HBM four times per tensor; with twiddles from one root per butterfly and a table of its steps
// (a 64-bit remainder and a root per value before) and the run-time plan above: K and V of 32768 x 1024
// 510 -> 370 us, 131072 x 256 494 -> 318 us, 6000 x 1024 147 -> 86 us.
constexpr int kFreqLongElems = 8192;
constexpr int kFreqLongThreads = 512;

// exp(sgn 2 pi i t / n), t < n < 2^24.  The angle is brought to within an eighth of a turn of a quarter in whole
// numbers first: what the rounded quotient is off by then counts little.
__device__ __forceinline__ float2 unit_root(int t, int n, float sgn) {
  const int q = (4 * t + n / 2) / n;               // nearest quarter turn, 0 ... 4
  const float turns2 = (float)(4 * t - q * n) * (0.5f / (float)n);   // half turns from there
  float s, c;
  sincospif(turns2, &s, &c);
  const float x = q & 1 ? -s : c, y = q & 1 ? c : s;
  return q & 2 ? make_float2(-x, -sgn * y) : make_float2(x, sgn * y);
}

// A: one workgroup = one n2 and one strip of 2^lg complex columns (pairs of real columns).
__global__ __launch_bounds__(kFreqLongThreads) void freq_long_a_kernel(const uint16_t* __restrict__ src, int32_t width,
                                                                       MixPlan p, int32_t n, int32_t n2_len,
                                                                       float2* __restrict__ scratch) {
  constexpr int T = kFreqLongThreads;
  extern __shared__ float2 data[];
  float2* const tw = data + ((size_t)p.rows() << p.lg_cp);
  float2* const steps = tw + p.tables();                 // exp(-2 pi i n2 R0 R1 i / n), i < R2
  const int strips = width >> p.lg_cp;
  const int strip = blockIdx.x % strips, n2 = blockIdx.x / strips;
  mix_tables(tw, p, T);
  if (threadIdx.x < p.r2) steps[threadIdx.x] = unit_root(n2 * p.r0 * p.r1 * (int)threadIdx.x, n, -1.f);
  __syncthreads();
  const uint32_t* base = reinterpret_cast<const uint32_t*>(src) + ((int64_t)strip << p.lg_cp) + (int64_t)n2 * width;
  by_radix(p.r0, [&](auto r) __attribute__((always_inline)) {
    mix_first<decltype(r)::value, T>(data, tw, p, [&](int, int row, int c) __attribute__((always_inline)) {
      const uint32_t pair = __builtin_nontemporal_load(base + (int64_t)row * n2_len * width + c);
      return make_float2(bf16_lo(pair), bf16_hi(pair));
    });
  });
  __syncthreads();
  if (p.r1 > 1) {
    by_radix(p.r1, [&](auto r) __attribute__((always_inline)) { mix_second<decltype(r)::value, T, false>(data, tw + 5 * p.r1 * p.r2, p); });
    __syncthreads();
  }
  float2* out = scratch + ((int64_t)strip << p.lg_cp) + (int64_t)n2 * width;
  by_radix(p.r2, [&](auto r) __attribute__((always_inline)) {
    constexpr int R = decltype(r)::value;
    mix_third<R, T, true, false>(data, p, [&](float2 (&y)[R], int bin0, int step, int c) __attribute__((always_inline)) {
      const float2 w = unit_root(n2 * bin0, n, -1.f);
#pragma unroll
      for (int i = 0; i < R; ++i) out[(int64_t)(bin0 + step * i) * n2_len * width + c] = cmul(cmul(y[i], w), steps[i]);
    });
  });
}

// B: one workgroup = one k1 and one strip; rows k1 N2 ... k1 N2 + N2 - 1 of the scratch array, in place.
__global__ __launch_bounds__(kFreqLongThreads) void freq_long_b_kernel(float2* __restrict__ scratch, int32_t width, MixPlan p,
                                                                       int32_t n, int32_t n1_len, int32_t cutoff) {
  constexpr int T = kFreqLongThreads;
  extern __shared__ float2 data[];
  float2* const tw = data + ((size_t)p.rows() << p.lg_cp);
  float2* const steps = tw + p.tables();                 // exp(2 pi i k1 R1 R2 i / n), i < R0
  const int strips = width >> p.lg_cp;
  const int strip = blockIdx.x % strips, k1 = blockIdx.x / strips;
  mix_tables(tw, p, T);
  if (threadIdx.x < p.r0) steps[threadIdx.x] = unit_root(k1 * p.r1 * p.r2 * (int)threadIdx.x, n, 1.f);
  __syncthreads();
  float2* rows = scratch + (int64_t)k1 * p.n * width + ((int64_t)strip << p.lg_cp);
  by_radix(p.r0, [&](auto r) __attribute__((always_inline)) {
    mix_first<decltype(r)::value, T>(data, tw, p, [&](int, int row, int c) __attribute__((always_inline)) {
      return rows[(int64_t)row * width + c];
    });
  });
  __syncthreads();
  if (p.r1 > 1) {
    by_radix(p.r1, [&](auto r) __attribute__((always_inline)) { mix_second<decltype(r)::value, T, false>(data, tw + 5 * p.r1 * p.r2, p); });
    __syncthreads();
  }
  by_radix(p.r2, [&](auto r) __attribute__((always_inline)) {
    constexpr int R = decltype(r)::value;
    // Eq. 3: bin k = k1 + N1 k2 goes when cutoff <= k <= N - cutoff
    mix_third<R, T, true, true>(data, p, [&](float2 (&y)[R], int bin0, int step, int) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < R; ++i) {
        const int bin = k1 + n1_len * (bin0 + step * i);
        if (bin >= cutoff && bin <= n - cutoff) y[i] = make_float2(0.f, 0.f);
      }
    });
  });
  __syncthreads();
  if (p.r1 > 1) {
    by_radix(p.r1, [&](auto r) __attribute__((always_inline)) { mix_second<decltype(r)::value, T, true>(data, tw + 5 * p.r1 * p.r2, p); });
    __syncthreads();
  }
  by_radix(p.r0, [&](auto r) __attribute__((always_inline)) {
    constexpr int R = decltype(r)::value;
    mix_last<R, T>(data, tw, p, [&](float2 (&y)[R], int u, int m0, int c) __attribute__((always_inline)) {
      const float2 w = unit_root(k1 * u, n, 1.f);
#pragma unroll
      for (int i = 0; i < R; ++i) rows[(int64_t)(u + i * m0) * width + c] = cmul(cmul(y[i], w), steps[i]);
    });
  });
}

// C: one workgroup = one n2 and `per` strips; partial[(strip / per) * n + token] = sum over the strips of |N x~|^2.
__global__ __launch_bounds__(kFreqLongThreads) void freq_long_c_kernel(const float2* __restrict__ scratch, int32_t width,
                                                                       MixPlan p, int32_t n, int32_t n2_len, int32_t per,
                                                                       float* __restrict__ partial) {
  constexpr int T = kFreqLongThreads;
  extern __shared__ float2 data[];
  float2* const tw = data + ((size_t)p.rows() << p.lg_cp);
  const int groups = (width >> p.lg_cp) / per;
  const int group = blockIdx.x % groups, n2 = blockIdx.x / groups;
  mix_tables(tw, p, T);
  float* out = partial + (int64_t)group * n + n2;
  for (int q = 0; q < per; ++q) {
    const float2* in = scratch + ((int64_t)(group * per + q) << p.lg_cp) + (int64_t)n2 * width;
    by_radix(p.r2, [&](auto r) __attribute__((always_inline)) {
      constexpr int R = decltype(r)::value;
      mix_third<R, T, false, true>(data, p, [&](float2 (&y)[R], int bin0, int step, int c) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < R; ++i) y[i] = in[(int64_t)(bin0 + step * i) * n2_len * width + c];
      });
    });
    __syncthreads();
    if (p.r1 > 1) {
      by_radix(p.r1, [&](auto r) __attribute__((always_inline)) { mix_second<decltype(r)::value, T, true>(data, tw + 5 * p.r1 * p.r2, p); });
      __syncthreads();
    }
    by_radix(p.r0, [&](auto r) __attribute__((always_inline)) {
      constexpr int R = decltype(r)::value;
      mix_last<R, T>(data, tw, p, [&](float2 (&y)[R], int u, int m0, int c) __attribute__((always_inline)) {
        // the same thread adds the next strip's squares
        write_energy<R>(y, p.lg_cp, c, out + (int64_t)u * n2_len, (int64_t)m0 * n2_len, q > 0);
      });
    });
    __syncthreads();
  }
}

// Eq. 5-6: s_i = (||K~_i|| + ||V~_i||) / 2.  64 tokens per workgroup; its four waves each add a quarter of
// the groups (group g by wave g mod 4), so that enough loads are in flight to read the partial sums at
// memory speed (32 x 2048 tokens, 64 groups: 7 us against 19 us with a thread per token), and the
// quarters are added in a fixed order.
__global__ __launch_bounds__(256) void freq_finish_kernel(const float* __restrict__ partial, int32_t n, int32_t groups,
                                                          float* __restrict__ scores) {
  __shared__ float part[2][4][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int blocks = (n + 63) / 64;                 // workgroups per sequence
  const int b = blockIdx.x / blocks, t = (blockIdx.x % blocks) * 64 + lane;
  float sk = 0.f, sv = 0.f;
  if (t < n) {
    const float* pk = partial + (int64_t)(b * 2) * groups * n + t;
    const float* pv = pk + (int64_t)groups * n;
#pragma unroll 8
    for (int g = wave; g < groups; g += 4) {
      sk += pk[(int64_t)g * n];
      sv += pv[(int64_t)g * n];
    }
  }
  part[0][wave][lane] = sk;
  part[1][wave][lane] = sv;
  __syncthreads();
  if (wave != 0 || t >= n) return;
  sk = (part[0][0][lane] + part[0][1][lane]) + (part[0][2][lane] + part[0][3][lane]);
  sv = (part[1][0][lane] + part[1][1][lane]) + (part[1][2][lane] + part[1][3][lane]);
  scores[(int64_t)b * n + t] = 0.5f * (sqrtf(sk) + sqrtf(sv)) / (float)n;
}

// ---- TopK ---------------------------------------------------------------------------------
__device__ __forceinline__ uint32_t score_key(float s) {
  uint32_t b = __float_as_uint(s);
  if (b == 0x80000000u) b = 0;                                   // -0 ties with +0
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);             // larger score <=> larger key
}

// One workgroup per sequence; scores stay in L2, so what counts is the chain of loads, atomics and barriers: loads
// go out kTopkBatch at a time, scores that share the first byte (nearly all do) are added by one lane, and each
// wave sweeps a stretch of its own without barriers.  15 % of 32768 scores: 92 -> 38 us, of 4 x 1500 8.4 -> 7.2 us.
// KEYS > 0: up to KEYS scores per thread, which stay in registers through all passes (wave w holds the stretch it sweeps): 15 % of 512
// scores 8.4 -> 6.6 us, of 300 x 1024 10.2 -> 7.6 us, of 4 x 1500 6.8 -> 5.0, of 16384 20.7 -> 14.0,
// of 32768 37 -> 25; beyond that there are not registers enough.
constexpr int kTopkBatch = 8;
template <int KEYS>
__global__ __launch_bounds__(1024) void topk_kernel(const float* __restrict__ scores, int32_t n_tokens, int32_t k,
                                                    int32_t* __restrict__ idx_out) {
  __shared__ uint32_t hist[256];
  __shared__ uint32_t sh_prefix, sh_need;
  __shared__ uint32_t n_above[16], n_tie[16];
  const float* s = scores + (int64_t)blockIdx.x * n_tokens;
  int32_t* out = idx_out + (int64_t)blockIdx.x * k;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const uint32_t n = n_tokens;     // (unsigned: positions run past the end by up to a batch)
  if (k <= 0) return;
  uint32_t own[KEYS > 0 ? KEYS : 1];
  // Wave w holds and sweeps a stretch of its own, equal ones: n of a launch lies in (512 KEYS, 1024 KEYS], so that the upper half of
  // the registers may go unused, the same ones in all waves.
  const uint32_t stretch = (n + 1023) / 1024 * 64, begin = wv * stretch, end = min(n, begin + stretch);
  auto used = [&](int b) __attribute__((always_inline)) { return KEYS <= 2 || b < KEYS / 2 || b * 64u < stretch; };
  const uint32_t own0 = KEYS > 0 ? begin + lane : 0;      // token of own[0], the others 64 apart
#pragma unroll
  for (int b = 0; b < KEYS; ++b)
    if (used(b)) own[b] = own0 + b * 64 < n ? score_key(s[own0 + b * 64]) : 0u;
  // n, opaque (and the threshold below): compared again in each pass instead of results being kept, two scalar registers per key
  auto count_of = [&]() __attribute__((always_inline)) {
    uint32_t m = n;
    if (KEYS > 1) asm volatile("" : "+s"(m));
    return m;
  };
  // radix select, most significant byte first: after the loop `prefix` is the key of the k-th
  // largest score and `need` the number of tokens with exactly that key that are still taken
  uint32_t prefix = 0, need = (uint32_t)k;
  for (int shift = 24; shift >= 0; shift -= 8) {
    if (tid < 256) hist[tid] = 0;
    __syncthreads();
    const uint32_t himask = shift == 24 ? 0u : (0xffffffffu << (shift + 8));
    // adds the keys of a wave's lanes that are `in` (all lanes come here) and agree with the prefix
    auto count = [&](uint32_t key, bool in) __attribute__((always_inline)) {
      const uint32_t bin = (key >> shift) & 255u;
      bool left = in && (key & himask) == prefix;
      if (shift == 24) {     // the first byte is the same for most: added by one lane for all that share it
        const uint64_t live = __ballot(left);
        if (live != 0) {
          const int first = __ffsll((unsigned long long)live) - 1;
          const bool same = left && bin == (uint32_t)__builtin_amdgcn_readlane((int)bin, first);
          const uint64_t who = __ballot(same);
          if (lane == first) atomicAdd(&hist[bin], (uint32_t)__popcll(who));
          left = left && !same;
        }
      }
      if (left) atomicAdd(&hist[bin], 1u);
    };
    if constexpr (KEYS > 0) {
      const uint32_t n = count_of();
      if (KEYS > 1 && shift == 24) {
        // one bin per wave is counted in a register: that of its first token
        const uint32_t common = (uint32_t)__builtin_amdgcn_readfirstlane((int)(own[0] >> 24));
        uint32_t same = 0;
#pragma unroll
        for (int b = 0; b < KEYS; ++b) {
          if (!used(b)) continue;
          const bool in = own0 + b * 64 < n;
          same += __popcll(__ballot(in && (own[b] >> 24) == common));
          if (in && (own[b] >> 24) != common) atomicAdd(&hist[own[b] >> 24], 1u);
        }
        if (lane == 0 && same > 0) atomicAdd(&hist[common], same);
      } else {
#pragma unroll
        for (int b = 0; b < KEYS; ++b)
          if (used(b)) count(own[b], own0 + b * 64 < n);
      }
    } else {
      for (uint32_t i0 = tid; i0 - tid < n; i0 += 1024 * kTopkBatch) {
        float x[kTopkBatch];
#pragma unroll
        for (int b = 0; b < kTopkBatch; ++b) x[b] = i0 + b * 1024 < n ? s[i0 + b * 1024] : 0.f;
#pragma unroll
        for (int b = 0; b < kTopkBatch; ++b) {
          if (i0 - tid + b * 1024 >= n) break;
          count(score_key(x[b]), i0 + b * 1024 < n);
        }
      }
    }
    __syncthreads();
    if (tid < 64) {
      // the first wave walks the histogram from the top: lane l owns bins 4l .. 4l+3; a suffix
      // scan over the lanes gives the count above each lane's bins, and the one lane whose bins
      // take the running count to `need` publishes the bin and what is left to take inside it
      const uint32_t h0 = hist[4 * tid], h1 = hist[4 * tid + 1], h2 = hist[4 * tid + 2], h3 = hist[4 * tid + 3];
      const uint32_t tot = h0 + h1 + h2 + h3;
      uint32_t incl = tot;
#pragma unroll
      for (int off = 1; off < 64; off <<= 1) {
        const uint32_t y = __shfl_down(incl, off, 64);
        if (tid + off < 64) incl += y;
      }
      uint32_t above = incl - tot;
      if (above < need && need <= above + tot) {
        int bin = 4 * tid + 3;
        uint32_t left = need - above;
        if (h3 < left) { left -= h3; bin = 4 * tid + 2;
          if (h2 < left) { left -= h2; bin = 4 * tid + 1;
            if (h1 < left) { left -= h1; bin = 4 * tid; } } }
        sh_prefix = prefix | ((uint32_t)bin << shift);
        sh_need = left;
      }
    }
    __syncthreads();
    prefix = sh_prefix;
    need = sh_need;
    __syncthreads();
  }
  // ordered sweep: tokens above the threshold, and the first `need` tokens on it.  A wave counts both kinds in its
  // stretch, and what the waves before it hold says where it writes.
  auto sweep = [&](auto&& body) __attribute__((always_inline)) {
    if constexpr (KEYS > 0) {
      const uint32_t n = count_of();
      uint32_t limit = prefix;
      if (KEYS > 1) asm volatile("" : "+v"(limit));
#pragma unroll
      for (int b = 0; b < KEYS; ++b) {
        if (!used(b)) continue;
        const uint32_t i = own0 + b * 64;
        body(i, i < n && own[b] > limit, i < n && own[b] == limit);
      }
      return;
    }
    for (uint32_t i0 = begin; i0 < end; i0 += 64 * kTopkBatch) {
      float x[kTopkBatch];
#pragma unroll
      for (int b = 0; b < kTopkBatch; ++b) x[b] = i0 + b * 64 + lane < end ? s[i0 + b * 64 + lane] : 0.f;
#pragma unroll
      for (int b = 0; b < kTopkBatch; ++b) {
        if (i0 + b * 64 >= end) break;
        const uint32_t i = i0 + b * 64 + lane;
        const uint32_t key = score_key(x[b]);
        body(i, i < end && key > prefix, i < end && key == prefix);
      }
    }
  };
  uint32_t above_here = 0, ties_here = 0;
  sweep([&](uint32_t, bool above, bool tie) __attribute__((always_inline)) {
    above_here += __popcll(__ballot(above));
    ties_here += __popcll(__ballot(tie));
  });
  if (lane == 0) {
    n_above[wv] = above_here;
    n_tie[wv] = ties_here;
  }
  __syncthreads();
  uint32_t ties = 0, at = 0;
  for (int q = 0; q < wv; ++q) {
    ties += n_tie[q];
    at += n_above[q];
  }
  at += min(ties, need);
  const uint64_t before = (1ull << lane) - 1ull;
  sweep([&](uint32_t i, bool above, bool tie) __attribute__((always_inline)) {
    const uint64_t tie_lanes = __ballot(tie);
    const bool take = above || (tie && ties + __popcll(tie_lanes & before) < need);
    const uint64_t take_lanes = __ballot(take);
    if (take) out[at + __popcll(take_lanes & before)] = (int32_t)i;
    ties += __popcll(tie_lanes);
    at += __popcll(take_lanes);
  });
}

// ---- host side ------------------------------------------------------------------------------
// Radices of a run-time plan: the split of n with the least estimated vector instructions for a strip of
// n << lg values (a wave's instructions for one butterfly: its sums and products, 8 per twiddle, LDS accesses
// and addresses).  It depends on the shape alone, so a sequence gets the same bits whatever it is batched with.
static bool make_mix_plan(int32_t n, int lg, int elems, size_t lds_cap, MixPlan* out) {
  static const int radix[15] = {1, 2, 3, 4, 5, 6, 8, 9, 10, 12, 15, 16, 18, 25, 27};
  static const int sums[15] = {0, 4, 14, 16, 36, 40, 60, 90, 92, 96, 160, 190, 200, 400, 400};
  double best = 0;
  bool found = false;
  if ((int64_t)n << lg > elems) return false;
  for (int a = 0; a < 15; ++a)
    for (int b = 0; b < 15; ++b) {
      const int r0 = radix[a], r1 = radix[b];
      if (n % (r0 * r1) != 0) continue;
      const int r2 = n / (r0 * r1);
      int c = 0;
      while (c < 15 && radix[c] != r2) ++c;
      if (c == 15) continue;
      MixPlan p = {};
      p.n = n;
      p.lg_cp = lg;
      p.r0 = r0;
      p.r1 = r1;
      p.r2 = r2;
      p.pitch = r2 > 1 && r2 % 2 == 0 && lg < 5 ? r2 + 1 : r2;
      if (p.lds_bytes(32) > lds_cap) p.pitch = r2;
      if (p.lds_bytes(32) > lds_cap) continue;
      p.mg1 = r1 > 1 ? (uint32_t)((1ull << 32) / r1 + 1) : 0;
      p.mg2 = r2 > 1 ? (uint32_t)((1ull << 32) / r2 + 1) : 0;
      auto waves = [&](int r) { return (double)((((int64_t)n << lg) / r + 255) / 256); };   // per SIMD, rounded up
      double cost = 2 * waves(r0) * (sums[a] + 11 * r0 + 30) + waves(r2) * (2 * sums[c] + 4 * r2 + 30) + 200;
      if (r1 > 1) cost += 2 * waves(r1) * (sums[b] + 12 * r1 + 30) + 400;
      if (!found || cost < best) {
        best = cost;
        *out = p;
        found = true;
      }
    }
  return found;
}

static int32_t cutoff_bins(int32_t n, double alpha) {
  const int bins = n / 2 + 1;
  int c = (int)floor(alpha * bins + 1e-9);
  if (c < 0) c = 0;
  if (c > bins) c = bins;
  return c;
}

// Long sequences: N = N1 N2 with N1 <= N2 <= kFreqMaxTokens, N1 the largest such divisor.
struct LongPlan {
  MixPlan p1, p2;
  int32_t width;        // complex columns per row = row_elems / 2
  int32_t per;          // strips that a workgroup of the last kernel adds up
  int32_t cutoff;
  size_t partial_bytes, scratch_bytes;
};
static bool make_long_plan(int32_t n, int32_t row_elems, double alpha, LongPlan* lp) {
  if (row_elems % 2 != 0 || n >= (1 << 24)) return false;
  int n1 = 0;
  for (int d = (int)floor(sqrt((double)n)); d >= 2; --d)
    if (n % d == 0) {
      if (n / d <= kFreqMaxTokens) n1 = d;
      break;                       // the largest divisor below the root; smaller ones have larger cofactors
    }
  if (n1 == 0) return false;
  *lp = LongPlan{};
  lp->width = row_elems / 2;
  const int len[2] = {n1, n / n1};
  for (int i = 0; i < 2; ++i) {
    int lg = 0;
    while (((int64_t)len[i] << (lg + 1)) <= kFreqLongElems && lp->width % (2 << lg) == 0) ++lg;
    if (i == 0) lp->per = lg > 6 ? 1 << (lg - 6) : 1;
    if (lg > 6) lg = 6;             // a token's squares are summed within a wave
    // (a second workgroup fits beside this one unless rows are very few and long)
    if (!make_mix_plan(len[i], lg, kFreqLongElems, 80 * 1024, i == 0 ? &lp->p1 : &lp->p2) &&
        !make_mix_plan(len[i], lg, kFreqLongElems, 160 * 1024, i == 0 ? &lp->p1 : &lp->p2))
      return false;
  }
  lp->cutoff = cutoff_bins(n, alpha);
  const size_t strips_c = ((size_t)lp->width >> lp->p1.lg_cp) / lp->per;
  lp->partial_bytes = strips_c * n * sizeof(float);                            // per tensor
  lp->scratch_bytes = ((size_t)n * lp->width * sizeof(float2) + 255) & ~(size_t)255;
  return true;
}
// Sequences that fit LDS: 2^lg complex columns per strip, one strip at a time per workgroup.
struct StripPlan {
  int lg, groups, cutoff;      // groups: strips per tensor
  MixPlan mix;
};
static bool make_plan(int32_t n, int32_t row_elems, double alpha, StripPlan* p) {
  int lg = 0;
  while ((2 << lg) <= 64 && (int64_t)n * (2 << lg) <= kFreqMaxElems && row_elems % (4 << lg) == 0) ++lg;
  if (row_elems % (2 << lg) != 0) return false;
  p->lg = lg;
  p->groups = row_elems / (2 << lg);
  p->cutoff = cutoff_bins(n, alpha);
  if (!make_mix_plan(n, lg, kFreqMaxElems, 160 * 1024, &p->mix)) return false;
  p->mix.cutoff = p->cutoff;
  return true;
}

}  // namespace ct

using namespace ct;

extern "C" {

size_t ct_frequency_workspace_bytes(int32_t n_batch, int32_t n_tokens, int32_t row_elems) {
  StripPlan p;
  if (n_batch <= 0 || n_tokens <= 0 || row_elems <= 0) return 0;
  if (n_tokens > kFreqMaxTokens) {
    LongPlan lp;
    if (!make_long_plan(n_tokens, row_elems, 0.5, &lp)) return 0;
    return (((size_t)n_batch * 2 * lp.partial_bytes + 255) & ~(size_t)255) + lp.scratch_bytes;
  }
  if (!make_plan(n_tokens, row_elems, 0.5, &p)) return 0;
  return (size_t)n_batch * 2 * p.groups * n_tokens * sizeof(float);
}

ct_status ct_frequency_scores(const void* k, const void* v, int32_t n_batch, int64_t batch_stride, int32_t n_tokens,
                              int32_t row_elems, double alpha, float* scores, void* workspace, size_t workspace_bytes,
                              void* stream) {
  if (n_batch < 0 || n_tokens < 0 || row_elems <= 0) return fail(CT_ERR_SHAPE, "negative size");
  if (n_batch == 0 || n_tokens == 0) return CT_OK;
  if (k == nullptr || v == nullptr || scores == nullptr) return fail(CT_ERR_NULL, "k, v and scores must be non-NULL");
  if (!(alpha >= 0.0 && alpha <= 1.0)) return fail(CT_ERR_RATIO, "alpha %g is outside [0, 1]", alpha);
  if (row_elems % 2 != 0) return fail(CT_ERR_SHAPE, "row_elems %d must be even", row_elems);
  if (n_batch > 1 && batch_stride < (int64_t)n_tokens * row_elems)
    return fail(CT_ERR_SHAPE, "batch_stride %lld is smaller than one sequence", (long long)batch_stride);
  hipStream_t s = (hipStream_t)stream;
  if (n_tokens > kFreqMaxTokens) {
    LongPlan lp;
    if (!make_long_plan(n_tokens, row_elems, alpha, &lp))
      return fail(CT_ERR_UNSUPPORTED,
                  "n_tokens %d: needs a divisor pair N1 N2 with both at most %d and no prime factor above 5, below 2^24",
                  n_tokens, kFreqMaxTokens);
    const size_t partial_all = ((size_t)n_batch * 2 * lp.partial_bytes + 255) & ~(size_t)255;
    const size_t need = partial_all + lp.scratch_bytes;
    if (workspace == nullptr || workspace_bytes < need)
      return fail(CT_ERR_WORKSPACE, "workspace of %zu bytes, %zu needed", workspace_bytes, need);
    if (((uintptr_t)workspace & 255) != 0) return fail(CT_ERR_WORKSPACE, "workspace is not 256-byte aligned");
    for (const void* fn : {(const void*)freq_long_a_kernel, (const void*)freq_long_b_kernel, (const void*)freq_long_c_kernel}) {
      hipError_t ea = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
      if (ea != hipSuccess) return hip_fail(ea, "hipFuncSetAttribute(long-sequence frequency kernels)");
    }
    float* partial = (float*)workspace;
    float2* scratch = (float2*)((char*)workspace + partial_all);
    const int n1 = lp.p1.n, n2 = lp.p2.n;
    const unsigned grid_ac = (unsigned)((size_t)n2 * (lp.width >> lp.p1.lg_cp));
    const unsigned grid_b = (unsigned)((size_t)n1 * (lp.width >> lp.p2.lg_cp));
    const int groups = (lp.width >> lp.p1.lg_cp) / lp.per;
    // one tensor at a time through the one scratch array (the launches of a stream run in order)
    for (int t = 0; t < n_batch * 2; ++t) {
      const uint16_t* src = (const uint16_t*)((t & 1) ? v : k) + (int64_t)(t >> 1) * batch_stride;
      launch_kernel(KC_FREQ, freq_long_a_kernel, dim3(grid_ac), dim3(kFreqLongThreads), (unsigned)lp.p1.lds_bytes(32), s, src,
                    lp.width, lp.p1, n_tokens, n2, scratch);
      launch_kernel(KC_FREQ, freq_long_b_kernel, dim3(grid_b), dim3(kFreqLongThreads), (unsigned)lp.p2.lds_bytes(32), s, scratch,
                    lp.width, lp.p2, n_tokens, n1, lp.cutoff);
      launch_kernel(KC_FREQ, freq_long_c_kernel, dim3((unsigned)n2 * groups), dim3(kFreqLongThreads), (unsigned)lp.p1.lds_bytes(32), s,
                    (const float2*)scratch, lp.width, lp.p1, n_tokens, n2, lp.per,
                    partial + (size_t)t * (lp.partial_bytes / sizeof(float)));
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "long-sequence frequency score launch");
    launch_kernel(KC_FREQ, freq_finish_kernel, dim3((unsigned)((int64_t)n_batch * ((n_tokens + 63) / 64))), dim3(256), 0, s,
                  (const float*)partial, n_tokens, groups, scores);
    e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "frequency score finish launch");
    return CT_OK;
  }
  StripPlan p;
  if (!make_plan(n_tokens, row_elems, alpha, &p))
    return fail(CT_ERR_UNSUPPORTED, "n_tokens %d has a prime factor above 5", n_tokens);
  const size_t need = (size_t)n_batch * 2 * p.groups * n_tokens * sizeof(float);
  if (workspace == nullptr || workspace_bytes < need)
    return fail(CT_ERR_WORKSPACE, "workspace of %zu bytes, %zu needed", workspace_bytes, need);
  const int n_work = n_batch * 2 * p.groups;
  const unsigned grid = n_work < kNumCUs ? n_work : kNumCUs;   // a workgroup fills a compute unit and goes on to further strips
  // power-of-two lengths from 256 on whose strips hold the full kFreqMaxElems values take the kernel
  // with the plan compiled in (it keeps offsets in 32 bits); everything else the one that reads the plan at run time
  using Kernel = void (*)(const uint16_t*, const uint16_t*, int64_t, int32_t, int32_t, int32_t, int32_t, float*);
  Kernel kern = nullptr;
  size_t lds = 0;
  if ((int64_t)n_tokens << p.lg == kFreqMaxElems && (int64_t)n_tokens * row_elems < (1 << 30)) {
    switch (n_tokens) {
      case 256: kern = freq_fixed_kernel<256>, lds = FixedPlan<256>::LDS_BYTES; break;
      case 512: kern = freq_fixed_kernel<512>, lds = FixedPlan<512>::LDS_BYTES; break;
      case 1024: kern = freq_fixed_kernel<1024>, lds = FixedPlan<1024>::LDS_BYTES; break;
      case 2048: kern = freq_fixed_kernel<2048>, lds = FixedPlan<2048>::LDS_BYTES; break;
      case 4096: kern = freq_fixed_kernel<4096>, lds = FixedPlan<4096>::LDS_BYTES; break;
      default: break;
    }
  }
  const void* fn = kern != nullptr ? (const void*)kern : (const void*)freq_mixed_kernel;
  hipError_t ea = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
  if (ea != hipSuccess) return hip_fail(ea, "hipFuncSetAttribute(frequency score kernel)");
  if (kern != nullptr)
    launch_kernel(KC_FREQ, kern, dim3(grid), dim3(kFreqThreads), (unsigned)lds, s, (const uint16_t*)k, (const uint16_t*)v,
                  batch_stride, row_elems, n_work, p.groups, p.cutoff, (float*)workspace);
  else
    launch_kernel(KC_FREQ, freq_mixed_kernel, dim3(grid), dim3(kFreqThreads), (unsigned)p.mix.lds_bytes(0), s,
                  (const uint16_t*)k, (const uint16_t*)v, batch_stride, row_elems, n_work, p.groups, p.mix, (float*)workspace);
  launch_kernel(KC_FREQ, freq_finish_kernel, dim3((unsigned)((int64_t)n_batch * ((n_tokens + 63) / 64))), dim3(256), 0, s,
                (const float*)workspace, n_tokens, p.groups, scores);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, "frequency score launch");
  return CT_OK;
}

ct_status ct_topk_indices(const float* scores, int32_t n_batch, int32_t n_tokens, int32_t k, int32_t* idx_out,
                          void* stream) {
  if (n_batch < 0 || n_tokens < 0 || k < 0) return fail(CT_ERR_SHAPE, "negative size");
  if (k > n_tokens) return fail(CT_ERR_SHAPE, "k %d exceeds n_tokens %d", k, n_tokens);
  if (n_batch == 0 || k == 0) return CT_OK;
  if (scores == nullptr || idx_out == nullptr) return fail(CT_ERR_NULL, "scores and idx_out must be non-NULL");
  hipStream_t s = (hipStream_t)stream;
  auto kern = n_tokens <= 1024 ? topk_kernel<1> : n_tokens <= 2048 ? topk_kernel<2> : n_tokens <= 4096 ? topk_kernel<4>
            : n_tokens <= 8192 ? topk_kernel<8> : n_tokens <= 16384 ? topk_kernel<16> : n_tokens <= 32768 ? topk_kernel<32> : topk_kernel<0>;
  launch_kernel(KC_TOPK, kern, dim3(n_batch), dim3(1024), 0, s, scores,
                n_tokens, k, idx_out);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, "topk launch");
  return CT_OK;
}

int32_t ct_frequency_n_selected(int32_t n_tokens, double ratio) {
  if (n_tokens <= 0 || !(ratio > 0.0)) return 0;
  if (ratio >= 1.0) return n_tokens;
  int64_t n = (int64_t)floor(ratio * (double)n_tokens + 1e-9);
  return (int32_t)(n < 1 ? 1 : n);
}

ct_status ct_select_frequency(const void* k, const void* v, int32_t n_batch, int64_t batch_stride, int32_t n_tokens,
                              int32_t row_elems, double alpha, double ratio, int32_t* idx_out, float* scores,
                              void* workspace, size_t workspace_bytes, void* stream) {
  if (!(ratio >= 0.0 && ratio <= 1.0)) return fail(CT_ERR_RATIO, "ratio %g is outside [0, 1]", ratio);
  ct_status st = ct_frequency_scores(k, v, n_batch, batch_stride, n_tokens, row_elems, alpha, scores, workspace,
                                     workspace_bytes, stream);
  if (st != CT_OK) return st;
  return ct_topk_indices(scores, n_batch, n_tokens, ct_frequency_n_selected(n_tokens, ratio), idx_out, stream);
}

}  // extern "C"
