// The dense filter step on bfloat16 matrix instructions (gfx950): the product
// C = epilogue(A (D^{-1} R_Y)) of the residual filter (Algorithm 3, loop body)
// and of the plain one, with FP32 or BF16 operands.
//
// FP32 operands (P = 3 planes).  Every FP32 value is the exact sum of three
// bfloat16 values, x = x0 + x1 + x2 (x0: x truncated to 8 significant bits, x1:
// the rest rounded to 8, x2: what is left, at most 8 bits).  The product keeps
// the six terms x_i y_j with i + j <= 2, each exact in the FP32 accumulator's
// input; the three left out are below 2^-23 of |x y| each, have no common sign
// and vanish next to the accumulation's own FP32 rounding.  The matrix units do
// bfloat16 at sixteen times the FP32 rate, so six products cost 6/16 of one.
// BF16 operands (P = 1): the operator's bfloat16 copy and bfloat16(D^{-1} R_Y),
// both rounded to nearest even.
//
// A non-finite operand gives a non-finite result where it did before, but
// possibly NaN where an FP32 product gave an infinity.
//
// A complex Hermitian operator acts on planar columns (real parts, then
// imaginary parts) as [A_r | A_i] [[Z_r, Z_i], [-Z_i, Z_r]]: two k-segments of n
// rows (nseg = 2) whose right operands are Z with its halves swapped, one negated.
#include "internal.h"

#include <algorithm>

namespace chfsi {

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));   // any element alignment
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kSlice = 32;   // k values per packed slice

struct StepArgs {
  const void* A;             // packed operator (see k_pack_operator)
  const float* B;            // R_Y: n x N, ld ldb
  int64_t ldb;
  const float* ks;           // D^{-1} (n) or null
  unsigned short* Bp;        // packed right operand (see pack_offset)
  unsigned short* Bn;        // where the next step's goes (may be Bp: large path)
  float* partial;            // splits x (n x N)
  float* C;
  int64_t ldc;
  Epilogue<float> epi;
  int n, N, Np, half;        // Np: packed columns; half: N / 2 when nseg = 2
  int nseg, sps, slices;     // slices of a segment, and in all
  int splits, spc;           // split count, slices per split
  int tiles_m, tiles_n;
};

// dispatch is round-robin over the 8 XCDs: consecutive logical tiles on one XCD
__device__ __forceinline__ int xcd_tile(int h, int G) {
  const int xcd = h & 7, slot = h >> 3, full = G >> 3, rem = G & 7;
  return xcd < rem ? xcd * (full + 1) + slot : rem * (full + 1) + (xcd - rem) * full + slot;
}

__device__ __forceinline__ uint32_t pack_hi(float a, float b) {
  return __builtin_amdgcn_perm(__float_as_uint(b), __float_as_uint(a), 0x07060302u);
}
__device__ __forceinline__ uint32_t pack_rne(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2));
}
// two values to P bfloat16 planes
template <int P>
__device__ __forceinline__ void split2(float a, float b, uint32_t (&w)[P]) {
  if constexpr (P == 1) {
    w[0] = pack_rne(a, b);
  } else {
    w[0] = pack_hi(a, b);
    const float ra = a - __uint_as_float(__float_as_uint(a) & 0xffff0000u);
    const float rb = b - __uint_as_float(__float_as_uint(b) & 0xffff0000u);
    w[1] = pack_rne(ra, rb);
    w[2] = pack_hi(ra - __uint_as_float(w[1] << 16), rb - __uint_as_float(w[1] & 0xffff0000u));
  }
}
template <int P>
__device__ __forceinline__ void split8(f32x4 x, f32x4 y, bf16x8 (&f)[P]) {
  u32x4 v[P];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    uint32_t w[P];
    if (i < 2)
      split2<P>(x[2 * i], x[2 * i + 1], w);
    else
      split2<P>(y[2 * i - 4], y[2 * i - 3], w);
#pragma unroll
    for (int q = 0; q < P; ++q) v[q][i] = w[q];
  }
#pragma unroll
  for (int q = 0; q < P; ++q) f[q] = __builtin_bit_cast(bf16x8, v[q]);
}

// Packed right operand: per slice of 32 k values and plane, four chunks of 8 k
// values, each the chunk of every column side by side (16 bytes a column), so
// that a workgroup stages contiguous runs and the lanes of a fragment read
// consecutive 16-byte words of LDS.  Offset in elements of (slice, plane, chunk, column):
template <int P>
__device__ __forceinline__ int64_t pack_offset(int64_t slice, int q, int chunk, int64_t col,
                                               int64_t Np) {
  return (((slice * P + q) * 4 + chunk) * Np + col) * 8;
}

// 4 values (rows k, k + 1, .. of one column, k a multiple of 4) into the packed operand
template <int P>
__device__ __forceinline__ void pack4(const StepArgs& a, int k, int col, f32x4 v) {
  uint32_t w0[P], w1[P];
  split2<P>(v[0], v[1], w0);
  split2<P>(v[2], v[3], w1);
  const int slice = k / kSlice, kk = k % kSlice;
#pragma unroll
  for (int q = 0; q < P; ++q) {
    if (a.nseg == 1) {
      *reinterpret_cast<u32x2*>(a.Bn + pack_offset<P>(slice, q, kk / 8, col, a.Np) + (kk & 4)) =
          u32x2{w0[q], w1[q]};
    } else {
      // Z in the first segment; its real (imaginary) part as it is (negated) in
      // the imaginary (real) columns of the second
      const bool im = col >= a.half;
      const uint32_t neg = im ? 0x80008000u : 0u;
      *reinterpret_cast<u32x2*>(a.Bn + pack_offset<P>(slice, q, kk / 8, col, a.Np) + (kk & 4)) =
          u32x2{w0[q], w1[q]};
      *reinterpret_cast<u32x2*>(a.Bn +
                                pack_offset<P>(a.sps + slice, q, kk / 8,
                                               im ? col - a.half : col + a.half, a.Np) +
                                (kk & 4)) = u32x2{w0[q] ^ neg, w1[q] ^ neg};
    }
  }
}

// The operator in FP32 (T = float) or bfloat16 (rounded to FP32, then to nearest
// even), packed: per 32 rows and slice of 32 k values, the 16-byte words that a
// wave's lanes hold (lane l: row l % 32, k values of half l / 32 of the slice) one
// instruction after the other, so that each load of the products is 1 KB in one
// piece.  (Rows with a power-of-two stride, read 128 bytes each, all fall on one
// channel of the L2: 8192 x 320 in FP32 took
// 253 us a step that way, 239 so.)
// Rows and k values past n are zeros.
template <typename T>
__global__ __launch_bounds__(256) void k_pack_operator(const double* __restrict__ A, int64_t lda,
                                                       int n, int sps, int slices, int cplx,
                                                       u32x4* __restrict__ out, int64_t total) {
  constexpr int W = 16 / sizeof(T), AV = 8 / W;
  for (int64_t idx = blockIdx.x * int64_t(256) + threadIdx.x; idx < total;
       idx += int64_t(gridDim.x) * 256) {
    const int lane = idx & 63, word = int(idx >> 6) % (2 * AV);
    const int64_t ts = (idx >> 6) / (2 * AV);
    const int s = int(ts % slices), seg = s / sps;
    const int m = int(ts / slices) * 32 + (lane & 31);
    const int k = (s - seg * sps) * kSlice + (lane >> 5) * 16 + word * W;
    float x[W];
#pragma unroll
    for (int i = 0; i < W; ++i) {
      double v = 0.0;
      if (m < n && k + i < n) {
        const int64_t o = k + i + m * lda;
        v = !cplx ? A[o] : seg == 0 ? A[2 * o] : -A[2 * o + 1];
      }
      x[i] = float(v);
    }
    u32x4 w;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if constexpr (W == 4)
        w[i] = __float_as_uint(x[i]);
      else
        w[i] = pack_rne(x[2 * i], x[2 * i + 1]);
    }
    out[idx] = w;
  }
}

// First step's right operand: ks .* B packed; 32 rows x 32 columns a workgroup,
// rows past n as zeros.
template <int P>
__global__ __launch_bounds__(256) void k_pack(StepArgs a) {
  const int m = blockIdx.x * kSlice + (threadIdx.x & 7) * 4;
  const int c = blockIdx.y * 32 + (threadIdx.x >> 3);
  if (c >= a.N) return;
  f32x4 v;
#pragma unroll
  for (int i = 0; i < 4; ++i)
    v[i] = m + i < a.n ? a.B[m + i + c * a.ldb] * (a.ks ? a.ks[m + i] : 1.f) : 0.f;
  pack4<P>(a, m, c, v);
}

// rows m .. m + 3 of column c: the epilogue's operands, and its value
struct EpiRegs {
  f32x4 c1, c2, c3;
  float f3;
};
__device__ __forceinline__ f32x4 load4(const float* p, int left) {
  if (left >= 4) return *reinterpret_cast<const f32x4u*>(p);
  f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < 3; ++i)
    if (i < left) v[i] = p[i];
  return v;
}
// (an absent operand counts as zero, with no branch around its value's use)
__device__ __forceinline__ EpiRegs epi_load(const Epilogue<float>& e, int m, int c, int left) {
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  EpiRegs r = {zero, zero, zero, e.delta};
  if (e.C1) r.c1 = load4(e.C1 + m + c * e.ldc1, left);
  if (e.C2) r.c2 = load4(e.C2 + m + c * e.ldc2, left);
  if (e.C3) {
    r.c3 = load4(e.C3 + m + c * e.ldc3, left);
    if (e.colscale3) r.f3 *= e.colscale3[c];
  }
  return r;
}
__device__ __forceinline__ f32x4 epi_value(const Epilogue<float>& e, const EpiRegs& r, f32x4 s, int m,
                                           int left) {
  f32x4 v = e.alpha * s;
  if (e.rowscale) v *= load4(e.rowscale + m, left);
  v += e.beta * r.c1;
  v += e.gamma * r.c2;
  v += r.f3 * r.c3;
  return v;
}
__device__ __forceinline__ void store4(float* p, f32x4 v, int left) {
  if (left >= 4) {
    *reinterpret_cast<f32x4u*>(p) = v;
  } else {
#pragma unroll
    for (int i = 0; i < 3; ++i)
      if (i < left) p[i] = v[i];
  }
}

// rows m .. m + 3 of column c (left of them below n) into the next step's right
// operand, rows past n as zeros up to the end of the last slice
template <int P>
__device__ __forceinline__ void pack_next(const StepArgs& a, int m, int c, int left, f32x4 v) {
  if (m >= a.sps * kSlice) return;
  f32x4 x;
#pragma unroll
  for (int i = 0; i < 4; ++i) x[i] = i < left ? v[i] * (a.ks ? a.ks[m + i] : 1.f) : 0.f;
  pack4<P>(a, m, c, x);
}

// Sum of the split-K partials in split order, the epilogue, and (pack) the next
// step's right operand from the values just formed.  32 rows x 32 columns a workgroup.
template <int P>
__global__ __launch_bounds__(256) void k_step_reduce(StepArgs a, int pack) {
  const int m = blockIdx.x * kSlice + (threadIdx.x & 7) * 4;
  const int c = blockIdx.y * 32 + (threadIdx.x >> 3);
  if (c >= a.N) return;
  const int left = a.n - m;
  f32x4 v = {0.f, 0.f, 0.f, 0.f};
  if (left > 0) {
    const int64_t MN = int64_t(a.n) * a.N;
    const float* p = a.partial + m + int64_t(c) * a.n;
    const EpiRegs er = epi_load(a.epi, m, c, left);
    f32x4 s = load4(p, left);
    for (int q = 1; q < a.splits; ++q) s += load4(p + q * MN, left);
    v = epi_value(a.epi, er, s, m, left);
    store4(a.C + m + c * a.ldc, v, left);
  }
  if (pack) pack_next<P>(a, m, c, left, v);
}

// ---------------------------------------------------------------------------
// Large products: split-K over workgroups, right operand packed.
//  * Four waves along m, each a 32 x 32 TN tile on v_mfma_f32_32x32x16_bf16 (TN <=
//    5: with three planes two accumulators of 16 TN registers each), two
//    workgroups per CU, so that one's matrix instructions cover the other's
//    splitting, waits and barriers.
//  * The left operand goes from memory straight into registers a stage ahead and
//    is split there, under the matrix instructions of the step before: the
//    operator is read as 4 bytes an element, not 6.
//  * The right operand goes straight into LDS, double-buffered; a step reads one
//    plane's fragments while the plane before is multiplied.
// Measured, us a step with its reduction (FP32 / bfloat16 matrix instructions with
// split-K before): FP32 8192 x 320 239 (399), 4096 x 272 71; BF16 8192 x 320 67
// (88), 4096 x 272 31 (145: its block was no multiple of the tile).  The matrix
// units reach about 1800 TFLOP/s on random operands here (clock), which is 143 us
// for 8192 x 320 in FP32; operand traffic through L2 (1.3 GB a step) holds it
// above that.
// ---------------------------------------------------------------------------
// 16 bytes per lane from global memory straight into LDS: lane l's at dst + 16 l
// (dst the same for the whole wave)
__device__ __forceinline__ void load_to_lds(const void* src, void* dst) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                   (__attribute__((address_space(3))) void*)dst, 16, 0, 0);
}

template <int TN, int P, int SL>
__global__ __launch_bounds__(256, 2) void k_step_large(StepArgs a) {
  constexpr int NT = 256, BM = 128, BN = 32 * TN;
  constexpr int VEC = P * 4 * BN;                 // 16-byte words of a staged slice
  constexpr int NV = (VEC * SL + NT - 1) / NT;
  constexpr int AV = P == 1 ? 1 : 2;              // 16-byte words of A per lane and half slice
  constexpr int ST = 2 * SL;                      // 16-deep steps of a stage
  static_assert(VEC * SL % 64 == 0, "whole waves stage");
  __shared__ __attribute__((aligned(16))) u32x4 Bs[2][VEC * SL];
  const int t = xcd_tile(blockIdx.x, gridDim.x);
  const int n_tile = t % a.tiles_n, r = t / a.tiles_n;
  const int m_tile = r % a.tiles_m, split = r / a.tiles_m;
  const int s_beg = split * a.spc, s_end = min(a.slices, s_beg + a.spc);
  const int nst = (s_end - s_beg + SL - 1) / SL;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int l32 = lane & 31, h = lane >> 5;
  const int m0 = m_tile * BM + wave * 32, n0 = n_tile * BN;
  // the lane's 8 values of step e (half slice e & 1 of slice e / 2) of stage st;
  // stages past the range repeat the last one, unused
  u32x4 raw[ST][AV];
  // (waves past the last row tile repeat it, unused)
  const int mt = min(m0 / 32, (a.n + 31) / 32 - 1);
  const char* Al = static_cast<const char*>(a.A) +
                   (int64_t(mt) * a.slices + s_beg) * (2048 * AV) + lane * 16;
  auto load_a = [&](int st, int e) __attribute__((always_inline)) {
    const char* p = Al + int64_t(min(st, nst - 1)) * (2048 * AV * SL) + e * (1024 * AV);
#pragma unroll
    for (int i = 0; i < AV; ++i) raw[e][i] = *reinterpret_cast<const u32x4*>(p + 1024 * i);
  };
  // staged word v of a stage: slice v / VEC, (plane, chunk) row, column
  uint32_t boff[NV];
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int v = threadIdx.x + i * NT;
    boff[i] = (uint32_t(v / BN) * a.Np + v % BN) * 16u;
  }
  const char* Bg = reinterpret_cast<const char*>(
      a.Bp + (int64_t(s_beg) * P * 4 * a.Np + n0) * 8);
  const int64_t bstride = int64_t(SL) * P * 4 * a.Np * 16;
  auto stage_b = [&](int st, int buf) __attribute__((always_inline)) {
    const char* p = Bg + min(st, nst - 1) * bstride;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      if (VEC * SL % NT != 0 && i * NT + wave * 64 >= VEC * SL) break;
      load_to_lds(p + boff[i], &Bs[buf][i * NT + wave * 64]);
    }
  };
  // three planes: the leading terms and the five small ones in accumulators of
  // their own, so that only one rounding at the sum's own size falls on 16 k values
  constexpr int NA = P == 1 ? 1 : 2;
  f32x16 acc[NA][TN];
#pragma unroll
  for (int v = 0; v < NA; ++v)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[v][j][i] = 0.f;

  bf16x8 af[ST][P];
  auto split_a = [&](int e) __attribute__((always_inline)) {
    if constexpr (P == 3)
      split8<P>(__builtin_bit_cast(f32x4, raw[e][0]), __builtin_bit_cast(f32x4, raw[e][1]), af[e]);
  };
  // the right operand's fragments of group g: step g / P, plane P - 1 - g % P
  bf16x8 bf[2][TN];
  auto read_b = [&](int buf, int g) __attribute__((always_inline)) {
    const int e = g / P, q = P - 1 - g % P;
#pragma unroll
    for (int j = 0; j < TN; ++j)
      bf[g & 1][j] = __builtin_bit_cast(
          bf16x8, Bs[buf][(e / 2) * VEC + (q * 4 + 2 * h + (e & 1)) * BN + j * 32 + l32]);
  };
  auto mult = [&](int g) __attribute__((always_inline)) {
    const int e = g / P, q = P - 1 - g % P;
#pragma unroll
    for (int p = P - 1 - q; p >= 0; --p)
#pragma unroll
      for (int j = 0; j < TN; ++j)
        acc[p + q > 0][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
            P == 1 ? __builtin_bit_cast(bf16x8, raw[e][0]) : af[e][p], bf[g & 1][j],
            acc[p + q > 0][j], 0, 0, 0);
  };

  // The waits below count outstanding loads, which return in order: a wave's
  // part of a stage is in LDS once only the A loads requested after it are
  // outstanding.  (The fences keep the compiler from moving loads across.)
  constexpr int kA = ST * AV;
  static_assert(kA == 4, "the wait count below");
  stage_b(0, 0);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int e = 0; e < ST; ++e) load_a(0, e);
  split_a(0);
  if constexpr (P == 3) load_a(1, 0);
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_waitcnt(0x0f70);             // vmcnt(0)
  __syncthreads();
  for (int st = 0; st < nst; ++st) {
    stage_b(st + 1, (st + 1) & 1);
    __builtin_amdgcn_sched_barrier(0);
    read_b(st & 1, 0);
#pragma unroll
    for (int e = 0; e < ST; ++e) {
      // three planes: the next step's values are split under this step's
      // products and their registers requested anew; one plane: this step's
      constexpr int A1 = P == 3 ? 1 : 0;
      const int en = (e + A1) % ST;
      if constexpr (P == 3) split_a(en);
#pragma unroll
      for (int g = e * P; g < (e + 1) * P; ++g) {
        if (g + 1 < ST * P) read_b(st & 1, g + 1);
        mult(g);
      }
      __builtin_amdgcn_sched_barrier(0);
      load_a(st + 1 + (e + A1) / ST, en);
    }
    __builtin_amdgcn_sched_barrier(0);
    // (a barrier by its builtin or __syncthreads would wait for every load)
    asm volatile("s_waitcnt vmcnt(4) lgkmcnt(0)\n\ts_barrier" ::: "memory");
  }
  __builtin_amdgcn_s_waitcnt(0x0f70);             // nothing outstanding into LDS at the end

  if constexpr (P == 3) {
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      asm volatile("" : "+v"(acc[1][j]));         // the sum stays outside the loop
      acc[0][j] += acc[1][j];
    }
  }
  // element 4 g + i of tile j: row 8 g + 4 h + i, column l32
  float* Pp = a.partial + int64_t(split) * a.n * a.N;
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int c = n0 + j * 32 + l32;
    if (c >= a.N) continue;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int m = m0 + 8 * g + 4 * h;
      if (m < a.n)
        store4(Pp + m + int64_t(c) * a.n,
               f32x4{acc[0][j][4 * g], acc[0][j][4 * g + 1], acc[0][j][4 * g + 2],
                     acc[0][j][4 * g + 3]}, a.n - m);
    }
  }
}

// ---------------------------------------------------------------------------
// Small products: the whole step in one launch.  A workgroup forms a 32 x (32 TN)
// tile; its eight waves take the k-slices in turn (both operands packed, straight
// from L2), add their partial tiles through LDS in wave order, and 4 TN of
// them apply the epilogue, whose operands were requested first, and pack the next
// step's right operand into the other of two buffers.  L2 latency and the launch bound
// it: 1024 x 80 in FP32 takes 8.0 us a step, against 16.7 in two launches.  (More
// slices in flight per wave change nothing.)  A branch around the use of an absent
// operand made the compiler keep the arguments in LDS, at an address that needs the
// dispatch packet in host memory: 14.3 us.
// ---------------------------------------------------------------------------
template <int P, int TN>
__global__ __launch_bounds__(512) void k_step_small(StepArgs a, int pack) {
  constexpr int NW = 8, AV = P == 1 ? 1 : 2;
  __shared__ __attribute__((aligned(16))) f32x4 red[NW][TN][4][64];
  const int t = xcd_tile(blockIdx.x, gridDim.x);
  const int n_tile = t % a.tiles_n, m_tile = t / a.tiles_n;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int l32 = lane & 31, h = lane >> 5;
  const int n0 = n_tile * 32 * TN;
  const char* Al = static_cast<const char*>(a.A) + int64_t(m_tile) * a.slices * (2048 * AV) + lane * 16;
  const char* Bl = reinterpret_cast<const char*>(a.Bp) + (int64_t(2 * h) * a.Np + n0 + l32) * 16;
  // the second column half, or (past the packed columns) the first again, unused
  const int second = n0 + 32 < a.Np ? 512 : 0;
  // this thread's part of the epilogue: four rows of one column
  const int ew = wave & 3, et = wave >> 2;
  const int em = m_tile * 32 + 8 * ew + 4 * h, ec = n0 + 32 * et + l32, eleft = a.n - em;
  const bool mine = et < TN && ec < a.N;
  EpiRegs er;
  if (mine && eleft > 0) er = epi_load(a.epi, em, ec, eleft);

  struct Slice {
    u32x4 x[2][AV], y[2][TN][P];
  };
  auto load = [&](int s) __attribute__((always_inline)) {
    Slice r;
    const char* p = Al + int64_t(s) * (2048 * AV);
    const char* b = Bl + int64_t(s) * (P * 64) * a.Np;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
#pragma unroll
      for (int i = 0; i < AV; ++i)
        r.x[u][i] = *reinterpret_cast<const u32x4*>(p + (AV * u + i) * 1024);
#pragma unroll
      for (int c = 0; c < TN; ++c)
#pragma unroll
        for (int q = 0; q < P; ++q)
          r.y[u][c][q] =
              *reinterpret_cast<const u32x4*>(b + int64_t(q * 4 + u) * 16 * a.Np + c * second);
    }
    return r;
  };
  f32x16 acc[TN], low[TN];                         // P = 3: x0 y0, and the five small terms
#pragma unroll
  for (int c = 0; c < TN; ++c)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[c][i] = low[c][i] = 0.f;
  auto compute = [&](const Slice& r) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      bf16x8 af[P];
      if constexpr (P == 3)
        split8<P>(__builtin_bit_cast(f32x4, r.x[u][0]), __builtin_bit_cast(f32x4, r.x[u][1]), af);
      else
        af[0] = __builtin_bit_cast(bf16x8, r.x[u][0]);
#pragma unroll
      for (int q = P - 1; q >= 0; --q)
#pragma unroll
        for (int p = P - 1 - q; p >= 0; --p)
#pragma unroll
          for (int c = 0; c < TN; ++c) {
            f32x16& into = p + q == 0 ? acc[c] : low[c];
            into = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                af[p], __builtin_bit_cast(bf16x8, r.y[u][c][q]), into, 0, 0, 0);
          }
    }
  };
  // (slices past n, which fill up a segment for the large path, hold nothing)
  const int valid = (a.n + kSlice - 1) / kSlice, ns = valid * a.nseg;
  if (wave < ns) {
    Slice cur = load(wave < valid ? wave : a.sps + wave - valid);
    for (int i = wave + NW; i < ns; i += NW) {
      const Slice nxt = load(i < valid ? i : a.sps + i - valid);
      compute(cur);
      cur = nxt;
    }
    compute(cur);
  }
#pragma unroll
  for (int c = 0; c < TN; ++c) {
    if constexpr (P == 3) acc[c] += low[c];
#pragma unroll
    for (int g = 0; g < 4; ++g)
      red[wave][c][g][lane] =
          f32x4{acc[c][4 * g], acc[c][4 * g + 1], acc[c][4 * g + 2], acc[c][4 * g + 3]};
  }
  __syncthreads();
  if (!mine) return;
  f32x4 v = {0.f, 0.f, 0.f, 0.f};
  if (eleft > 0) {
    f32x4 s = red[0][et][ew][lane];
#pragma unroll
    for (int w = 1; w < NW; ++w) s += red[w][et][ew][lane];
    v = epi_value(a.epi, er, s, em, eleft);
    store4(a.C + em + ec * a.ldc, v, eleft);
  }
  if (pack) pack_next<P>(a, em, ec, eleft, v);
}

template <int P, int SL>
hipError_t launch_large(const StepArgs& a, int tn, hipStream_t st) {
  const dim3 grid(unsigned(a.tiles_m) * a.tiles_n * a.splits), block(256);
  switch (tn) {
    case 1: k_step_large<1, P, SL><<<grid, block, 0, st>>>(a); break;
    case 2: k_step_large<2, P, SL><<<grid, block, 0, st>>>(a); break;
    case 3: k_step_large<3, P, SL><<<grid, block, 0, st>>>(a); break;
    case 4: k_step_large<4, P, SL><<<grid, block, 0, st>>>(a); break;
    default: k_step_large<5, P, SL><<<grid, block, 0, st>>>(a); break;
  }
  return hipGetLastError();
}

template <int P>
hipError_t launch_small(const StepArgs& a, int tn, int pack, hipStream_t st) {
  if (tn == 2)
    k_step_small<P, 2><<<dim3(unsigned(a.tiles_m) * a.tiles_n), dim3(512), 0, st>>>(a, pack);
  else
    k_step_small<P, 1><<<dim3(unsigned(a.tiles_m) * a.tiles_n), dim3(512), 0, st>>>(a, pack);
  return hipGetLastError();
}

size_t align256(size_t v) { return (v + 255) / 256 * 256; }

// slices of one k-segment: whole stages of the large kernel
int segment_slices(int64_t n, int planes) {
  const int64_t w = planes == 1 ? 2 * kSlice : kSlice;
  return int((n + w - 1) / w * w / kSlice);
}

// the large path's column tiles (of 32 tn columns; as equal as that allows)
int column_tiles(int64_t N, int* tn) {
  const int c32 = int((N + 31) / 32), tiles = (c32 + 4) / 5;
  *tn = (c32 + tiles - 1) / tiles;
  return tiles;
}

// bytes of a packed right operand
size_t packed_bytes(int64_t n, int64_t N, int nseg, int planes) {
  int tn;
  const int tiles = column_tiles(N, &tn);
  return align256(size_t(nseg) * segment_slices(n, planes) * kSlice * tiles * tn * 32 * planes * 2);
}

}  // namespace

size_t filter_operator_bytes(int64_t n, int nseg, int planes) {
  return size_t((n + 31) / 32) * nseg * segment_slices(n, planes) * 1024 * (planes == 1 ? 2 : 4);
}

hipError_t pack_filter_operator(const double* A, int64_t lda, int64_t n, int nseg, int planes,
                                void* out, hipStream_t st) {
  const int sps = segment_slices(n, planes);
  const int64_t total = int64_t(filter_operator_bytes(n, nseg, planes) / 16);
  const dim3 grid(unsigned(std::min<int64_t>((total + 255) / 256, 1 << 20)));
  if (planes == 1)
    k_pack_operator<unsigned short><<<grid, dim3(256), 0, st>>>(
        A, lda, int(n), sps, sps * nseg, nseg - 1, static_cast<u32x4*>(out), total);
  else
    k_pack_operator<float><<<grid, dim3(256), 0, st>>>(A, lda, int(n), sps, sps * nseg, nseg - 1,
                                                       static_cast<u32x4*>(out), total);
  return hipGetLastError();
}

size_t filter_product_bytes(int64_t n, int64_t N, int nseg, int planes) {
  return 2 * packed_bytes(n, N, nseg, planes);
}

hipError_t filter_product(const FilterProduct& d, hipStream_t st, const Workspace& ws,
                          int force_splits, int* packed) {
  const int was_packed = *packed;
  *packed = 0;
  if (d.n <= 0 || d.N <= 0) return hipSuccess;
  if ((d.planes != 1 && d.planes != 3) || (d.nseg != 1 && d.nseg != 2)) return hipErrorInvalidValue;
  const int64_t c32 = (d.N + 31) / 32;
  if (d.n >= (int64_t(1) << 30) || c32 > 65535) return hipErrorInvalidValue;
  const size_t pbytes = packed_bytes(d.n, d.N, d.nseg, d.planes);
  if (!ws.ptr || ws.bytes < 2 * pbytes) return hipErrorInvalidValue;
  StepArgs a;
  a.A = d.A;
  a.B = d.B;
  a.ldb = d.ldb;
  a.ks = d.kscale;
  a.C = d.C;
  a.ldc = d.ldc;
  a.epi = d.epi;
  a.n = int(d.n);
  a.N = int(d.N);
  a.half = a.N / 2;
  a.nseg = d.nseg;
  a.sps = segment_slices(d.n, d.planes);
  a.slices = a.sps * a.nseg;
  int tn;
  a.tiles_n = column_tiles(d.N, &tn);
  a.Np = a.tiles_n * tn * 32;
  char* buf[2] = {static_cast<char*>(ws.ptr), static_cast<char*>(ws.ptr) + pbytes};
  a.partial = reinterpret_cast<float*>(buf[1]);
  // k-splits of the large path: two workgroups per CU, at least 8 slices each
  a.tiles_m = (a.n + 127) / 128;
  const int64_t tiles = int64_t(a.tiles_m) * a.tiles_n;
  int splits = force_splits > 0 ? force_splits : int(std::max<int64_t>(1, 512 / tiles));
  splits = std::min(splits, std::max(1, a.slices / 8));
  splits = int(std::min<size_t>(splits, (ws.bytes - pbytes) / (size_t(d.n) * d.N * sizeof(float))));
  // one launch below this much work (n N slices): it re-reads the operands per 32 x 32
  // tile, but the second launch and the partials' round trip are saved.  Measured, us a
  // step, one launch / two: three planes 1024 x 80 (2.6e6) 8.0 / 16.7, 2048 x 144 20.1 /
  // 26.7, 3072 x 160 (4.7e7) 28.5 / 40.9, 4096 x 144 (7.5e7) 51.3 / 49.3, 8192 x 64 (1.3e8)
  // 90.6 / 71.1; one plane 1024 x 80 6.3 / 11.1, 4096 x 144 21.0 / 24.9, 8192 x 64 27.3 /
  // 31.4, 4096 x 272 (1.4e8) 31.7 / 31.3, 8192 x 128 (2.7e8) 52.6 / 38.9
  const bool large = splits > 0 && (force_splits > 0 || double(d.n) * d.N * a.slices >=
                                                             (d.planes == 3 ? 7e7 : 1.4e8));
  const dim3 grid32(unsigned(a.sps), unsigned(c32));
  const int pack = d.pack_next ? 1 : 0;
  if (!was_packed) {
    a.Bn = reinterpret_cast<unsigned short*>(buf[0]);
    if (d.planes == 3)
      k_pack<3><<<grid32, dim3(256), 0, st>>>(a);
    else
      k_pack<1><<<grid32, dim3(256), 0, st>>>(a);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (large) {
    a.spc = (a.slices + splits - 1) / splits;
    if (d.planes == 1) a.spc = (a.spc + 1) / 2 * 2;
    a.splits = (a.slices + a.spc - 1) / a.spc;
    if (tiles * a.splits > 0x7fffffff) return hipErrorInvalidValue;
    a.Bp = a.Bn = reinterpret_cast<unsigned short*>(buf[0]);
    const hipError_t e = d.planes == 3 ? launch_large<3, 1>(a, tn, st) : launch_large<1, 2>(a, tn, st);
    if (e != hipSuccess) return e;
    if (d.planes == 3)
      k_step_reduce<3><<<grid32, dim3(256), 0, st>>>(a, pack);
    else
      k_step_reduce<1><<<grid32, dim3(256), 0, st>>>(a, pack);
    *packed = pack;
    return hipGetLastError();
  }
  const int from = was_packed == 2 ? 1 : 0;
  a.Bp = reinterpret_cast<unsigned short*>(buf[from]);
  a.Bn = reinterpret_cast<unsigned short*>(buf[1 - from]);
  a.tiles_m = (a.n + 31) / 32;
  // Two column tiles a workgroup (the operator is split once for both) where that and not
  // one leaves at most a workgroup to each CU.  Measured, us a step, one / two: FP32
  // 2048 x 144 19.9 / 17.7, 3001 x 128 27.0 / 23.3, complex 1500 x 300 30.1 / 25.5, BF16
  // 8192 x 64 27.6 / 24.6; FP32 1024 x 160 (160 tiles) 8.5 / 10.9, 4096 x 64 (256) 20.1 /
  // 28.6, 2500 x 200 (553, in pairs 316) 34.0 / 37.5.
  auto tiles_of = [&](int tn) { return int64_t(a.tiles_m) * ((a.N + 32 * tn - 1) / (32 * tn)); };
  const int small_tn = tiles_of(1) > 256 && tiles_of(2) <= 256 ? 2 : 1;
  a.tiles_n = (a.N + 32 * small_tn - 1) / (32 * small_tn);
  a.splits = 1;
  a.spc = a.slices;
  if (int64_t(a.tiles_m) * a.tiles_n > 0x7fffffff) return hipErrorInvalidValue;
  *packed = pack ? 2 - from : 0;
  return d.planes == 3 ? launch_small<3>(a, small_tn, pack, st) : launch_small<1>(a, small_tn, pack, st);
}

}  // namespace chfsi
