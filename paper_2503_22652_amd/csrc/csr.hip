// Sparse symmetric operators in compressed sparse row form: the operator
// products of the filter (Algorithms 2 and 3) and of Rayleigh-Ritz for the
// finite-element-type matrices of Section 4.2.
//
// Blocks are column-major n x b.  One workgroup owns a tile of 64 consecutive
// rows: it stages the tile's column indices and values in LDS as a padded
// [k][row] array (ELL layout within the tile; padding entries carry weight 0
// and a valid index), then its four waves sweep the block's columns, one
// column per wave at a time, one row per lane.  The matrix is read from HBM
// once per launch, whatever b is; the gathered source entries of neighbouring
// rows fall in the same cache lines for banded / grid-ordered matrices; the
// epilogue (the filter's three-term update, or the row scaling of the plain
// filter) reads and writes each output element once, coalesced across lanes.
// For the residual filter's A (D^{-1} R_Y), D^{-1} is folded into the staged
// values (column side).  Rows longer than kLdsKmax use a plain kernel with one
// thread per (row, column).
//
// The gathers bound that sweep: 64^3 grid, 27 entries a row, 64 FP32 columns took 153 us
// a step.  The residual filter therefore keeps its blocks in groups of G columns of 16
// bytes a row, element (i, j) at (j / G * n + i) G + j % G and the last b % G columns
// column by column: a gather is then one aligned 16-byte load for G columns and the
// addresses and staged entries are shared.  113 us a step, 93 of them the L1 lookups (two
// per 64 bytes for a row's shifted neighbours).  128- and 256-row tiles, whose gathers
// could share lines in L1, take 124 and 134 us; round-robin tiles over the XCDs 127.
#include "internal.h"
#include "stencil_api.h"

#include <algorithm>

namespace chfsi {

namespace {

constexpr int kRows = 64;
constexpr int kThreads = 256;
constexpr int kLdsKmax = 80;   // staged row length: 64 x 80 x 12 B = 60 KB of LDS at most

enum { MODE_APPLY = 0, MODE_RSTEP = 1, MODE_CSTEP = 2 };

__device__ __forceinline__ double load_as(const double* p, int64_t i, double) { return p[i]; }
__device__ __forceinline__ float load_as(const float* p, int64_t i, float) { return p[i]; }
__device__ __forceinline__ float load_as(const uint16_t* p, int64_t i, float) {
  return __uint_as_float(uint32_t(p[i]) << 16);
}
__device__ __forceinline__ void store_to(double* p, int64_t i, double v) { p[i] = v; }
__device__ __forceinline__ void store_to(float* p, int64_t i, float v) { p[i] = v; }
__device__ __forceinline__ void store_to(uint16_t* p, int64_t i, float v) {
  // round to nearest even (v_cvt_pk_bf16_f32)
  p[i] = __builtin_bit_cast(uint16_t, static_cast<__bf16>(v));
}

template <typename S, typename AT, typename VT>
struct CsrArgs {
  int64_t n, b;
  const int64_t* rowptr;
  const int32_t* col;
  const VT* val;
  int kmax;
  const AT* cdinv;     // column-side scaling of the values (residual filter), or null
  const AT* rdinv;     // row-side scaling of the product (plain filter), or null
  const S* src;
  int64_t lds;
  S* dst;
  int64_t ldd;
  const S* prev;       // may alias dst
  int64_t ldp;
  const S* forc;
  int64_t ldf;
  const AT* colcoef;
  AT alpha, beta, gamma, delta;
};

// workgroups go round-robin over the 8 XCDs: neighbouring tiles, which share source
// entries, on one XCD
__device__ __forceinline__ int64_t xcd_unit(int64_t h, int64_t total) {
  const int64_t xcd = h & 7, slot = h >> 3, full = total >> 3, rem = total & 7;
  return xcd < rem ? xcd * (full + 1) + slot : rem * (full + 1) + (xcd - rem) * full + slot;
}

template <typename S, typename AT, typename VT, int MODE>
__device__ __forceinline__ void epilogue(const CsrArgs<S, AT, VT>& a, int64_t row, int64_t j,
                                         AT acc) {
  AT out;
  if (MODE == MODE_APPLY) {
    out = acc;
  } else if (MODE == MODE_RSTEP) {
    out = a.alpha * acc + a.beta * load_as(a.src, row + j * a.lds, AT()) +
          a.gamma * load_as(a.prev, row + j * a.ldp, AT()) +
          a.delta * a.colcoef[j] * load_as(a.forc, row + j * a.ldf, AT());
  } else {
    const AT d = a.rdinv ? a.rdinv[row] : AT(1);
    out = a.alpha * d * acc + a.beta * load_as(a.src, row + j * a.lds, AT());
    if (a.prev) out += a.gamma * load_as(a.prev, row + j * a.ldp, AT());
  }
  store_to(a.dst, row + j * a.ldd, out);
}

template <typename S, typename AT, typename VT, int MODE>
__global__ __launch_bounds__(kThreads) void k_csr_tile(CsrArgs<S, AT, VT> a) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int kmax = a.kmax;
  int32_t* lc = reinterpret_cast<int32_t*>(smem);
  VT* lv = reinterpret_cast<VT*>(smem + ((size_t(kmax) * kRows * sizeof(int32_t) + 15) & ~size_t(15)));
  const int64_t row0 = xcd_unit(blockIdx.x, gridDim.x) * kRows;
  for (int idx = threadIdx.x; idx < kmax * kRows; idx += kThreads) {
    const int r = idx & (kRows - 1), k = idx / kRows;
    const int64_t row = row0 + r;
    int32_t c = 0;
    VT v = VT(0);
    if (row < a.n) {
      c = int32_t(row);   // padding: this row's own index with weight 0
      const int64_t s = a.rowptr[row], e = a.rowptr[row + 1];
      if (k < e - s) {
        c = a.col[s + k];
        v = a.val[s + k];
        if (a.cdinv) v = VT(AT(v) * a.cdinv[c]);
      }
    }
    lc[idx] = c;
    lv[idx] = v;
  }
  __syncthreads();
  const int lane = threadIdx.x & (kRows - 1), wave = threadIdx.x / kRows;
  const int64_t row = row0 + lane;
  if (row >= a.n) return;   // no barrier follows
  for (int64_t j = wave; j < a.b; j += kThreads / kRows) {
    const S* sj = a.src + j * a.lds;
    AT acc = AT(0);
    for (int k = 0; k < kmax; ++k)
      acc += AT(lv[k * kRows + lane]) * load_as(sj, lc[k * kRows + lane], AT());
    epilogue<S, AT, VT, MODE>(a, row, j, acc);
  }
}

// ---------------------------------------------------------------------------
// Residual-filter blocks in groups of columns
// ---------------------------------------------------------------------------
template <typename S>
constexpr int kGroup = 16 / int(sizeof(S));
template <typename S>
struct GroupOf {
  typedef S type __attribute__((ext_vector_type(16 / sizeof(S))));
};

// element (i, j)
template <typename S>
__device__ __forceinline__ int64_t group_index(int64_t i, int64_t j, int64_t n, int64_t b) {
  constexpr int G = kGroup<S>;
  const int64_t full = b / G * G;
  return j < full ? (j / G * n + i) * G + j % G : j * n + i;
}

// the filter's start: RY = scale R, RX = 0 and (Yc given) Yc = R
template <typename S, typename AT>
__global__ __launch_bounds__(kThreads) void k_csr_init(const double* R, int64_t ldr, int64_t n,
                                                       int64_t b, double scale, S* RY, S* RX, S* Yc) {
  constexpr int G = kGroup<S>;
  typedef typename GroupOf<S>::type V;
  const int64_t ng = b / G, items = n * (ng + b % G);
  for (int64_t idx = int64_t(blockIdx.x) * kThreads + threadIdx.x; idx < items;
       idx += int64_t(gridDim.x) * kThreads) {
    const int64_t q = idx / n, i = idx - q * n;
    if (q < ng) {
      V y, z, r;
#pragma unroll
      for (int c = 0; c < G; ++c) {
        const double v = R[i + (q * G + c) * ldr];
        S t;
        store_to(&t, 0, AT(scale * v));
        y[c] = t;
        store_to(&t, 0, AT(v));
        r[c] = t;
        z[c] = S(0);
      }
      reinterpret_cast<V*>(RY)[idx] = y;
      reinterpret_cast<V*>(RX)[idx] = z;
      if (Yc) reinterpret_cast<V*>(Yc)[idx] = r;
    } else {
      const int64_t j = ng * G + (q - ng), at = j * n + i;
      const double v = R[i + j * ldr];
      store_to(RY, at, AT(scale * v));
      store_to(RX, at, AT(0));
      if (Yc) store_to(Yc, at, AT(v));
    }
  }
}

// the filter's end: Yp = D^{-1} RY + X Lambda_Y
template <typename S, typename AT>
__global__ __launch_bounds__(kThreads) void k_csr_reconstruct(const S* RY, const double* dinv,
                                                              const double* X, int64_t ldx,
                                                              const double* lamY, double* Yp,
                                                              int64_t ldy, int64_t n, int64_t b) {
  constexpr int G = kGroup<S>;
  typedef typename GroupOf<S>::type V;
  const int64_t ng = b / G, items = n * (ng + b % G);
  for (int64_t idx = int64_t(blockIdx.x) * kThreads + threadIdx.x; idx < items;
       idx += int64_t(gridDim.x) * kThreads) {
    const int64_t q = idx / n, i = idx - q * n;
    const bool group = q < ng;
    const int64_t j0 = group ? q * G : ng * G + (q - ng);
    V y;
    if (group)
      y = reinterpret_cast<const V*>(RY)[idx];
    else
      y[0] = RY[j0 * n + i];
#pragma unroll
    for (int c = 0; c < G; ++c) {
      if (c > 0 && !group) break;
      const S t = y[c];
      double r = double(load_as(&t, 0, AT()));
      if (dinv) r *= dinv[i];
      Yp[i + (j0 + c) * ldy] = r + X[i + (j0 + c) * ldx] * lamY[j0 + c];
    }
  }
}

// The step RX <- alpha A (D^{-1} RY) + beta RY + gamma RX + delta colcoef[j] Yf on such
// blocks (forc with ldf >= 0: column-major).  `parts` workgroups share a tile's columns.
template <typename S, typename AT, typename VT>
__global__ __launch_bounds__(kThreads) void k_csr_group(CsrArgs<S, AT, VT> a, int parts) {
  constexpr int G = kGroup<S>, CW = kThreads / kRows;
  typedef typename GroupOf<S>::type V;
  extern __shared__ __align__(16) unsigned char smem[];
  const int kmax = a.kmax;
  uint32_t* lo = reinterpret_cast<uint32_t*>(smem);          // byte offset of a row's group
  VT* lv = reinterpret_cast<VT*>(smem + size_t(kmax) * kRows * sizeof(uint32_t));
  const int64_t unit = xcd_unit(blockIdx.x, gridDim.x), row0 = unit / parts * kRows;
  {
    const int r = threadIdx.x % kRows;
    const int64_t row = row0 + r;
    const int64_t s = row < a.n ? a.rowptr[row] : 0, e = row < a.n ? a.rowptr[row + 1] : 0;
#pragma unroll 4
    for (int k = threadIdx.x / kRows; k < kmax; k += CW) {
      int32_t c = row < a.n ? int32_t(row) : 0;   // padding: this row's own index with weight 0
      VT v = VT(0);
      if (k < e - s) {
        c = a.col[s + k];
        v = a.val[s + k];
        if (a.cdinv) v = VT(AT(v) * a.cdinv[c]);
      }
      lo[k * kRows + r] = uint32_t(c) * 16u;
      lv[k * kRows + r] = v;
    }
  }
  __syncthreads();
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t row = row0 + lane;
  if (row >= a.n) return;   // no barrier follows
  lo += lane;
  lv += lane;
  const int64_t ng = a.b / G, first = unit % parts * CW + wave;
  const int64_t step = int64_t(parts) * CW;
  for (int64_t q = first; q < ng; q += step) {
    const char* src = reinterpret_cast<const char*>(reinterpret_cast<const V*>(a.src) + q * a.n);
    const int64_t at = q * a.n + row;
    const V s = reinterpret_cast<const V*>(a.src)[at], p = reinterpret_cast<const V*>(a.prev)[at];
    V f;
    if (a.ldf < 0)
      f = reinterpret_cast<const V*>(a.forc)[at];
    else
#pragma unroll
      for (int c = 0; c < G; ++c) f[c] = a.forc[row + (q * G + c) * a.ldf];
    AT acc[G];
#pragma unroll
    for (int c = 0; c < G; ++c) acc[c] = AT(0);
#pragma unroll 9
    for (int k = 0; k < kmax; ++k) {
      const AT v = AT(lv[k * kRows]);
      const V x = *reinterpret_cast<const V*>(src + lo[k * kRows]);
#pragma unroll
      for (int c = 0; c < G; ++c) {
        const S t = x[c];
        acc[c] += v * load_as(&t, 0, AT());
      }
    }
    V out;
#pragma unroll
    for (int c = 0; c < G; ++c) {
      const S ts = s[c], tp = p[c], tf = f[c];
      S to;
      store_to(&to, 0, a.alpha * acc[c] + a.beta * load_as(&ts, 0, AT()) +
                           a.gamma * load_as(&tp, 0, AT()) +
                           a.delta * a.colcoef[q * G + c] * load_as(&tf, 0, AT()));
      out[c] = to;
    }
    reinterpret_cast<V*>(a.dst)[at] = out;
  }
  for (int64_t j = ng * G + first; j < a.b; j += step) {
    const S* sj = a.src + j * a.n;
    AT acc = AT(0);
#pragma unroll 9
    for (int k = 0; k < kmax; ++k)
      acc += AT(lv[k * kRows]) * load_as(sj, lo[k * kRows] / 16u, AT());
    const int64_t at = j * a.n + row;
    store_to(a.dst, at, a.alpha * acc + a.beta * load_as(sj, row, AT()) +
                            a.gamma * load_as(a.prev, at, AT()) +
                            a.delta * a.colcoef[j] *
                                load_as(a.forc, a.ldf < 0 ? at : row + j * a.ldf, AT()));
  }
}

// rows longer than kLdsKmax: one thread per (row, column), entries from global memory
template <typename S, typename AT, typename VT, int MODE>
__global__ __launch_bounds__(kThreads) void k_csr_plain(CsrArgs<S, AT, VT> a) {
  const int64_t total = a.n * a.b;
  for (int64_t idx = int64_t(blockIdx.x) * kThreads + threadIdx.x; idx < total;
       idx += int64_t(gridDim.x) * kThreads) {
    const int64_t j = idx / a.n, row = idx - j * a.n;
    const S* sj = a.src + j * a.lds;
    AT acc = AT(0);
    for (int64_t p = a.rowptr[row]; p < a.rowptr[row + 1]; ++p) {
      const int32_t c = a.col[p];
      AT v = AT(a.val[p]);
      if (a.cdinv) v *= a.cdinv[c];
      acc += v * load_as(sj, c, AT());
    }
    epilogue<S, AT, VT, MODE>(a, row, j, acc);
  }
}

// structure checks and the longest row: flags[0] |= 1 bad rowptr, 2 bad
// column index; flags[1] = max row length
__global__ __launch_bounds__(kThreads) void k_csr_check(int64_t n, const int64_t* rowptr,
                                                        const int32_t* col, int64_t nnz,
                                                        int* flags) {
  for (int64_t row = int64_t(blockIdx.x) * kThreads + threadIdx.x; row < n;
       row += int64_t(gridDim.x) * kThreads) {
    const int64_t s = rowptr[row], e = rowptr[row + 1];
    if (row == 0 && s != 0) atomicOr(flags, 1);
    if (row == n - 1 && e != nnz) atomicOr(flags, 1);
    if (e < s || s < 0 || e > nnz) {
      atomicOr(flags, 1);
      continue;
    }
    const int64_t len = e - s;
    atomicMax(flags + 1, int(std::min<int64_t>(len, 0x7fffffff)));
    for (int64_t p = s; p < e; ++p)
      if (col[p] < 0 || int64_t(col[p]) >= n) atomicOr(flags, 2);
  }
}

template <typename S, typename AT, typename VT, int MODE>
hipError_t launch(const CsrArgs<S, AT, VT>& a, hipStream_t st) {
  if (a.n <= 0 || a.b <= 0) return hipSuccess;
  if (a.kmax <= kLdsKmax) {
    const int k = std::max(a.kmax, 1);
    CsrArgs<S, AT, VT> a2 = a;
    a2.kmax = k;
    const size_t lds = ((size_t(k) * kRows * sizeof(int32_t) + 15) & ~size_t(15)) +
                       size_t(k) * kRows * sizeof(VT);
    const int64_t tiles = (a.n + kRows - 1) / kRows;
    if (tiles > 0x7fffffff) return hipErrorInvalidValue;
    k_csr_tile<S, AT, VT, MODE><<<dim3(unsigned(tiles)), kThreads, lds, st>>>(a2);
  } else {
    const int64_t g = std::min<int64_t>((a.n * a.b + kThreads - 1) / kThreads, 65536);
    k_csr_plain<S, AT, VT, MODE><<<dim3(unsigned(g)), kThreads, 0, st>>>(a);
  }
  return hipGetLastError();
}

// blocks in groups: rows short enough to stage, 32-bit byte offsets
bool grouped(const CsrMat& A) {
  return A.kmax <= kLdsKmax && A.n <= int64_t(0xffffffff) / 16;
}

// one residual-filter step on the layout of csr_rchfsi_init
template <typename S, typename AT, typename VT>
hipError_t launch_rstep(CsrArgs<S, AT, VT> a, bool group, hipStream_t st) {
  if (a.n <= 0 || a.b <= 0) return hipSuccess;
  if (!group) {
    if (a.ldf < 0) a.ldf = a.n;
    return launch<S, AT, VT, MODE_RSTEP>(a, st);
  }
  a.kmax = std::max(a.kmax, 1);
  const size_t lds = size_t(a.kmax) * kRows * (sizeof(uint32_t) + sizeof(VT));
  const int64_t tiles = (a.n + kRows - 1) / kRows;
  // few tiles: columns split over workgroups, down to a group a wave, up to four a CU
  const int64_t units = a.b / kGroup<S> + a.b % kGroup<S>;
  const int parts = int(std::max<int64_t>(1, std::min((units + 3) / 4, 1024 / tiles)));
  if (tiles * parts > 0x7fffffff) return hipErrorInvalidValue;
  k_csr_group<S, AT, VT><<<dim3(unsigned(tiles * parts)), kThreads, lds, st>>>(a, parts);
  return hipGetLastError();
}

inline unsigned grid_for(int64_t items) {
  return unsigned(std::max<int64_t>(1, std::min<int64_t>((items + kThreads - 1) / kThreads, 65536)));
}

template <typename S, typename AT, typename VT>
CsrArgs<S, AT, VT> base_args(const CsrMat& A, int64_t b) {
  CsrArgs<S, AT, VT> a{};
  a.n = A.n;
  a.b = b;
  a.rowptr = A.rowptr;
  a.col = A.col;
  a.val = static_cast<const VT*>(A.val);
  a.kmax = A.kmax;
  return a;
}

}  // namespace

hipError_t csr_check(const chfsi_operator& op, int* flags_dev, int* flags_host, int* kmax,
                     hipStream_t st) {
  hipError_t e = fill_zero(flags_dev, 2 * sizeof(int), st);
  if (e != hipSuccess) return e;
  const int64_t g = std::max<int64_t>(1, std::min<int64_t>((op.n + kThreads - 1) / kThreads, 4096));
  k_csr_check<<<dim3(unsigned(g)), kThreads, 0, st>>>(op.n, op.rowptr, op.colind, op.nnz, flags_dev);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if ((e = hipMemcpyAsync(flags_host, flags_dev, 2 * sizeof(int), hipMemcpyDeviceToHost, st)) !=
      hipSuccess)
    return e;
  if ((e = hipStreamSynchronize(st)) != hipSuccess) return e;
  *kmax = flags_host[1];
  return flags_host[0] == 0 ? hipSuccess : hipErrorInvalidValue;
}

hipError_t csr_apply_f64(const CsrMat& A, const double* X, int64_t ldx, double* Y, int64_t ldy,
                         int64_t b, hipStream_t st) {
  auto a = base_args<double, double, double>(A, b);
  a.src = X;
  a.lds = ldx;
  a.dst = Y;
  a.ldd = ldy;
  return launch<double, double, double, MODE_APPLY>(a, st);
}

hipError_t csr_rchfsi_init(const CsrMat& A, int prec, const double* R, int64_t ldr, int64_t b,
                           double scale, void* RY, void* RX, void* Yc, hipStream_t st) {
  const int64_t n = A.n;
  if (!grouped(A)) {
    if (prec == CHFSI_PREC_FP64)
      return rchfsi_init_f64(R, ldr, n, b, scale, static_cast<double*>(RY), static_cast<double*>(RX),
                             n, st);
    if (prec == CHFSI_PREC_FP32)
      return rchfsi_init_f32(R, ldr, n, b, scale, static_cast<float*>(RY), static_cast<float*>(RX),
                             static_cast<float*>(Yc), n, st);
    return rchfsi_init_bf16(R, ldr, n, b, scale, RY, RX, Yc, st);
  }
  if (prec == CHFSI_PREC_FP64)
    k_csr_init<double, double><<<grid_for(n * b / 2), kThreads, 0, st>>>(
        R, ldr, n, b, scale, static_cast<double*>(RY), static_cast<double*>(RX), nullptr);
  else if (prec == CHFSI_PREC_FP32)
    k_csr_init<float, float><<<grid_for(n * b / 4), kThreads, 0, st>>>(
        R, ldr, n, b, scale, static_cast<float*>(RY), static_cast<float*>(RX),
        static_cast<float*>(Yc));
  else
    k_csr_init<uint16_t, float><<<grid_for(n * b / 8), kThreads, 0, st>>>(
        R, ldr, n, b, scale, static_cast<uint16_t*>(RY), static_cast<uint16_t*>(RX),
        static_cast<uint16_t*>(Yc));
  return hipGetLastError();
}

hipError_t csr_rchfsi_reconstruct(const CsrMat& A, int prec, const void* RY, const double* dinv,
                                  const double* X, int64_t ldx, const double* lamY, double* Yp,
                                  int64_t ldy, int64_t b, hipStream_t st) {
  const int64_t n = A.n;
  if (!grouped(A)) {
    if (prec == CHFSI_PREC_FP64)
      return rchfsi_reconstruct_f64(static_cast<const double*>(RY), n, dinv, X, ldx, lamY, Yp, ldy,
                                    n, b, st);
    if (prec == CHFSI_PREC_FP32)
      return rchfsi_reconstruct_f32(static_cast<const float*>(RY), n, dinv, X, ldx, lamY, Yp, ldy,
                                    n, b, st);
    return rchfsi_reconstruct_bf16(RY, dinv, X, ldx, lamY, Yp, ldy, n, b, st);
  }
  if (prec == CHFSI_PREC_FP64)
    k_csr_reconstruct<double, double><<<grid_for(n * b / 2), kThreads, 0, st>>>(
        static_cast<const double*>(RY), dinv, X, ldx, lamY, Yp, ldy, n, b);
  else if (prec == CHFSI_PREC_FP32)
    k_csr_reconstruct<float, float><<<grid_for(n * b / 4), kThreads, 0, st>>>(
        static_cast<const float*>(RY), dinv, X, ldx, lamY, Yp, ldy, n, b);
  else
    k_csr_reconstruct<uint16_t, float><<<grid_for(n * b / 8), kThreads, 0, st>>>(
        static_cast<const uint16_t*>(RY), dinv, X, ldx, lamY, Yp, ldy, n, b);
  return hipGetLastError();
}

hipError_t csr_rchfsi_step_f64(const CsrMat& A, const double* dinv, const double* RY, double* RX,
                               const double* Yf, int64_t ldf, const double* colcoef,
                               StencilStep s, int64_t b, hipStream_t st) {
  auto a = base_args<double, double, double>(A, b);
  a.cdinv = dinv;
  a.src = RY;
  a.lds = A.n;
  a.dst = RX;
  a.ldd = A.n;
  a.prev = RX;
  a.ldp = A.n;
  a.forc = Yf;
  a.ldf = ldf;              // the caller's residuals: column-major
  a.colcoef = colcoef;
  a.alpha = s.alpha;
  a.beta = s.beta;
  a.gamma = s.gamma;
  a.delta = s.delta;
  return launch_rstep<double, double, double>(a, grouped(A), st);
}

template <typename S>
static hipError_t rstep_lowp(const CsrMat& A32, const float* dinv, const S* RY, S* RX, const S* Yf,
                             const float* colcoef, StencilStep s, int64_t b, hipStream_t st) {
  auto a = base_args<S, float, float>(A32, b);
  a.cdinv = dinv;
  a.src = RY;
  a.lds = A32.n;
  a.dst = RX;
  a.ldd = A32.n;
  a.prev = RX;
  a.ldp = A32.n;
  a.forc = Yf;
  a.ldf = -1;               // in the blocks' layout
  a.colcoef = colcoef;
  a.alpha = float(s.alpha);
  a.beta = float(s.beta);
  a.gamma = float(s.gamma);
  a.delta = float(s.delta);
  return launch_rstep<S, float, float>(a, grouped(A32), st);
}

hipError_t csr_rchfsi_step_f32(const CsrMat& A32, const float* dinv, const float* RY, float* RX,
                               const float* Yf, const float* colcoef, StencilStep s, int64_t b,
                               hipStream_t st) {
  return rstep_lowp<float>(A32, dinv, RY, RX, Yf, colcoef, s, b, st);
}

hipError_t csr_rchfsi_step_bf16(const CsrMat& A32, const float* dinv, const void* RY, void* RX,
                                const void* Yf, const float* colcoef, StencilStep s, int64_t b,
                                hipStream_t st) {
  return rstep_lowp<uint16_t>(A32, dinv, static_cast<const uint16_t*>(RY),
                              static_cast<uint16_t*>(RX), static_cast<const uint16_t*>(Yf),
                              colcoef, s, b, st);
}

hipError_t csr_chfsi_step_f64(const CsrMat& A, const double* dinv, const double* src,
                              int64_t lds, const double* prev, int64_t ldp, double* dst,
                              StencilStep s, int64_t b, hipStream_t st) {
  auto a = base_args<double, double, double>(A, b);
  a.rdinv = dinv;
  a.src = src;
  a.lds = lds;
  a.dst = dst;
  a.ldd = A.n;
  a.prev = prev;
  a.ldp = ldp;
  a.alpha = s.alpha;
  a.beta = s.beta;
  a.gamma = s.gamma;
  return launch<double, double, double, MODE_CSTEP>(a, st);
}

}  // namespace chfsi
