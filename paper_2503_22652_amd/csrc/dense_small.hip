// Small dense FP64 linear algebra of the Rayleigh-Ritz step (b x b, b up to a
// few thousand): blocked Cholesky, blocked triangular solve and a
// block-parallel Jacobi symmetric eigensolver.
//
// Rayleigh-Ritz (Algorithm 1, step 2) solves the projected pencil
// (Y^T A Y) E = (Y^T B Y) E Lambda.  The library reduces it with the Cholesky
// factor of the column-scaled Gram matrix Y^T B Y (CholQR) and diagonalises the
// resulting standard symmetric matrix with Jacobi rotations.
//
// Jacobi is chosen for the GPU because (i) a round of disjoint rotations is
// embarrassingly parallel, (ii) it converges quadratically when the matrix is
// nearly diagonal -- which is what the projected matrix becomes as subspace
// iteration converges -- and (iii) it is accurate to a small multiple of the
// unit roundoff.  The block variant pairs JB-wide column blocks (JB = 16) in a
// round-robin tournament, applies one inner sweep of rotations to every
// JP x JP pair subproblem (JP = 2 JB = 32) in LDS (one workgroup each, waves
// specialised so that a round costs one barrier: the next round's rotations,
// this round's update, the accumulation of U), and applies the resulting
// orthogonal JP x JP factors to the rest of the matrix and to the eigenvector
// accumulator with MFMA, in one launch per outer round.  Sweeps repeat until no
// rotation is applied or a cap of 40 sweeps is reached (then reported).
#include "internal.h"

#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <utility>
#include <vector>

namespace chfsi {

namespace {

constexpr int NB = 64;          // Cholesky / TRSM block
constexpr int kCholTiles = 8;   // 16-row tiles of the largest one-workgroup Cholesky (LDS)
constexpr int JB = 16;          // Jacobi column block
constexpr int JP = 2 * JB;      // Jacobi pair subproblem size
constexpr int LDJ = JP + 1;     // padded LDS leading dimension

// Cholesky factor L and its inverse of one matrix of up to 16 NT rows, in one
// workgroup of eight waves, the matrix in LDS in 16 x 16 tiles (padded with the
// identity).  Per tile column: wave 0 factors and inverts the 16 x 16 diagonal tile
// in registers (lane i holds row i; the pivots and the entries of L travel by
// readlane; 1/sqrt(d) from the hardware estimate and one step of third order), all waves
// form the tiles below with the inverse and update the trailing tiles on
// v_mfma_f64_16x16x4.  Then each wave forms the inverse's tiles of one tile column
// from the top down, Linv_ij = -Linv_ii sum_k L_ik Linv_kj (the sum's accumulator has
// the right operand's layout).  L fills the lower triangle of the LDS matrix, L^{-1}
// transposed the strictly upper one, its diagonal an array of its own.
// A chain of dependent FP64 operations bounds it (16 pivots a tile).  Straight-line
// code over all 64 columns in one wave, 53 us for 64 rows, spent its time fetching
// instructions; this takes 33 us for 64 rows, and
// 42 us for 80 with the whole inverse (before, two such blocks and a dozen products
// and copies).
//   A (lda): jb x jb in, L out (upper part zeroed).  Li (li_n x li_n, ldi): L^{-1},
// identity-padded past jb.  A pivot that is not above piv_tol (or not finite) sets
// *info to j0 + its 1-based column, and nothing is written.
typedef double chol_f64x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ double readlane_f64(double v, int lane) {
  const unsigned long long u = __double_as_longlong(v);
  const unsigned lo = __builtin_amdgcn_readlane(unsigned(u), lane);
  const unsigned hi = __builtin_amdgcn_readlane(unsigned(u >> 32), lane);
  return __longlong_as_double((static_cast<unsigned long long>(hi) << 32) | lo);
}

// 1/sqrt(x) for normal x > 0: the hardware estimate (within 2^-24) and one step of
// third order, y (1 + e/2 + 3 e^2 / 8) with e = 1 - x y^2
__device__ __forceinline__ double rsqrt_f64(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double e = fma(-(x * y), y, 1.0);
  return fma(y * e, fma(0.375, e, 0.5), y);
}

template <int NT>
__global__ __launch_bounds__(512) void k_chol_inv(double* A, int64_t lda, int jb, int* info, int j0,
                                                  double* Li, int64_t ldi, int li_n,
                                                  double piv_tol) {
  constexpr int LD = 16 * NT + 1;
  __shared__ double S[16 * NT * LD];
  __shared__ double invd[16 * NT];
  __shared__ int bad;
  if (*info != 0) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l16 = lane & 15, g = lane >> 4;
  const int nt = (std::max(jb, li_n) + 15) / 16, np = 16 * nt;
  if (tid == 0) bad = 0;
  for (int idx = tid; idx < np * np; idx += 512) {
    const int i = idx % np, j = idx / np;
    S[i + j * LD] = (i < jb && j < jb) ? (i >= j ? A[i + j * lda] : 0.0) : (i == j ? 1.0 : 0.0);
  }
  __syncthreads();
  // entry (i, k) of the inverse of diagonal tile t
  auto inv_diag = [&](int t, int i, int k) __attribute__((always_inline)) {
    const double up = S[(16 * t + k) + (16 * t + i) * LD];
    return k < i ? up : (k == i ? invd[16 * t + i] : 0.0);
  };
  for (int p = 0; p < nt; ++p) {
    const int c0 = 16 * p;
    if (wave == 0) {
      double r[16], x[16], gd[16];
#pragma unroll
      for (int j = 0; j < 16; ++j) r[j] = S[(c0 + l16) + (c0 + j) * LD];
      int failed = -1;
#pragma unroll
      for (int k = 0; k < 16; ++k) {
        const double d = readlane_f64(r[k], k);
        if (failed < 0 && (!(d > piv_tol) || !isfinite(d))) failed = k;
        gd[k] = rsqrt_f64(d);
        const double l = l16 == k ? d * gd[k] : r[k] * gd[k];
        r[k] = l;
#pragma unroll
        for (int j = k + 1; j < 16; ++j) r[j] = fma(-l, readlane_f64(l, j), r[j]);
      }
      if (failed >= 0) {
        if (lane == 0) {
          bad = 1;
          atomicCAS(info, 0, j0 + c0 + failed + 1);
        }
      } else {
        // column l16 of the tile's inverse
#pragma unroll
        for (int k = 0; k < 16; ++k) {
          double s0 = l16 == k ? 1.0 : 0.0, s1 = 0.0;
#pragma unroll
          for (int j = 0; j < k; ++j) {
            const double lkj = readlane_f64(r[j], k);
            if (j & 1)
              s1 = fma(-lkj, x[j], s1);
            else
              s0 = fma(-lkj, x[j], s0);
          }
          x[k] = (s0 + s1) * gd[k];
        }
        if (lane < 16) {
#pragma unroll
          for (int j = 0; j < 16; ++j) {
            if (j <= l16) S[(c0 + l16) + (c0 + j) * LD] = r[j];
            // Linv(j, l16), j > l16, transposed
            if (j > l16) S[(c0 + l16) + (c0 + j) * LD] = x[j];
          }
#pragma unroll
          for (int j = 0; j < 16; ++j)
            if (j == l16) invd[c0 + j] = x[j];
        }
      }
    }
    __syncthreads();
    if (bad) return;
    // the tiles below: L_tp = A_tp Linv_pp^T
    for (int t = p + 1 + wave; t < nt; t += 8) {
      chol_f64x4 acc = {0.0, 0.0, 0.0, 0.0};
      double a[4], b[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        a[q] = S[(16 * t + l16) + (c0 + 4 * q + g) * LD];
        b[q] = inv_diag(p, l16, 4 * q + g);
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[q], b[q], acc, 0, 0, 0);
#pragma unroll
      for (int q = 0; q < 4; ++q) S[(16 * t + g + 4 * q) + (c0 + l16) * LD] = acc[q];
    }
    __syncthreads();
    // the trailing tiles: A_ts -= L_tp L_sp^T
    const int m = nt - 1 - p, ntile = m * (m + 1) / 2;
    for (int u = wave; u < ntile; u += 8) {
      int ti = 0, rem = u;
      while (rem > ti) {
        rem -= ti + 1;
        ++ti;
      }
      const int rt = 16 * (p + 1 + ti), ct = 16 * (p + 1 + rem);
      chol_f64x4 acc = {0.0, 0.0, 0.0, 0.0};
      double a[4], b[4], o[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        a[q] = S[(rt + l16) + (c0 + 4 * q + g) * LD];
        b[q] = S[(ct + l16) + (c0 + 4 * q + g) * LD];
        o[q] = S[(rt + g + 4 * q) + (ct + l16) * LD];
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[q], b[q], acc, 0, 0, 0);
#pragma unroll
      for (int q = 0; q < 4; ++q) S[(rt + g + 4 * q) + (ct + l16) * LD] = o[q] - acc[q];
    }
    __syncthreads();
  }
  // the inverse's tiles below the diagonal, tile column j by wave j (its own
  // results only: no barrier)
  for (int j = wave; j < nt; j += 8) {
    for (int i = j + 1; i < nt; ++i) {
      chol_f64x4 acc = {0.0, 0.0, 0.0, 0.0};
      for (int k = j; k < i; ++k) {
        double a[4], b[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int kk = 4 * q + g;
          a[q] = S[(16 * i + l16) + (16 * k + kk) * LD];
          b[q] = k == j ? inv_diag(j, kk, l16) : S[(16 * j + l16) + (16 * k + kk) * LD];
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
          acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[q], b[q], acc, 0, 0, 0);
      }
      chol_f64x4 o = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int q = 0; q < 4; ++q)
        o = __builtin_amdgcn_mfma_f64_16x16x4f64(inv_diag(i, l16, 4 * q + g), -acc[q], o, 0, 0, 0);
#pragma unroll
      for (int q = 0; q < 4; ++q) S[(16 * j + l16) + (16 * i + g + 4 * q) * LD] = o[q];
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    }
  }
  __syncthreads();
  for (int idx = tid; idx < jb * jb; idx += 512) {
    const int i = idx % jb, j = idx / jb;
    A[i + j * lda] = i >= j ? S[i + j * LD] : 0.0;
  }
  for (int idx = tid; idx < li_n * li_n; idx += 512) {
    const int i = idx % li_n, j = idx / li_n;
    Li[i + j * ldi] = i > j ? S[j + i * LD] : (i == j ? invd[i] : 0.0);
  }
}

__global__ __launch_bounds__(256) void k_zero_upper(double* A, int64_t lda, int64_t b) {
  const int64_t total = b * b;
  for (int64_t idx = blockIdx.x * int64_t(256) + threadIdx.x; idx < total;
       idx += int64_t(gridDim.x) * 256) {
    const int64_t i = idx % b, j = idx / b;
    if (i < j) A[i + j * lda] = 0.0;
  }
}

// ---------------------------------------------------------------------------
// Jacobi
// ---------------------------------------------------------------------------
// round-robin ("circle") schedule: n players (even), round r in [0, n-1),
// slot 0 fixed, slots 1..n-1 rotate; pair k joins slots k and n-1-k.
__device__ __forceinline__ int rr_slot(int slot, int r, int n) {
  return slot == 0 ? 0 : 1 + (slot - 1 + r) % (n - 1);
}

typedef double f64x4_t __attribute__((ext_vector_type(4)));

// Block indices of pair k in round r of the block tournament (nblk blocks).
__device__ __forceinline__ void block_pair(int k, int r, int nblk, int* I, int* J) {
  int a = rr_slot(k, r, nblk), b = rr_slot(nblk - 1 - k, r, nblk);
  *I = a < b ? a : b;
  *J = a < b ? b : a;
}

// index of local row l (0..JP-1) of pair (I,J) in the padded matrix
__device__ __forceinline__ int pair_index(int l, int I, int J) {
  return l < JB ? I * JB + l : J * JB + (l - JB);
}

// ---------------------------------------------------------------------------
// Pair subproblem, wave-specialised (one sweep of JP - 1 rounds, one barrier
// per round).
// Round r of the circle schedule pairs slots (k, JP-1-k), k < JP/2; between
// rounds every index moves from slot s to slot sigma(s) = s - 1 (1 -> JP-1,
// slot 0 fixed).  The subproblem is therefore stored by slot, not by index:
// round r reads LDS buffer r % 2 and writes the shifted entries into buffer
// (r + 1) % 2, so every thread touches the same addresses in every round and
// no index arithmetic remains inside the loop.  Only the lower triangle (in
// slot order) is kept.  The rotation of pair k acts on (first, second) =
// (slot k, slot JP-1-k): J = [[c, s], [-s, c]], a <- J^T a J.
//  * wave 0, lane k < JP/2: the rotation of pair k in the NEXT round.  The
//    three entries it needs after this round are formed with the same arithmetic
//    (rot_entry, rot_block, same operand order) as in the update waves, so they are
//    bit-identical to what those waves store: the diagonal, kept in registers and moved
//    on between lanes, and one entry of this round's buffer.
//  * waves 1..3 (k1 >= k2 of 16 x 16 pair blocks, 136 threads): this round's
//    two-sided update of one 2 x 2 block each.
//  * waves 4..7, 16 lanes a row: two rows of the accumulated rotation U, by slot, in
//    registers; the slots move on between lanes.
// Wave 0's chain (barrier, LDS, one entry, two square roots) bounds a round.  Unrolled
// loops (25 KB of code for U, 60 KB for wave 0), with all of it in LDS, took 15.8 us a
// launch on average at 80 columns and 18.8 at 300; so it takes 12.2 and 14.9.
// ---------------------------------------------------------------------------
constexpr int kHalf = JP / 2;       // rotations per round
constexpr int kRounds = JP - 1;     // rounds per sweep
constexpr int kPairThreads = 8 * 64;

// lower-triangle LDS offset of symmetric entry (i, j) (slot coordinates)
__device__ __forceinline__ int sym_idx(int i, int j) { return i >= j ? i + j * LDJ : j + i * LDJ; }
// slot of an index after one round
__device__ __forceinline__ int slot_next(int s) { return s == 0 ? 0 : (s == 1 ? JP - 1 : s - 1); }
// out = J1^T X J2 for the 2 x 2 block X (rows first/second of pair 1,
// columns first/second of pair 2); explicit fma so that every caller rounds
// alike
__device__ __forceinline__ void rot_block(double x11, double x12, double x21, double x22,
                                          double c1, double s1, double c2, double s2,
                                          double* o11, double* o12, double* o21, double* o22) {
  const double y11 = fma(c1, x11, -(s1 * x21)), y12 = fma(c1, x12, -(s1 * x22));
  const double y21 = fma(s1, x11, c1 * x21), y22 = fma(s1, x12, c1 * x22);
  *o11 = fma(c2, y11, -(s2 * y12));
  *o12 = fma(s2, y11, c2 * y12);
  *o21 = fma(c2, y21, -(s2 * y22));
  *o22 = fma(s2, y21, c2 * y22);
}

// one output of rot_block with the same operations: (p1, q1) = (c1, -s1) for a first
// row, (s1, c1) for a second one, (p2, q2) likewise for the column
__device__ __forceinline__ double rot_entry(double x11, double x12, double x21, double x22,
                                            double p1, double q1, double p2, double q2) {
  const double y1 = fma(p1, x11, q1 * x21), y2 = fma(p1, x12, q1 * x22);
  return fma(p2, y1, q2 * y2);
}

// rotation (c, s) with J^T [[app, apq], [apq, aqq]] J diagonal (apq != 0):
// t = tan(phi) = sign(d) e / (|d| + sqrt(d^2 + e^2)), d = aqq - app, e = 2 apq,
// c = 1 / sqrt(1 + t^2), s = t c -- written with g = |d| + sqrt(d^2 + e^2) as
// c = g / sqrt(g^2 + e^2), s = sign(d) e / sqrt(g^2 + e^2), two square roots
// and no division.  Outside the range where d^2 + e^2 is a normal number the
// textbook form with divisions is used.
// No rotation (c = 1, s = 0) at |apq| <= thresh.
__device__ __forceinline__ void jacobi_cs(double app, double aqq, double apq, double thresh,
                                          double* c, double* s) {
  const double d = aqq - app, e = 2.0 * apq;
  const double e2 = e * e, h2 = fma(e, e, d * d);
  const double g = fma(h2, rsqrt_f64(h2), fabs(d));
  const double r = rsqrt_f64(fma(g, g, e2));
  const bool rot = fabs(apq) > thresh, normal = h2 > 1e-300 && h2 < 1e300;
  double cc = g * r, ss = (d < 0.0 ? -e : e) * r;
  if (__builtin_expect(rot && !normal, 0)) {
    const double theta = d / e;
    const double t = fabs(theta) > 1e150
                         ? 0.5 / theta
                         : copysign(1.0, theta) / (fabs(theta) + sqrt(theta * theta + 1.0));
    cc = 1.0 / sqrt(t * t + 1.0);
    ss = t * cc;
  }
  *c = rot ? cc : 1.0;
  *s = rot ? ss : 0.0;
}

// LDS of one pair subproblem: the slot-ordered lower triangle (ping-pong
// buffers), the rotations of the current and next round, the wave maxima
struct PairSmem {
  double buf[2][JP * LDJ];
  double2 cs[2][kHalf];
  double wmax[kPairThreads / 64];
  int nrot_total;
};

// value of lane + 1 (shl) or lane - 1 (shr) within each 16 lanes, `edge` in the last
// (first) of them
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double edge, double v) {
  const unsigned long long o = __double_as_longlong(edge), u = __double_as_longlong(v);
  const unsigned lo = __builtin_amdgcn_update_dpp(int(o), int(u), CTRL, 0xf, 0xf, false);
  const unsigned hi =
      __builtin_amdgcn_update_dpp(int(o >> 32), int(u >> 32), CTRL, 0xf, 0xf, false);
  return __longlong_as_double((static_cast<unsigned long long>(hi) << 32) | lo);
}
__device__ __forceinline__ double lane_shl(double edge, double v) { return dpp_f64<0x101>(edge, v); }
__device__ __forceinline__ double lane_shr(double edge, double v) { return dpp_f64<0x111>(edge, v); }

// lane k of 16 holds the values in slots k (v1) and JP - 1 - k (v2): move them on by
// one round
__device__ __forceinline__ void slot_shift(int k, double* v1, double* v2) {
  const double up = lane_shl(*v2, *v1);    // from slot k + 1
  *v2 = lane_shr(up, *v2);                 // from slot JP - k; pair 0's from slot 1
  *v1 = k == 0 ? *v1 : up;
}

// One inner sweep of the pair subproblem held in S.buf[0] (lower triangle,
// local order = slot order of round 0); `mx` is this thread's largest
// off-diagonal magnitude among the entries it stored.  Skips (skip_out = 1)
// when the subproblem is already diagonal to the threshold, else writes the
// accumulated JP x JP rotation to Uo (skip_out = 0) and adds its rotation
// count to the sweep counter.
__device__ __forceinline__ void pair_solve_core(PairSmem& S, double mx, const double* scale,
                                                double tol, double* Uo, int* skip_out,
                                                int* counter) {
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  auto& buf = S.buf;
  auto& cs = S.cs;
  auto& wmax = S.wmax;
  int& nrot_total = S.nrot_total;
  for (int off = 32; off > 0; off >>= 1) mx = fmax(mx, __shfl_xor(mx, off));
  if (lane == 0) wmax[wave] = mx;
  if (tid == 0) nrot_total = 0;
  __syncthreads();
  mx = wmax[0];
#pragma unroll
  for (int w = 1; w < kPairThreads / 64; ++w) mx = fmax(mx, wmax[w]);
  const double thresh = tol * (*scale);
  if (!(mx > thresh)) {
    if (tid == 0) *skip_out = 1;
    return;
  }
  // wave 0, every 16 lanes alike: lane k holds its pair's three entries (diagonal d1,
  // d2, off-diagonal od) and rotation
  const int k = lane & (kHalf - 1);
  double d1 = 0.0, d2 = 0.0, od = 0.0, c = 1.0, sn = 0.0;
  if (wave == 0) {
    const int s = JP - 1 - k;
    d1 = buf[0][sym_idx(k, k)];
    d2 = buf[0][sym_idx(s, s)];
    od = buf[0][sym_idx(s, k)];
    jacobi_cs(d1, d2, od, thresh, &c, &sn);
    if (lane < kHalf) cs[0][lane] = make_double2(c, sn);
  }
  __syncthreads();
  if (wave == 0) {
    // next-round pair k joins this round's slots h and l, of the pairs k + 1 (15: its
    // own) and k - 1 (0: its own); entry (h, l) is one of that block pair's four
    const int kh = k < kHalf - 1 ? k + 1 : k, kl = k > 0 ? k - 1 : 0;
    const int fh = kh, sh = JP - 1 - kh, fl = kl, sl = JP - 1 - kl;
    const int b11 = sym_idx(fh, fl), b12 = sym_idx(fh, sl), b21 = sym_idx(sh, fl),
              b22 = sym_idx(sh, sl);
    int count = sn != 0.0;
    // the chain that bounds the kernel: first on its SIMD
    __builtin_amdgcn_s_setprio(3);
#pragma unroll 1
    for (int r = 0; r + 1 < kRounds; ++r) {
      const double* a = buf[r & 1];
      const double x11 = a[b11], x12 = a[b12], x21 = a[b21], x22 = a[b22];
      // row factors of h: (c, -s) of a first slot, (s, c) of a second one; columns of l
      const double ph = lane_shl(sn, c), qh = lane_shl(c, -sn);
      const double pl = lane_shr(c, sn), ql = lane_shr(-sn, c);
      double o12, o21, n1, n2;
      rot_block(d1, od, od, d2, c, sn, c, sn, &n1, &o12, &o21, &n2);
      slot_shift(k, &n1, &n2);
      d1 = n1;
      d2 = n2;
      od = rot_entry(x11, x12, x21, x22, ph, qh, pl, ql);
      jacobi_cs(d1, d2, od, thresh, &c, &sn);
      if (lane < kHalf) cs[(r + 1) & 1][lane] = make_double2(c, sn);
      count += sn != 0.0;
      __syncthreads();
    }
    __builtin_amdgcn_s_setprio(0);
    __syncthreads();
    if (lane < kHalf && count > 0) atomicAdd(&nrot_total, count);
  } else if (wave < 4) {
    // block (k1, k2), k1 >= k2, of the 16 x 16 pair blocks (136 of 192 threads)
    const int idx = tid - 64;
    int k1 = 0, k2 = 0;
    {
      int rem = idx;
      while (k1 < kHalf && rem > k1) {
        rem -= k1 + 1;
        ++k1;
      }
      k2 = rem;
    }
    const bool active = idx < kHalf * (kHalf + 1) / 2;
    const int f1 = k1, s1 = JP - 1 - k1, f2 = k2, s2 = JP - 1 - k2;
    const int i11 = sym_idx(f1, f2), i12 = sym_idx(f1, s2), i21 = sym_idx(s1, f2),
              i22 = sym_idx(s1, s2);
    const int o11i = sym_idx(slot_next(f1), slot_next(f2)),
              o12i = sym_idx(slot_next(f1), slot_next(s2)),
              o21i = sym_idx(slot_next(s1), slot_next(f2)),
              o22i = sym_idx(slot_next(s1), slot_next(s2));
#pragma unroll 1
    for (int r = 0; r < kRounds; ++r) {
      if (active) {
        const double* a = buf[r & 1];
        double* o = buf[(r + 1) & 1];
        const double2 t1 = cs[r & 1][k1], t2 = cs[r & 1][k2];
        const double x21 = a[i21];       // a pair's own block: entry (1, 2) is the same one
        double v11, v12, v21, v22;
        rot_block(a[i11], a[i12], x21, a[i22], t1.x, t1.y, t2.x, t2.y, &v11, &v12, &v21, &v22);
        if (k1 == k2) v12 = v21 = t1.y != 0.0 ? 0.0 : x21;
        o[o11i] = v11;
        o[o12i] = v12;
        o[o21i] = v21;
        o[o22i] = v22;
      }
      __syncthreads();
    }
  } else {
    // rows i and i + JP / 2 of U, columns by slot (after kRounds shifts slot = index)
    const int i = 4 * (wave - 4) + (lane >> 4);
    double ua1 = i == k, ua2 = 0.0, ub1 = 0.0, ub2 = i + kHalf == JP - 1 - k;
#pragma unroll 1
    for (int r = 0; r < kRounds; ++r) {
      const double2 t = cs[r & 1][k];
      const double na1 = fma(t.x, ua1, -(t.y * ua2)), na2 = fma(t.y, ua1, t.x * ua2);
      const double nb1 = fma(t.x, ub1, -(t.y * ub2)), nb2 = fma(t.y, ub1, t.x * ub2);
      ua1 = na1;
      ua2 = na2;
      ub1 = nb1;
      ub2 = nb2;
      slot_shift(k, &ua1, &ua2);
      slot_shift(k, &ub1, &ub2);
      __syncthreads();
    }
    // into LDS (the subproblem itself is no longer needed)
    buf[0][i + k * LDJ] = ua1;
    buf[0][i + (JP - 1 - k) * LDJ] = ua2;
    buf[0][i + kHalf + k * LDJ] = ub1;
    buf[0][i + kHalf + (JP - 1 - k) * LDJ] = ub2;
  }
  __syncthreads();
  for (int idx = tid; idx < JP * JP; idx += kPairThreads) {
    const int i = idx % JP, j = idx / JP;
    Uo[i + j * JP] = buf[0][i + j * LDJ];
  }
  if (tid == 0) {
    *skip_out = 0;
    if (nrot_total > 0) atomicAdd(counter, nrot_total);
  }
}

// One workgroup per pair of the outer round: gather the JP x JP subproblem,
// skip it when already diagonal (to the threshold), else one Jacobi sweep.
// Writes U (JP x JP) and skip[pair] (1 = U is the identity).
__global__ __launch_bounds__(kPairThreads) void k_jacobi_pair_solve(
    const double* A, int64_t lda, int nblk, int round, const double* scale, double tol, double* U,
    int* skip, int* counter) {
  __shared__ PairSmem S;
  const int tid = threadIdx.x;
  int I, J;
  block_pair(blockIdx.x, round, nblk, &I, &J);
  // round 0 has index s in slot s
  double mx = 0.0;
  for (int idx = tid; idx < JP * JP; idx += kPairThreads) {
    const int i = idx % JP, j = idx / JP;
    if (i < j) continue;
    const double v = A[pair_index(i, I, J) + int64_t(pair_index(j, I, J)) * lda];
    S.buf[0][i + j * LDJ] = v;
    if (i != j) mx = fmax(mx, fabs(v));
  }
  pair_solve_core(S, mx, scale, tol, U + int64_t(blockIdx.x) * JP * JP, skip + blockIdx.x,
                  counter);
}


// out = op(X) * Y for JP x JP matrices in LDS (ld LDJ) on FP64 MFMA
// (v_mfma_f64_16x16x4f64: lane l supplies X(l%16, l/16) and Y(l/16, l%16);
// output element r of lane l is row l/16 + 4r, column l%16).  Each of the
// four waves computes one JP/2 x JP/2 quadrant as NT x NT tiles of 16 x 16.
// TX: X is read transposed.
constexpr int NT = JP / 32;
template <bool TX>
__device__ __forceinline__ void lds_mm(const double* X, const double* Y, double out[NT][NT][4]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int qm = (wave & 1) * (JP / 2), qn = (wave >> 1) * (JP / 2);
  const int l16 = lane & 15, g = lane >> 4;
  f64x4_t acc[NT][NT];
#pragma unroll
  for (int i = 0; i < NT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[i][j] = f64x4_t{0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
  for (int k0 = 0; k0 < JP; k0 += 4) {
    const int k = k0 + g;
    double xa[NT], yb[NT];
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      const int m = qm + i * 16 + l16;
      xa[i] = TX ? X[k + m * LDJ] : X[m + k * LDJ];
    }
#pragma unroll
    for (int j = 0; j < NT; ++j) yb[j] = Y[k + (qn + j * 16 + l16) * LDJ];
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(xa[i], yb[j], acc[i][j], 0, 0, 0);
  }
#pragma unroll
  for (int i = 0; i < NT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) out[i][j][r] = acc[i][j][r];
}

// row / column (local) of output element r of tile (i, j) held by this lane
__device__ __forceinline__ int mm_row(int i, int r) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  return (wave & 1) * (JP / 2) + i * 16 + (lane >> 4) + 4 * r;
}
__device__ __forceinline__ int mm_col(int j) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  return (wave >> 1) * (JP / 2) + j * 16 + (lane & 15);
}

__device__ __forceinline__ void lds_mm_store(double* Z, const double v[NT][NT][4]) {
#pragma unroll
  for (int i = 0; i < NT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) Z[mm_row(i, r) + mm_col(j) * LDJ] = v[i][j][r];
}

__device__ __forceinline__ void load_u_or_identity(double* dst, const double* U, bool identity) {
  for (int idx = threadIdx.x; idx < JP * JP; idx += 256) {
    const int i = idx % JP, j = idx / JP;
    dst[i + j * LDJ] = identity ? (i == j ? 1.0 : 0.0) : U[i + j * JP];
  }
}

// The outer round's rotations, one launch: blockIdx.y < npairs updates the
// matrix block pair (P, Q) = (blockIdx.x, blockIdx.y), P >= Q:
// A[SP, SQ] <- U_P^T A[SP, SQ] U_Q, written with its transpose into A[SQ, SP];
// blockIdx.y >= npairs updates JP rows (chunk blockIdx.y - npairs) of the
// eigenvector accumulator: V[rows, SP] <- V[rows, SP] U_P.
__global__ __launch_bounds__(256) void k_jacobi_apply(double* A, int64_t lda, double* V,
                                                      int64_t ldv, int nblk, int npairs,
                                                      int round, const double* U,
                                                      const int* skip) {
  __shared__ double m[JP * LDJ];
  __shared__ double up[JP * LDJ];
  __shared__ double uq[JP * LDJ];
  const int P = blockIdx.x;
  int IP, JPb;
  block_pair(P, round, nblk, &IP, &JPb);
  double t[NT][NT][4];
  if (int(blockIdx.y) >= npairs) {
    if (skip[P]) return;
    const int64_t r0 = int64_t(blockIdx.y - npairs) * JP;
    for (int idx = threadIdx.x; idx < JP * JP; idx += 256) {
      const int i = idx % JP, j = idx / JP;
      m[i + j * LDJ] = V[r0 + i + int64_t(pair_index(j, IP, JPb)) * ldv];
    }
    load_u_or_identity(up, U + int64_t(P) * JP * JP, false);
    __syncthreads();
    lds_mm<false>(m, up, t);
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          V[r0 + mm_row(i, r) + int64_t(pair_index(mm_col(j), IP, JPb)) * ldv] = t[i][j][r];
    return;
  }
  const int Q = blockIdx.y;
  if (P < Q) return;
  const bool sp = skip[P] != 0, sq = skip[Q] != 0;
  if (sp && sq) return;
  int IQ, JQ;
  block_pair(Q, round, nblk, &IQ, &JQ);
  for (int idx = threadIdx.x; idx < JP * JP; idx += 256) {
    const int i = idx % JP, j = idx / JP;
    m[i + j * LDJ] = A[pair_index(i, IP, JPb) + int64_t(pair_index(j, IQ, JQ)) * lda];
  }
  load_u_or_identity(up, U + int64_t(P) * JP * JP, sp);
  load_u_or_identity(uq, U + int64_t(Q) * JP * JP, sq);
  __syncthreads();
  lds_mm<true>(up, m, t);         // U_P^T M
  __syncthreads();
  lds_mm_store(m, t);
  __syncthreads();
  lds_mm<false>(m, uq, t);        // (U_P^T M) U_Q
  __syncthreads();
  lds_mm_store(m, t);
  __syncthreads();
  for (int idx = threadIdx.x; idx < JP * JP; idx += 256) {
    const int i = idx % JP, j = idx / JP;
    A[pair_index(i, IP, JPb) + int64_t(pair_index(j, IQ, JQ)) * lda] = m[i + j * LDJ];
  }
  if (P != Q) {
    for (int idx = threadIdx.x; idx < JP * JP; idx += 256) {
      const int i = idx % JP, j = idx / JP;
      A[pair_index(i, IQ, JQ) + int64_t(pair_index(j, IP, JPb)) * lda] = m[j + i * LDJ];
    }
  }
}

// ---------------------------------------------------------------------------
// Pipelined outer rounds: one launch carries the pair solves of round r and
// the rotations of round r - 1.  The pair workgroups do not wait for the
// rotated matrix: each forms the three 16 x 16 blocks of it that its
// subproblem needs from the matrix before round r - 1 and that round's
// factors, with the same products in the same order as the rotation
// workgroups (so the entries are bit-identical to the ones those store),
// while the rotation workgroups write the rotated matrix into the other
// buffer.  A sweep of R rounds takes R + 1 launches instead of 2 R, and the
// rotations leave the critical path.
// ---------------------------------------------------------------------------

// pair of round r that holds block x, and x's offset (0 or JB) in it
__device__ __forceinline__ void block_locate(int x, int r, int nblk, int* pair, int* off) {
  const int n1 = nblk - 1;
  const int s = x == 0 ? 0 : 1 + ((x - 1 - r) % n1 + n1) % n1;
  const int k = s < nblk / 2 ? s : nblk - 1 - s;
  int I, J;
  block_pair(k, r, nblk, &I, &J);
  *pair = k;
  *off = x == I ? 0 : JB;
}

constexpr int LDZ = JB + 1;   // leading dimension of a 16-row slice in LDS

// rows oR..oR+15 of U_R^T M (both 16-column halves), M = A[S_R, S_C] (pair R
// rows (IR, JR), pair C columns (IC, JC)); operands from global memory with the
// values and the k order of lds_mm<true>(U_R, M).  idR: U_R is the identity.
__device__ __forceinline__ void rot_rows(const double* A, int64_t lda, const double* UR, bool idR,
                                         int oR, int IR, int JR, int IC, int JC, f64x4_t* acc0,
                                         f64x4_t* acc1) {
  const int lane = threadIdx.x & 63, l16 = lane & 15, g = lane >> 4;
  const int m = oR + l16;
  const int64_t col0 = int64_t(pair_index(l16, IC, JC)) * lda;
  const int64_t col1 = int64_t(pair_index(JB + l16, IC, JC)) * lda;
  double xa[JP / 4], y0[JP / 4], y1[JP / 4];
#pragma unroll
  for (int t = 0; t < JP / 4; ++t) {
    const int k = 4 * t + g;
    const int64_t row = pair_index(k, IR, JR);
    xa[t] = idR ? (k == m ? 1.0 : 0.0) : UR[k + m * JP];
    y0[t] = A[row + col0];
    y1[t] = A[row + col1];
  }
  f64x4_t a0 = {0.0, 0.0, 0.0, 0.0}, a1 = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int t = 0; t < JP / 4; ++t) {
    a0 = __builtin_amdgcn_mfma_f64_16x16x4f64(xa[t], y0[t], a0, 0, 0, 0);
    a1 = __builtin_amdgcn_mfma_f64_16x16x4f64(xa[t], y1[t], a1, 0, 0, 0);
  }
  *acc0 = a0;
  *acc1 = a1;
}

// U_C[:, oC..oC+15] in the lane order of the B operand of rot_cols
__device__ __forceinline__ void load_ucols(const double* UC, bool idC, int oC, double (&yb)[JP / 4]) {
  const int lane = threadIdx.x & 63, l16 = lane & 15, g = lane >> 4;
  const int n = oC + l16;
#pragma unroll
  for (int t = 0; t < JP / 4; ++t) {
    const int k = 4 * t + g;
    yb[t] = idC ? (k == n ? 1.0 : 0.0) : UC[k + n * JP];
  }
}

// the 16 x 16 tile Z U_C[:, oC..oC+15] for a 16-row slice Z (LDS, ld LDZ),
// with the values and the k order of lds_mm<false>(Z, U_C)
__device__ __forceinline__ f64x4_t rot_cols(const double* Z, const double (&yb)[JP / 4]) {
  const int lane = threadIdx.x & 63, l16 = lane & 15, g = lane >> 4;
  f64x4_t acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int t = 0; t < JP / 4; ++t) {
    const int k = 4 * t + g;
    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(Z[l16 + k * LDZ], yb[t], acc, 0, 0, 0);
  }
  return acc;
}

// the workgroup's largest of the threads' m (not NaN, not negative) into *out; every
// thread of the workgroup takes part.  red: one entry a wave
template <int THREADS>
__device__ __forceinline__ void publish_max(double m, double* red, unsigned long long* out) {
  for (int off = 32; off > 0; off >>= 1) m = fmax(m, __shfl_xor(m, off));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < THREADS / 64; ++w) m = fmax(m, red[w]);
    if (m > 0.0) atomicMax(out, static_cast<unsigned long long>(__double_as_longlong(m)));
  }
}

union RoundSmem {
  struct {
    PairSmem ps;
    double z[3][JP * LDZ];
  } pair;
  struct {
    double m[JP * LDJ];
    double up[JP * LDJ];
    double uq[JP * LDJ];
  } apply;
};

// Workgroups [0, npairs) (when rcur >= 0): pair solves of round rcur on the
// matrix after round rprev (rprev < 0: Pin itself).  The rest (when
// rprev >= 0): round rprev's rotations as in k_jacobi_apply, Pin -> Pout (a
// block both of whose factors are identities is copied), V in place; offmax (given in a
// sweep's last launch) collects the largest off-diagonal magnitude.
__global__ __launch_bounds__(kPairThreads) void k_jacobi_round(
    const double* __restrict__ Pin, double* __restrict__ Pout, int64_t lda, double* V,
    int64_t ldv, int nblk, int npairs, int rprev, const double* Uprev, const int* skipprev,
    int rcur, double* Ucur, int* skipcur, const double* scale, double tol, int* counter,
    unsigned long long* offmax) {
  __shared__ RoundSmem sm;
  __shared__ double red[kPairThreads / 64];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int npw = rcur >= 0 ? npairs : 0;
  if (int(blockIdx.x) < npw) {
    PairSmem& S = sm.pair.ps;
    int I, J;
    block_pair(blockIdx.x, rcur, nblk, &I, &J);
    double mx = 0.0;
    if (rprev < 0) {
      for (int idx = tid; idx < JP * JP; idx += kPairThreads) {
        const int i = idx % JP, j = idx / JP;
        if (i < j) continue;
        const double v = Pin[pair_index(i, I, J) + int64_t(pair_index(j, I, J)) * lda];
        S.buf[0][i + j * LDJ] = v;
        if (i != j) mx = fmax(mx, fabs(v));
      }
    } else {
      int pI, oI, pJ, oJ;
      block_locate(I, rprev, nblk, &pI, &oI);
      block_locate(J, rprev, nblk, &pJ, &oJ);
      // tile 0: (I, I); tile 1: (J, J); tile 2: the (J, I) block, formed as
      // the rotation workgroup of the pair with the larger index forms it
      const bool jrow = pJ > pI;
      auto tile = [&](int t, int* R, int* oR, int* C, int* oC) {
        if (t == 0) { *R = pI; *oR = oI; *C = pI; *oC = oI; }
        else if (t == 1) { *R = pJ; *oR = oJ; *C = pJ; *oC = oJ; }
        else if (jrow) { *R = pJ; *oR = oJ; *C = pI; *oC = oI; }
        else { *R = pI; *oR = oI; *C = pJ; *oC = oJ; }
      };
      // waves 0..2: tile `wave`; the right factor of the second product is
      // loaded with the first product's operands
      const int l16 = lane & 15, g = lane >> 4;
      const int t = wave;
      int R = 0, oR = 0, C = 0, oC = 0;
      double ucol[JP / 4];
      if (wave < 3) {
        tile(t, &R, &oR, &C, &oC);
        int IR, JR, IC, JC;
        block_pair(R, rprev, nblk, &IR, &JR);
        block_pair(C, rprev, nblk, &IC, &JC);
        load_ucols(Uprev + int64_t(C) * JP * JP, skipprev[C] != 0, oC, ucol);
        f64x4_t a0, a1;
        rot_rows(Pin, lda, Uprev + int64_t(R) * JP * JP, skipprev[R] != 0, oR, IR, JR, IC, JC,
                 &a0, &a1);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          sm.pair.z[t][(g + 4 * r) + l16 * LDZ] = a0[r];
          sm.pair.z[t][(g + 4 * r) + (JB + l16) * LDZ] = a1[r];
        }
      }
      __syncthreads();
      if (wave < 3) {
        const f64x4_t acc = rot_cols(sm.pair.z[t], ucol);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int a = g + 4 * r, bcol = l16;   // element (a, bcol) of the tile
          int i, j;                              // local (slot) coordinates
          if (t == 0) { i = a; j = bcol; }
          else if (t == 1) { i = JB + a; j = JB + bcol; }
          else if (jrow) { i = JB + a; j = bcol; }
          else { i = JB + bcol; j = a; }
          if (i < j) continue;
          S.buf[0][i + j * LDJ] = acc[r];
          if (i != j) mx = fmax(mx, fabs(acc[r]));
        }
      }
    }
    pair_solve_core(S, mx, scale, tol, Ucur + int64_t(blockIdx.x) * JP * JP,
                    skipcur + blockIdx.x, counter);
    return;
  }
  if (rprev < 0) return;
  // rotations of round rprev
  const int a = int(blockIdx.x) - npw;
  const int P = a % npairs, y = a / npairs;
  int IP, JPb;
  block_pair(P, rprev, nblk, &IP, &JPb);
  double* m = sm.apply.m;
  double* up = sm.apply.up;
  double* uq = sm.apply.uq;
  double t[NT][NT][4];
  if (y >= npairs) {
    if (skipprev[P]) return;
    const int64_t r0 = int64_t(y - npairs) * JP;
    for (int idx = tid; idx < JP * JP; idx += kPairThreads) {
      const int i = idx % JP, j = idx / JP;
      m[i + j * LDJ] = V[r0 + i + int64_t(pair_index(j, IP, JPb)) * ldv];
      up[i + j * LDJ] = Uprev[int64_t(P) * JP * JP + i + j * JP];
    }
    __syncthreads();
    if (wave < 4) {
      lds_mm<false>(m, up, t);
#pragma unroll
      for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            V[r0 + mm_row(i, r) + int64_t(pair_index(mm_col(j), IP, JPb)) * ldv] = t[i][j][r];
    }
    return;
  }
  const int Q = y;
  if (P < Q) return;
  const bool sp = skipprev[P] != 0, sq = skipprev[Q] != 0;
  int IQ, JQ;
  block_pair(Q, rprev, nblk, &IQ, &JQ);
  double mx = 0.0;
  if (sp && sq) {
    for (int idx = tid; idx < JP * JP; idx += kPairThreads) {
      const int i = idx % JP, j = idx / JP;
      const int64_t o1 = pair_index(i, IP, JPb) + int64_t(pair_index(j, IQ, JQ)) * lda;
      const double v = Pin[o1];
      Pout[o1] = v;
      if (P != Q) {
        const int64_t o2 = pair_index(i, IQ, JQ) + int64_t(pair_index(j, IP, JPb)) * lda;
        Pout[o2] = Pin[o2];
      }
      if (P != Q || i != j) mx = fmax(mx, fabs(v));
    }
    if (offmax) publish_max<kPairThreads>(mx, red, offmax);
    return;
  }
  for (int idx = tid; idx < JP * JP; idx += kPairThreads) {
    const int i = idx % JP, j = idx / JP;
    m[i + j * LDJ] = Pin[pair_index(i, IP, JPb) + int64_t(pair_index(j, IQ, JQ)) * lda];
    up[i + j * LDJ] = sp ? (i == j ? 1.0 : 0.0) : Uprev[int64_t(P) * JP * JP + i + j * JP];
    uq[i + j * LDJ] = sq ? (i == j ? 1.0 : 0.0) : Uprev[int64_t(Q) * JP * JP + i + j * JP];
  }
  __syncthreads();
  if (wave < 4) lds_mm<true>(up, m, t);         // U_P^T M
  __syncthreads();
  if (wave < 4) lds_mm_store(m, t);
  __syncthreads();
  if (wave < 4) lds_mm<false>(m, uq, t);        // (U_P^T M) U_Q
  __syncthreads();
  if (wave < 4) lds_mm_store(m, t);
  __syncthreads();
  for (int idx = tid; idx < JP * JP; idx += kPairThreads) {
    const int i = idx % JP, j = idx / JP;
    const double v = m[i + j * LDJ];
    Pout[pair_index(i, IP, JPb) + int64_t(pair_index(j, IQ, JQ)) * lda] = v;
    if (P != Q) Pout[pair_index(j, IQ, JQ) + int64_t(pair_index(i, IP, JPb)) * lda] = v;
    if (P != Q || i != j) mx = fmax(mx, fabs(v));
  }
  if (offmax) publish_max<kPairThreads>(mx, red, offmax);
}

// padded copy of the symmetrised matrix, P (bp x bp) = [(A + A^T) / 2, 0; 0, 0], V = I,
// and each workgroup's partial sum of squares
constexpr int kFroParts = 256;
__global__ __launch_bounds__(256) void k_jacobi_setup(const double* A, int64_t lda, int64_t b,
                                                      double* P, double* V, int64_t bp,
                                                      double* part) {
  __shared__ double red[256];
  const int64_t total = bp * bp;
  double s = 0.0;
  for (int64_t idx = blockIdx.x * int64_t(256) + threadIdx.x; idx < total;
       idx += int64_t(gridDim.x) * 256) {
    const int64_t j = idx / bp, i = idx - j * bp;
    double v = 0.0;
    if (i < b && j < b) v = i == j ? A[i + j * lda] : 0.5 * (A[i + j * lda] + A[j + i * lda]);
    P[idx] = v;
    V[idx] = (i == j) ? 1.0 : 0.0;
    s += v * v;
  }
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

// the Frobenius norm from the partial sums (in a fixed order), and the sweep's rotation
// count and largest off-diagonal magnitude cleared
__global__ __launch_bounds__(64) void k_jacobi_begin(const double* part, double* out, int* counter,
                                                     unsigned long long* offmax) {
  double s = 0.0;
#pragma unroll
  for (int i = 0; i < kFroParts / 64; ++i) s += part[threadIdx.x + 64 * i];
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
  if (threadIdx.x == 0) {
    *out = sqrt(s) > 0 ? sqrt(s) : 1.0;
    *counter = 0;
    *offmax = 0;
  }
}

// a sweep's end: flags[0] = rotations, flags[1] = 1 if no off-diagonal magnitude is above
// thresh_rel * scal[0] (the Frobenius norm); both sources cleared for the next sweep.
// flags may be pinned host memory
__global__ __launch_bounds__(64) void k_sweep_end(const double* scal, double thresh_rel,
                                                  int* counter, unsigned long long* offmax,
                                                  int* flags) {
  if (threadIdx.x == 0) {
    flags[0] = *counter;
    flags[1] = __longlong_as_double(*offmax) <= thresh_rel * scal[0] ? 1 : 0;
    *counter = 0;
    *offmax = 0;
  }
}

// largest off-diagonal magnitude of the bp x bp matrix into *offmax (the rounds without
// the pipeline; else the last round's rotations collect it)
__global__ __launch_bounds__(256) void k_offmax(const double* P, int64_t bp,
                                                unsigned long long* offmax) {
  __shared__ double red[4];
  double m = 0.0;
  for (int64_t idx = blockIdx.x * int64_t(256) + threadIdx.x; idx < bp * bp;
       idx += int64_t(gridDim.x) * 256) {
    const int64_t j = idx / bp, i = idx - j * bp;
    if (i != j) m = fmax(m, fabs(P[idx]));
  }
  publish_max<256>(m, red, offmax);
}

// ascending sort of the diagonal (first b entries) by rank counting: one workgroup per
// entry finds its rank and moves its eigenvector column
__global__ __launch_bounds__(256) void k_jacobi_sort(const double* P, const double* V, int64_t bp,
                                                     int64_t b, double* w, double* out,
                                                     int64_t ldo) {
  __shared__ int cnt[4];
  const int64_t j = blockIdx.x;
  const double dj = P[j + j * bp];
  int c = 0;
  for (int64_t t = threadIdx.x; t < b; t += 256) {
    const double dt = P[t + t * bp];
    c += (dt < dj) || (dt == dj && t < j);
  }
  for (int off = 32; off > 0; off >>= 1) c += __shfl_xor(c, off);
  if ((threadIdx.x & 63) == 0) cnt[threadIdx.x >> 6] = c;
  __syncthreads();
  const int64_t rank = cnt[0] + cnt[1] + cnt[2] + cnt[3];
  if (threadIdx.x == 0) w[rank] = dj;
  for (int64_t i = threadIdx.x; i < b; i += 256) out[i + rank * ldo] = V[i + j * bp];
}

inline int64_t grid_for(int64_t total) {
  int64_t g = (total + 255) / 256;
  return std::max<int64_t>(1, std::min<int64_t>(g, 65536));
}

}  // namespace

size_t potrf_workspace_bytes(int64_t b) { return gemm_workspace_bytes(b, b, NB, sizeof(double)); }

size_t tri_workspace_bytes(int64_t b, int64_t nrhs) {
  const int64_t nblk = (b + NB - 1) / NB;
  return size_t(nblk * NB * NB + NB * std::max(b, nrhs)) * sizeof(double);
}

bool potrf_inverse_fits(int64_t b) { return b <= 16 * kCholTiles; }

hipError_t potrf_inverse(double* A, int64_t lda, int64_t b, int* info, double* Linv, int64_t ldi,
                         hipStream_t st, double piv_tol) {
  if (!potrf_inverse_fits(b)) return hipErrorInvalidValue;
  if (b <= NB)
    k_chol_inv<NB / 16><<<1, 512, 0, st>>>(A, lda, int(b), info, 0, Linv, ldi, int(b), piv_tol);
  else
    k_chol_inv<kCholTiles><<<1, 512, 0, st>>>(A, lda, int(b), info, 0, Linv, ldi, int(b), piv_tol);
  return hipGetLastError();
}

// Blocked right-looking Cholesky.  Per diagonal block: factor it in LDS,
// invert it (kept in tri for trsm_lower_left), form the panel below as a GEMM
// with the inverse, then update the trailing matrix with a GEMM.
hipError_t potrf_lower(double* A, int64_t lda, int64_t b, int* info, hipStream_t st,
                       const Workspace& ws, double* tri, double piv_tol) {
  hipError_t e = hipSuccess;
  const int64_t nblk = (b + NB - 1) / NB;
  double* tmp = tri + nblk * NB * NB;
  for (int64_t j0 = 0; j0 < b; j0 += NB) {
    const int jb = int(std::min<int64_t>(NB, b - j0));
    double* Li = tri + (j0 / NB) * NB * NB;
    k_chol_inv<NB / 16><<<1, 512, 0, st>>>(A + j0 + j0 * lda, lda, jb, info, int(j0), Li, NB, NB,
                                           piv_tol);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    const int64_t rows = b - j0 - jb;
    if (rows <= 0) break;
    {   // tmp (rows x jb) = A21 L11^{-T}; A21 <- tmp
      GemmDesc<double> g;
      g.M = rows;
      g.N = jb;
      g.K = jb;
      g.A = A + (j0 + jb) + j0 * lda;
      g.sam = 1;
      g.sak = lda;
      g.B = Li;           // B(k, n) = L11^{-1}(n, k)
      g.sbn = 1;
      g.sbk = NB;
      g.C = tmp;
      g.ldc = rows;
      if ((e = gemm<double>(g, st, ws, 1)) != hipSuccess) return e;
      if ((e = copy_block(tmp, rows, A + (j0 + jb) + j0 * lda, lda, rows, jb, st)) != hipSuccess)
        return e;
    }
    // A22 -= L21 L21^T
    GemmDesc<double> g;
    g.M = rows;
    g.N = rows;
    g.K = jb;
    g.A = A + (j0 + jb) + j0 * lda;
    g.sam = 1;
    g.sak = lda;
    g.B = A + (j0 + jb) + j0 * lda;
    g.sbn = 1;
    g.sbk = lda;
    g.C = A + (j0 + jb) + (j0 + jb) * lda;
    g.ldc = lda;
    g.epi.alpha = -1.0;
    g.epi.beta = 1.0;
    g.epi.C1 = g.C;
    g.epi.ldc1 = lda;
    if ((e = gemm<double>(g, st, ws, 1)) != hipSuccess) return e;
  }
  k_zero_upper<<<grid_for(b * b), 256, 0, st>>>(A, lda, b);
  return hipGetLastError();
}

// X <- L^{-1} X by block forward substitution with the diagonal blocks'
// inverses that potrf_lower left in tri for the same L.
hipError_t trsm_lower_left(const double* L, int64_t ldl, double* X, int64_t ldx, int64_t b,
                           int64_t nrhs, hipStream_t st, const Workspace& ws, double* tri) {
  hipError_t e = hipSuccess;
  const int64_t nblk = (b + NB - 1) / NB;
  double* tmp = tri + nblk * NB * NB;
  for (int64_t j0 = 0; j0 < b; j0 += NB) {
    const int jb = int(std::min<int64_t>(NB, b - j0));
    {   // tmp (jb x nrhs) = L_jj^{-1} X_j; X_j <- tmp
      GemmDesc<double> g;
      g.M = jb;
      g.N = nrhs;
      g.K = jb;
      g.A = tri + (j0 / NB) * NB * NB;
      g.sam = 1;
      g.sak = NB;
      g.B = X + j0;
      g.sbk = 1;
      g.sbn = ldx;
      g.C = tmp;
      g.ldc = jb;
      if ((e = gemm<double>(g, st, ws, 1)) != hipSuccess) return e;
      if ((e = copy_block(tmp, jb, X + j0, ldx, jb, nrhs, st)) != hipSuccess) return e;
    }
    const int64_t rows = b - j0 - jb;
    if (rows <= 0) break;
    GemmDesc<double> g;
    g.M = rows;
    g.N = nrhs;
    g.K = jb;
    g.A = L + (j0 + jb) + j0 * ldl;
    g.sam = 1;
    g.sak = ldl;
    g.B = X + j0;
    g.sbk = 1;
    g.sbn = ldx;
    g.C = X + j0 + jb;
    g.ldc = ldx;
    g.epi.alpha = -1.0;
    g.epi.beta = 1.0;
    g.epi.C1 = g.C;
    g.epi.ldc1 = ldx;
    if ((e = gemm<double>(g, st, ws, 1)) != hipSuccess) return e;
  }
  return hipSuccess;
}

static int64_t jacobi_padded(int64_t b) { return std::max<int64_t>(JP, (b + JP - 1) / JP * JP); }

size_t syev_workspace_bytes(int64_t b) {
  const int64_t bp = jacobi_padded(b);
  const int64_t npairs = bp / JP;
  return size_t(3 * bp * bp + 2 * npairs * JP * JP + 16 + kFroParts) * sizeof(double) +
         size_t(64 + 2 * npairs) * sizeof(int);
}

// pipelined outer rounds (knob CHFSI_JACOBI_PIPE=0: a pair-solve launch and a
// rotation launch per round; read at every call, so that tests can compare both)
static bool jacobi_pipelined() {
  const char* e = std::getenv("CHFSI_JACOBI_PIPE");
  return !(e && std::atoi(e) == 0);
}

hipError_t syev_jacobi(double* A, int64_t lda, int64_t b, double* w, double* V, int64_t ldv,
                       hipStream_t st, const Workspace& ws, int* sweeps_out,
                       int* unconverged_out, int* pinned_flags, hipEvent_t ev) {
  const int64_t bp = jacobi_padded(b);
  const int nblk = int(bp / JB);     // even
  const int npairs = nblk / 2;
  if (ws.bytes < syev_workspace_bytes(b)) return hipErrorInvalidValue;
  double* P = static_cast<double*>(ws.ptr);
  double* Vp = P + bp * bp;
  double* P2 = Vp + bp * bp;                      // the pipelined rounds' second buffer
  double* U = P2 + bp * bp;                       // two sets of npairs JP x JP factors
  double* scal = U + 2 * int64_t(npairs) * JP * JP;   // [0]: Frobenius norm
  auto* offmax = reinterpret_cast<unsigned long long*>(scal + 1);
  int* counter = reinterpret_cast<int*>(scal + 16 + kFroParts);   // [2], [3]: a sweep's flags
  int* skip = counter + 64;                       // two sets of npairs flags
  hipError_t e;
  k_jacobi_setup<<<kFroParts, 256, 0, st>>>(A, lda, b, P, Vp, bp, scal + 16);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  k_jacobi_begin<<<1, 64, 0, st>>>(scal + 16, scal, counter, offmax);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  const double tol = 1e-15;
  // sweep cap (knob CHFSI_JACOBI_MAX_SWEEPS, for tests of the cap's report)
  int max_outer = 40;
  if (const char* e = std::getenv("CHFSI_JACOBI_MAX_SWEEPS")) max_outer = std::max(1, std::atoi(e));
  int sweeps = 0;
  int host_count = 0;
  bool converged = false;
  const bool pipe = jacobi_pipelined();
  const int R = nblk - 1;                          // rounds per sweep
  const unsigned napply = unsigned(npairs) * unsigned(npairs + bp / JP);
  const int64_t usz = int64_t(npairs) * JP * JP;
  // launch r of the pipelined sweep: pair solves of round r (on the matrix
  // after round r - 1, formed in the pair workgroups) and round r - 1's
  // rotations P -> P2; launch R applies round R - 1
  auto launch = [&](int r) -> hipError_t {
    const bool solve = r < R, rotate = r > 0;
    const int cu = r & 1, pu = (r - 1) & 1;
    k_jacobi_round<<<dim3((solve ? unsigned(npairs) : 0u) + (rotate ? napply : 0u)), kPairThreads,
                     0, st>>>(
        P, P2, bp, Vp, bp, nblk, npairs, rotate ? r - 1 : -1, rotate ? U + pu * usz : nullptr,
        rotate ? skip + pu * npairs : nullptr, solve ? r : -1, solve ? U + cu * usz : nullptr,
        solve ? skip + cu * npairs : nullptr, scal, tol, counter, r == R ? offmax : nullptr);
    const hipError_t le = hipGetLastError();
    if (le == hipSuccess && rotate) std::swap(P, P2);
    return le;
  };
  // With a pinned flag buffer and an event, the first two launches of the
  // next sweep are queued before the convergence flags of this one are read
  // back, so the device does not idle while the host waits.  After
  // convergence those launches change nothing: every pair subproblem is below
  // the threshold (skipped), the rotation workgroups copy the matrix into the
  // other buffer, and only that buffer swap is undone.
  const bool early = pipe && pinned_flags && ev && R >= 2;
  int started = 0;   // launches of the current sweep already queued
  for (; sweeps < max_outer; ++sweeps) {
    if (pipe) {
      for (int r = started; r <= R; ++r)
        if ((e = launch(r)) != hipSuccess) return e;
      started = 0;
    } else {
      for (int r = 0; r < R; ++r) {
        k_jacobi_pair_solve<<<dim3(npairs), kPairThreads, 0, st>>>(P, bp, nblk, r, scal, tol, U,
                                                                   skip, counter);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        k_jacobi_apply<<<dim3(npairs, unsigned(npairs + bp / JP)), 256, 0, st>>>(
            P, bp, Vp, bp, nblk, npairs, r, U, skip);
        if ((e = hipGetLastError()) != hipSuccess) return e;
      }
    }
    // converged when the sweep rotated nothing, or when no off-diagonal entry
    // is left above the threshold (every pair of a further sweep would skip)
    if (!pipe) k_offmax<<<grid_for(bp * bp), 256, 0, st>>>(P, bp, offmax);
    k_sweep_end<<<1, 64, 0, st>>>(scal, tol, counter, offmax, early ? pinned_flags : counter + 2);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (early) {
      if ((e = hipEventRecord(ev, st)) != hipSuccess) return e;
      if (sweeps + 1 < max_outer) {
        for (int r = 0; r < 2; ++r)
          if ((e = launch(r)) != hipSuccess) return e;
        started = 2;
      }
      if ((e = hipEventSynchronize(ev)) != hipSuccess) return e;
      host_count = pinned_flags[0];
      if (host_count == 0 || pinned_flags[1] != 0) {
        if (started == 2) std::swap(P, P2);   // launch 1 copied the matrix into P2
        started = 0;
        converged = true;
        ++sweeps;
        break;
      }
      continue;
    }
    int host_flags[2] = {0, 0};
    if ((e = hipMemcpyAsync(host_flags, counter + 2, 2 * sizeof(int), hipMemcpyDeviceToHost, st)) !=
        hipSuccess)
      return e;
    if ((e = hipStreamSynchronize(st)) != hipSuccess) return e;
    host_count = host_flags[0];
    if (host_count == 0 || host_flags[1] != 0) {
      converged = true;
      ++sweeps;
      break;
    }
  }
  k_jacobi_sort<<<dim3(unsigned(b)), 256, 0, st>>>(P, Vp, bp, b, w, V, ldv);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if (sweeps_out) *sweeps_out = sweeps;
  // the tolerance was not met within the cap
  if (unconverged_out) *unconverged_out = converged ? 0 : 1;
  return hipSuccess;
}

}  // namespace chfsi
