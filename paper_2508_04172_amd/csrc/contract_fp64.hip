// FP64 form of the interpolant contraction Y = [Phi | P] W (Eq. rbfcoeff).  All
// kernels add the rows in one order with one MFMA, so the outputs do not depend on
// which of them a batch takes; fp64_parts.h holds the rules on sizes.
//
// Large batches, and the base of the others: the basis rows of a chunk of
// proposals are written to HBM by a VALU-only kernel (k_rows_fp64; small batches
// k_rows_small_fp64 or, with the epilogue's setups, k_rows_setup_fp64; plans
// k_ragged_rows_fp64), then a DGEMM-shaped FP64 MFMA kernel contracts them with
// the weights:
//   k_gemm_fp64            the handle's tile variant; 64 x 64 in batches of the
//                          middle sizes and for a short last round
//   k_gemm_small_fp64      32 x 32 tiles, four chunks in flight, small batches
//   k_gemm_lnl_fp64        128 x 128 tiles that finish ln L themselves
//   k_ragged_gemm_*        the same tiles over a plan's work list
// Why rows and product are two kernels: on gfx950 an FP64 MFMA and any VALU
// instruction of the same SIMD do not execute concurrently (the co-execution
// counter stays at zero), so the ~45 VALU instructions of each fused
// exp(-eps^2 d^2) row value (plus its recomputation for every column tile) are
// added to the MFMA time.  Apart from the rows the GEMM's inner loop issues only
// LDS reads and MFMAs; the rows cost one HBM round trip of 8 (N + M) bytes per
// proposal.
//   k_rows_gemm_fp64       is the exception: with one column tile every row value
//                          is used by one workgroup only, which forms it in LDS
//
// Layouts: rows Bt[r][q] (row r of proposal q, leading dimension ldb, a
// multiple of 8 >= nb, zero beyond nb); weights W[r][c] (Kp columns).
// v_mfma_f64_16x16x4f64 (lane l holds A[l%16][l/16], B[l/16][l%16]; accumulator
// element i is D[l/16 + 4i][l%16], measured on gfx950); a tile's WQ x WC waves
// hold RT x CT tiles of 16 x 16 each; chunks of KC rows of both operands are
// staged through LDS, double-buffered.
#include "basis_rows.h"
#include "epilogue_setup.h"
#include "fp64_parts.h"
#include "rbfl_internal.h"

namespace rbfl {

namespace {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef double d2 __attribute__((ext_vector_type(2)));

constexpr int kGemmThreads = 256;

// Basis rows 16*blockIdx.y .. +15 of proposals q = blockIdx.x*256 + tid (zero
// for nb <= q < ldb).
__global__ void __launch_bounds__(256) k_rows_fp64(const EvalConsts *__restrict__ cp,
                                                   const double *__restrict__ params, int64_t ld, int64_t b0,
                                                   int64_t nb, int64_t ldb, const double *__restrict__ nodes,
                                                   double *__restrict__ Bt) {
  const EvalConsts &c = *cp;
  const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (q >= ldb) return;
  const int r0 = 16 * blockIdx.y;
  if (q >= nb) {
#pragma unroll
    for (int k = 0; k < 16; ++k) Bt[(int64_t)(r0 + k) * ldb + q] = 0.0;
    return;
  }
  double x[4];
#pragma unroll
  for (int d = 0; d < 4; ++d) x[d] = params[d * ld + b0 + q] / c.semi[d];
  const int N = c.N, NM = c.N + c.M;
#pragma unroll 4
  for (int k = 0; k < 16; ++k) {
    const int r = r0 + k;
    Bt[(int64_t)r * ldb + q] = basis_row_fp64(r, N, NM, x, nodes + 4 * (int64_t)r, c.eps2, c.poly_idx);
  }
}

// Row r of proposal q (zero for q >= nb).
__device__ __forceinline__ double row_value(const EvalConsts &c, const double *__restrict__ params, int64_t ld,
                                            int64_t b0, int nb, int r, int q, const double *__restrict__ nodes) {
  if (q >= nb) return 0.0;
  double x[4];
#pragma unroll
  for (int d = 0; d < 4; ++d) x[d] = params[d * ld + b0 + q] / c.semi[d];
  return basis_row_fp64(r, c.N, c.N + c.M, x, nodes + 4 * (int64_t)r, c.eps2, c.poly_idx);
}

// The same rows for small batches, one row value per thread (t = r ldb + q):
// k_rows_fp64's 16 exponentials in a row per thread are a chain that a launch
// of few workgroups waits for.
__global__ void __launch_bounds__(256) k_rows_small_fp64(const EvalConsts *__restrict__ cp,
                                                         const double *__restrict__ params, int64_t ld, int64_t b0,
                                                         int nb, int ldb, int n_rows,
                                                         const double *__restrict__ nodes, double *__restrict__ Bt) {
  const EvalConsts &c = *cp;
  const unsigned t = blockIdx.x * 256 + threadIdx.x;
  const unsigned r = t / (unsigned)ldb, q = t - r * (unsigned)ldb;
  if (r >= (unsigned)n_rows) return;
  Bt[(int64_t)r * ldb + q] = row_value(c, params, ld, b0, nb, (int)r, (int)q, nodes);
}

// k_rows_small_fp64 whose first n_setup workgroups form the setups of the
// epilogue (kSetupGroup proposals each) instead: a chain of dependent steps that
// the row values of the others hide.
__global__ void __launch_bounds__(256) k_rows_setup_fp64(const EvalConsts *__restrict__ cp,
                                                         const double *__restrict__ params, int64_t ld, int64_t b0,
                                                         int nb, int ldb, int n_rows,
                                                         const double *__restrict__ nodes, double *__restrict__ Bt,
                                                         int n_setup, EpiSetup *__restrict__ setups) {
  const EvalConsts &c = *cp;
  if ((int)blockIdx.x < n_setup) {
    const int first = blockIdx.x * kSetupGroup;
    epi_setups_out(c, params, ld, b0, first, min(kSetupGroup, nb - first), setups);
    return;
  }
  const unsigned t = (blockIdx.x - n_setup) * 256 + threadIdx.x;
  const unsigned r = t / (unsigned)ldb, q = t - r * (unsigned)ldb;
  if (r >= (unsigned)n_rows) return;
  Bt[(int64_t)r * ldb + q] = row_value(c, params, ld, b0, nb, (int)r, (int)q, nodes);
}

// Workgroups are dealt to the 8 XCDs in turn; this gives each XCD a
// contiguous range of logical tiles (a bijection for any grid size), so the
// column tiles of one proposal tile run on one XCD and share its L2.
__device__ __forceinline__ int64_t xcd_logical_block(int64_t b, int64_t nblk) {
  const int64_t x = b & 7, slot = b >> 3, base = nblk >> 3, extra = nblk & 7;
  return x * base + (x < extra ? x : extra) + slot;
}

// One output tile of Y[q][c] = sum_r Bt[r][q] W[r][c]: proposals tq*QT ..,
// columns tc*CW ..; called by every thread of the workgroup.  Entries of a row
// from read_end on (even, at least nb) are not read and count as zeros.
template <int RT, int CT, int KC, int WQ = 2, int WC = 2>
__device__ __forceinline__ void gemm_tile(const double *__restrict__ Bt, int64_t nb, int64_t read_end, int64_t ldb,
                                          int rows,
                                          const double *__restrict__ W, int Kp, double *__restrict__ Y, int64_t tq,
                                          int tc) {
  constexpr int QT = WQ * RT * 16, CW = WC * CT * 16, NT = 64 * WQ * WC;
  constexpr int A2 = KC * QT / 2, W2 = KC * CW / 2;                 // double2 entries per chunk
  constexpr int LA = A2 / NT, LW = W2 / NT;
  static_assert(KC % 4 == 0 && A2 % NT == 0 && W2 % NT == 0, "whole k-steps, even staging");
  __shared__ double As[2][KC][QT];
  __shared__ double Ws[2][KC][CW];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wq = wave % WQ, wc = wave / WQ;
  const int c0 = tc * CW;
  const int64_t q0 = tq * QT;

  // per-thread source pointers of the staged entries, advanced by KC rows per chunk
  const double *pa[LA];
  const double *pw[LW];
  bool va[LA];
#pragma unroll
  for (int u = 0; u < LA; ++u) {
    const int e = tid + u * NT;
    const int k = e / (QT / 2), q2 = e % (QT / 2);
    pa[u] = Bt + (int64_t)k * ldb + q0 + 2 * q2;
    va[u] = q0 + 2 * q2 < read_end;
  }
#pragma unroll
  for (int u = 0; u < LW; ++u) {
    const int e = tid + u * NT;
    pw[u] = W + (int64_t)(e / (CW / 2)) * Kp + c0 + 2 * (e % (CW / 2));
  }
  const int64_t stepA = (int64_t)KC * ldb, stepW = (int64_t)KC * Kp;
  d2 ra[LA], rw[LW];
  auto fetch = [&]() {
#pragma unroll
    for (int u = 0; u < LA; ++u) {
      ra[u] = va[u] ? *reinterpret_cast<const d2 *>(pa[u]) : d2{0.0, 0.0};
      pa[u] += stepA;
    }
#pragma unroll
    for (int u = 0; u < LW; ++u) {
      rw[u] = *reinterpret_cast<const d2 *>(pw[u]);
      pw[u] += stepW;
    }
  };
  auto stash = [&](int buf) {
    // keeps the compiler from hoisting these LDS writes (and the wait for
    // their global loads) above the current chunk's MFMAs
    asm volatile("" ::: "memory");
#pragma unroll
    for (int u = 0; u < LA; ++u) {
      const int e = tid + u * NT;
      *reinterpret_cast<d2 *>(&As[buf][e / (QT / 2)][2 * (e % (QT / 2))]) = ra[u];
    }
#pragma unroll
    for (int u = 0; u < LW; ++u) {
      const int e = tid + u * NT;
      *reinterpret_cast<d2 *>(&Ws[buf][e / (CW / 2)][2 * (e % (CW / 2))]) = rw[u];
    }
  };

  d4 acc[RT][CT];
#pragma unroll
  for (int t = 0; t < RT; ++t)
#pragma unroll
    for (int u = 0; u < CT; ++u) acc[t][u] = d4{0.0, 0.0, 0.0, 0.0};

  const int kk = lane >> 4, ll = lane & 15;
  const int n_chunks = rows / KC;
  fetch();
  stash(0);
  __syncthreads();
  for (int ch = 0; ch < n_chunks; ++ch) {
    const int cur = ch & 1;
    if (ch + 1 < n_chunks) fetch();
#pragma unroll
    for (int s = 0; s < KC / 4; ++s) {
      const int k = 4 * s + kk;
      double a[RT], b[CT];
#pragma unroll
      for (int t = 0; t < RT; ++t) a[t] = As[cur][k][wq * RT * 16 + 16 * t + ll];
#pragma unroll
      for (int u = 0; u < CT; ++u) b[u] = Ws[cur][k][wc * CT * 16 + 16 * u + ll];
#pragma unroll
      for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int u = 0; u < CT; ++u) acc[t][u] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[t], b[u], acc[t][u], 0, 0, 0);
    }
    if (ch + 1 < n_chunks) stash(cur ^ 1);
    __syncthreads();
  }
#pragma unroll
  for (int t = 0; t < RT; ++t)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int64_t q = q0 + wq * RT * 16 + 16 * t + kk + 4 * i;
      if (q >= nb) continue;
#pragma unroll
      for (int u = 0; u < CT; ++u) Y[q * Kp + c0 + wc * CT * 16 + 16 * u + ll] = acc[t][u][i];
    }
}

// One-dimensional grid over (proposal tile, column tile), column tile fastest;
// WQ x WC waves per workgroup.
template <int RT, int CT, int KC, int WQ, int WC>
__global__ void __launch_bounds__(64 * WQ * WC, 512 / (64 * WQ * WC))
    k_gemm_fp64(const double *__restrict__ Bt, int64_t nb, int64_t read_end, int64_t ldb, int rows,
                const double *__restrict__ W, int Kp, int n_ct, double *__restrict__ Y) {
  const int64_t tile = xcd_logical_block(blockIdx.x, gridDim.x);
  gemm_tile<RT, CT, KC, WQ, WC>(Bt, nb, read_end, ldb, rows, W, Kp, Y, tile / n_ct, (int)(tile % n_ct));
}

constexpr int kFormRowsQ = 64;   // proposals per workgroup of k_rows_gemm_fp64

// Contraction that forms its own rows, for handles whose columns fit one tile
// (Kp = 128): 64 proposals x all columns per workgroup of 2 x 2 waves, each
// 2 x CT tiles of 16 x 16 (CT = the K / 32 rounded up), chunks of KC rows.  With one column tile every row
// value is used by one workgroup only, so writing it to HBM and reading it back
// buys nothing: each wave forms its share of the next chunk's rows (a lane per
// proposal, the nodes in scalar registers) straight into LDS before it
// multiplies the current one.  FP64 MFMA and VALU work of a SIMD add up, so the
// exponentials cost a third of the MFMA time (2900 cycles per chunk and
// workgroup against 2048 of MFMA alone); the rows' round trip costs more
// (1536 rows, 5e5 proposals: 3.68 ms against 1.22 ms of rows and 3.46 ms of
// product).  With 256 columns and 8 waves it does not (4.25 against 4.10 ms).
// With fewer columns only the tiles that
// hold them (41 columns, 208 rows, 3e5 proposals: 483 to 354 us for the whole
// evaluation).  Same row values, same MFMA order: the outputs are those of
// k_gemm_fp64 bit for bit.
template <int KC, int CT>
__global__ void __launch_bounds__(256)
    k_rows_gemm_fp64(const EvalConsts *__restrict__ cp, const double *__restrict__ params, int64_t ld, int64_t b0,
                     int64_t nb, const double *__restrict__ nodes, int rows, const double *__restrict__ W,
                     double *__restrict__ Y) {
  constexpr int RT = 2, WQ = 2, QT = kFormRowsQ, CW = 32 * CT, LD = 128, NT = 256, NW = 4;
  constexpr int LW = KC * CW / 2 / NT;     // double2 entries of W per thread and chunk
  constexpr int PR = KC / NW;              // rows of a chunk that a wave forms
  static_assert(KC * CW / 2 % NT == 0 && KC % NW == 0 && KC % 4 == 0, "even shares");
  __shared__ double As[2][KC][QT];
  __shared__ double Ws[2][KC][CW];
  const EvalConsts &c = *cp;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wq = wave % WQ, wc = wave / WQ, kk = lane >> 4, ll = lane & 15;
  const int64_t q0 = xcd_logical_block(blockIdx.x, gridDim.x) * QT;
  const int N = c.N, NM = c.N + c.M;
  const double eps2 = c.eps2;
  double x[4];
  const int64_t qx = q0 + lane < nb ? q0 + lane : nb - 1;     // past the batch: the last proposal again, not stored
#pragma unroll
  for (int d = 0; d < 4; ++d) x[d] = params[d * ld + b0 + qx] / c.semi[d];
  auto form = [&](int ch, int buf) {
    const int r0 = ch * KC + wave * PR;
    double v[PR];
    if (r0 + PR <= N) {
#pragma unroll
      for (int k = 0; k < PR; ++k) v[k] = gauss_row_fp64(x, nodes + 4 * (int64_t)(r0 + k), eps2);
    } else {
#pragma unroll
      for (int k = 0; k < PR; ++k)
        v[k] = basis_row_fp64(r0 + k, N, NM, x, nodes + 4 * (int64_t)(r0 + k), eps2, c.poly_idx);
    }
#pragma unroll
    for (int k = 0; k < PR; ++k) As[buf][wave * PR + k][lane] = v[k];
  };
  const double *pw[LW];
#pragma unroll
  for (int u = 0; u < LW; ++u) {
    const int e = tid + u * NT;
    pw[u] = W + (int64_t)(e / (CW / 2)) * LD + 2 * (e % (CW / 2));
  }
  d2 rw[LW];
  auto fetch = [&](int ch) {
#pragma unroll
    for (int u = 0; u < LW; ++u) rw[u] = *reinterpret_cast<const d2 *>(pw[u] + (int64_t)ch * KC * LD);
  };
  auto stash = [&](int buf) {
    asm volatile("" ::: "memory");
#pragma unroll
    for (int u = 0; u < LW; ++u) {
      const int e = tid + u * NT;
      *reinterpret_cast<d2 *>(&Ws[buf][e / (CW / 2)][2 * (e % (CW / 2))]) = rw[u];
    }
  };
  d4 acc[RT][CT];
#pragma unroll
  for (int t = 0; t < RT; ++t)
#pragma unroll
    for (int u = 0; u < CT; ++u) acc[t][u] = d4{0.0, 0.0, 0.0, 0.0};
  const int n_chunks = rows / KC;
  fetch(0);
  form(0, 0);
  stash(0);
  __syncthreads();
  for (int ch = 0; ch < n_chunks; ++ch) {
    const int cur = ch & 1;
    if (ch + 1 < n_chunks) {
      fetch(ch + 1);
      form(ch + 1, cur ^ 1);
    }
#pragma unroll
    for (int s = 0; s < KC / 4; ++s) {
      const int k = 4 * s + kk;
      double a[RT], b[CT];
#pragma unroll
      for (int t = 0; t < RT; ++t) a[t] = As[cur][k][wq * RT * 16 + 16 * t + ll];
#pragma unroll
      for (int u = 0; u < CT; ++u) b[u] = Ws[cur][k][wc * CT * 16 + 16 * u + ll];
#pragma unroll
      for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int u = 0; u < CT; ++u) acc[t][u] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[t], b[u], acc[t][u], 0, 0, 0);
    }
    if (ch + 1 < n_chunks) stash(cur ^ 1);
    __syncthreads();
  }
#pragma unroll
  for (int t = 0; t < RT; ++t)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int64_t q = q0 + wq * RT * 16 + 16 * t + kk + 4 * i;
      if (q >= nb) continue;
#pragma unroll
      for (int u = 0; u < CT; ++u) Y[q * LD + wc * CT * 16 + 16 * u + ll] = acc[t][u][i];
    }
}

// The accumulators of one output tile of Y[q][c] = sum_r Bt[r][q] W[r][c]
// (the K loop of gemm_tile, kept as a copy so that gemm_tile's code is not
// changed by this kernel):
// proposals tq*QT .., columns tc*CW ..; called by every thread of the
// workgroup; acc[t][u][i] of lane l is Y at proposal
// tq*QT + (wave % WQ)*RT*16 + 16t + l/16 + 4i and column
// tc*CW + (wave / WQ)*CT*16 + 16u + l%16.
template <int RT, int CT, int KC, int WQ = 2, int WC = 2>
__device__ __forceinline__ void gemm_accumulate(const double *__restrict__ Bt, int64_t ldb, int rows,
                                                const double *__restrict__ W, int Kp, int64_t tq, int tc,
                                                d4 (&acc)[RT][CT]) {
  constexpr int QT = WQ * RT * 16, CW = WC * CT * 16, NT = 64 * WQ * WC;
  constexpr int A2 = KC * QT / 2, W2 = KC * CW / 2;                 // double2 entries per chunk
  constexpr int LA = A2 / NT, LW = W2 / NT;
  static_assert(KC % 4 == 0 && A2 % NT == 0 && W2 % NT == 0, "whole k-steps, even staging");
  __shared__ double As[2][KC][QT];
  __shared__ double Ws[2][KC][CW];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wq = wave % WQ, wc = wave / WQ;
  const int c0 = tc * CW;
  const int64_t q0 = tq * QT;

  // per-thread source pointers of the staged entries, advanced by KC rows per chunk
  const double *pa[LA];
  const double *pw[LW];
  bool va[LA];
#pragma unroll
  for (int u = 0; u < LA; ++u) {
    const int e = tid + u * NT;
    const int k = e / (QT / 2), q2 = e % (QT / 2);
    pa[u] = Bt + (int64_t)k * ldb + q0 + 2 * q2;
    va[u] = q0 + 2 * q2 < ldb;
  }
#pragma unroll
  for (int u = 0; u < LW; ++u) {
    const int e = tid + u * NT;
    pw[u] = W + (int64_t)(e / (CW / 2)) * Kp + c0 + 2 * (e % (CW / 2));
  }
  const int64_t stepA = (int64_t)KC * ldb, stepW = (int64_t)KC * Kp;
  d2 ra[LA], rw[LW];
  auto fetch = [&]() {
#pragma unroll
    for (int u = 0; u < LA; ++u) {
      ra[u] = va[u] ? *reinterpret_cast<const d2 *>(pa[u]) : d2{0.0, 0.0};
      pa[u] += stepA;
    }
#pragma unroll
    for (int u = 0; u < LW; ++u) {
      rw[u] = *reinterpret_cast<const d2 *>(pw[u]);
      pw[u] += stepW;
    }
  };
  auto stash = [&](int buf) {
    // keeps the compiler from hoisting these LDS writes (and the wait for
    // their global loads) above the current chunk's MFMAs
    asm volatile("" ::: "memory");
#pragma unroll
    for (int u = 0; u < LA; ++u) {
      const int e = tid + u * NT;
      *reinterpret_cast<d2 *>(&As[buf][e / (QT / 2)][2 * (e % (QT / 2))]) = ra[u];
    }
#pragma unroll
    for (int u = 0; u < LW; ++u) {
      const int e = tid + u * NT;
      *reinterpret_cast<d2 *>(&Ws[buf][e / (CW / 2)][2 * (e % (CW / 2))]) = rw[u];
    }
  };

#pragma unroll
  for (int t = 0; t < RT; ++t)
#pragma unroll
    for (int u = 0; u < CT; ++u) acc[t][u] = d4{0.0, 0.0, 0.0, 0.0};

  const int kk = lane >> 4, ll = lane & 15;
  const int n_chunks = rows / KC;
  fetch();
  stash(0);
  __syncthreads();
  for (int ch = 0; ch < n_chunks; ++ch) {
    const int cur = ch & 1;
    if (ch + 1 < n_chunks) fetch();
#pragma unroll
    for (int s = 0; s < KC / 4; ++s) {
      const int k = 4 * s + kk;
      double a[RT], b[CT];
#pragma unroll
      for (int t = 0; t < RT; ++t) a[t] = As[cur][k][wq * RT * 16 + 16 * t + ll];
#pragma unroll
      for (int u = 0; u < CT; ++u) b[u] = Ws[cur][k][wc * CT * 16 + 16 * u + ll];
#pragma unroll
      for (int t = 0; t < RT; ++t)
#pragma unroll
        for (int u = 0; u < CT; ++u) acc[t][u] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[t], b[u], acc[t][u], 0, 0, 0);
    }
    if (ch + 1 < n_chunks) stash(cur ^ 1);
    __syncthreads();
  }
}

// The FP64 contraction that finishes ln L itself.  ln L is linear in the
// interpolated outputs, ln L = sum_c w_c Y[c], with the weights w_c of
// lnl_weight (the terms of Eq. logl_complete, corrected reading, as the
// epilogue kernel sums them).  After the same accumulation as k_gemm_fp64's
// 128 x 128 tile of 8 waves, each lane weights its 32 outputs, the 16 lanes
// of a row group and the two column waves add theirs (a fixed tree), and the
// tile writes one partial sum per proposal to part[column tile][proposal];
// Y is never written.  Proposals outside the domain contribute nothing here.
constexpr int kLnlRT = 2, kLnlCT = 4, kLnlKC = 8, kLnlWQ = 4, kLnlWC = 2;

__global__ void __launch_bounds__(64 * kLnlWQ * kLnlWC, 1)
    k_gemm_lnl_fp64(const double *__restrict__ Bt, int64_t nb, int64_t ldb, int rows, const double *__restrict__ W,
                    int Kp, const EvalConsts *__restrict__ cp, const EpiSetup *__restrict__ setups,
                    const double2 *__restrict__ basis4, const int4 *__restrict__ coldesc, double *__restrict__ part,
                    int64_t ldp) {
  constexpr int RT = kLnlRT, CT = kLnlCT, WQ = kLnlWQ, WC = kLnlWC;
  constexpr int QT = WQ * RT * 16, CW = WC * CT * 16;
  __shared__ double red[WC][QT];
  const int n_ct = Kp / CW;
  const int64_t tile = xcd_logical_block(blockIdx.x, gridDim.x);
  const int64_t tq = tile / n_ct;
  const int tc = (int)(tile % n_ct);
  d4 acc[RT][CT];
  gemm_accumulate<RT, CT, kLnlKC, WQ, WC>(Bt, ldb, rows, W, Kp, tq, tc, acc);
  const EvalConsts &c = *cp;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wq = wave % WQ, wc = wave / WQ, kk = lane >> 4, ll = lane & 15;
  const int n_modes = c.n_modes, T = c.T, q = c.q, K = c.K;
  const int64_t q0 = tq * QT;
  int4 dsc[CT];
#pragma unroll
  for (int u = 0; u < CT; ++u) {
    const int j = tc * CW + wc * CT * 16 + 16 * u + ll;
    dsc[u] = j < K ? coldesc[j] : make_int4(-1, 0, 0, 0);
  }
#pragma unroll
  for (int t = 0; t < RT; ++t)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = wq * RT * 16 + 16 * t + kk + 4 * i;
      const int64_t b = q0 + row;
      double sum = 0.0;
      if (b < nb && setups[b].status == 0) {
        const EpiSetup &o = setups[b];
#pragma unroll
        for (int u = 0; u < CT; ++u) {
          const int4 d = dsc[u];
          if (d.x < 0) continue;
          sum = fma(lnl_weight(d, o, n_modes, T, q, basis4), acc[t][u][i], sum);
        }
      }
#pragma unroll
      for (int m = 8; m >= 1; m >>= 1) sum += __shfl_xor(sum, m, 64);
      if (ll == 0) red[wc][row] = sum;
    }
  __syncthreads();
  for (int r = threadIdx.x; r < QT; r += 64 * WQ * WC) {
    const int64_t b = q0 + r;
    if (b >= nb) continue;
    double v = red[0][r];
#pragma unroll
    for (int w = 1; w < WC; ++w) v += red[w][r];
    part[(int64_t)tc * ldp + b] = v;
  }
}

// Multi-event batches: basis rows of every event in one launch.  blockIdx.y
// runs over the 16-row groups of all events (event e owns groups rg0 ..);
// blockIdx.x * 256 + tid is the proposal within the event.
__global__ void __launch_bounds__(256) k_ragged_rows_fp64(const EventDesc *__restrict__ ev, int n_ev,
                                                          const double *__restrict__ params, int64_t ld) {
  const int64_t gy = blockIdx.y;
  int lo = 0, hi = n_ev - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (ev[mid].rg0 <= gy) lo = mid;
    else hi = mid - 1;
  }
  const EventDesc &d = ev[lo];
  const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (q >= d.ldb) return;
  const int r0 = 16 * (int)(gy - d.rg0);
  if (q >= d.n) {
#pragma unroll
    for (int k = 0; k < 16; ++k) d.Bt[(int64_t)(r0 + k) * d.ldb + q] = 0.0;
    return;
  }
  const EvalConsts &c = *d.consts;
  double x[4];
#pragma unroll
  for (int dd = 0; dd < 4; ++dd) x[dd] = params[dd * ld + d.q0 + q] / c.semi[dd];
  const int N = c.N, NM = c.N + c.M;
#pragma unroll 4
  for (int k = 0; k < 16; ++k) {
    const int r = r0 + k;
    d.Bt[(int64_t)r * d.ldb + q] = basis_row_fp64(r, N, NM, x, d.nodes + 4 * (int64_t)r, c.eps2, c.poly_idx);
  }
}

// Persistent GEMM over the work list of every event: items are (event,
// proposal tile, column tile), column tile fastest within an event, events in
// decreasing row count; each workgroup takes the next item from an atomic
// counter until the list is exhausted (every workgroup reaches that exit).
template <int RT, int CT, int KC, int WQ = 2, int WC = 2>
__global__ void __launch_bounds__(64 * WQ * WC, 512 / (64 * WQ * WC))
    k_ragged_gemm_fp64(const EventDesc *__restrict__ ev, int n_ev, int64_t total_items,
                       unsigned long long *__restrict__ counter) {
  __shared__ long long item_s;
  for (;;) {
    if (threadIdx.x == 0) item_s = (long long)atomicAdd(counter, 1ull);
    __syncthreads();
    const int64_t item = item_s;
    __syncthreads();
    if (item >= total_items) break;
    const EventDesc &d = ev[work_event(ev, n_ev, item)];
    const int64_t local = item - d.item0;
    gemm_tile<RT, CT, KC, WQ, WC>(d.Bt, d.n, d.ldb, d.ldb, d.rows, d.W, d.Kp, d.Y, local / d.tiles_c,
                                  (int)(local % d.tiles_c));
  }
}

// Item of workgroup b of n: every other round of the 256 CUs is dealt backwards.
// The items come in decreasing length and the first rounds are all resident, so
// in order a CU that gets the longest item of one round gets that of each (12
// events of 250 proposals: 180 to 166 us, 6 of 1000: 225 to 211).
__device__ __forceinline__ int64_t dealt_item(int64_t b, int64_t n) {
  const int64_t round = b >> 8;
  return (round & 1) && ((round + 1) << 8) <= n ? (round << 8) + 255 - (b & 255) : b;
}

// The 64 x 64 tile over the work list, one workgroup per item: its items are too
// short to wait for the counter in between.
__global__ void __launch_bounds__(256, 2) k_ragged_gemm_mid_fp64(const EventDesc *__restrict__ ev, int n_ev) {
  const int64_t item = dealt_item(blockIdx.x, gridDim.x);
  const EventDesc &d = ev[work_event(ev, n_ev, item)];
  const int local = (int)(item - d.item0);
  gemm_tile<2, 2, 8>(d.Bt, d.n, d.ldb, d.ldb, d.rows, d.W, d.Kp, d.Y, local / d.tiles_c, local % d.tiles_c);
}

__global__ void k_zero_item_counter(unsigned long long *counter) {
  if (threadIdx.x == 0) *counter = 0ull;
}

// Rows the GEMMs contract: N + M rounded up to their chunk of KC rows.  The
// padded rows up to hc.rows hold zeros in W (and in the basis rows), so the
// chunks past this bound would only add zeros: the result is the same.
int gemm_rows(const EvalConsts &hc, int kc) { return (hc.N + hc.M + kc - 1) / kc * kc; }

// Small batches: 32 x 32 tiles of four waves (2 x 2), each one 16 x 16 tile;
// chunks of kTinyKC rows, the loads of the next four in flight in registers, the
// fragments of the next chunk read ahead.  Bound by the chain of one tile (rows /
// 4 dependent MFMAs of 64 cycles, 5.4 us for 808 rows) until there are several
// tiles per SIMD, then by LDS reads and MFMA.  The accumulation runs over the
// rows in the order of gemm_tile with the same MFMA, so the outputs are the same
// bit for bit.
constexpr int kTinyTile = 32, kTinyKC = 16;
constexpr int kTinyPad = 16;   // doubles per LDS row: two of a fragment's four rows per bank set
__device__ __forceinline__ void gemm_small_tile(const double *__restrict__ Bt, int nb, int end, int64_t ldb, int rows,
                                                const double *__restrict__ W, int Kp, double *__restrict__ Y, int q0,
                                                int c0) {
  constexpr int T = kTinyTile, KC = kTinyKC, KS = KC / 4, D = 4;
  static_assert(KC * T / 2 == 256, "one double2 of each operand per thread and chunk");
  __shared__ double As[2][KC][T + kTinyPad];
  __shared__ double Ws[2][KC][T + kTinyPad];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wq = wave & 1, wc = wave >> 1, kk = lane >> 4, ll = lane & 15;
  const int sk = tid / (T / 2), sm = 2 * (tid % (T / 2));
  // from entry `end` of a row on (even, at least nb) its last pair is read again: those outputs are not stored
  const double *pa = Bt + (int64_t)sk * ldb + (q0 + sm < end ? q0 + sm : end - 2);
  const double *pw = W + (int64_t)sk * Kp + c0 + sm;
  const int64_t stepA = KC * ldb, stepW = (int64_t)KC * Kp;
  const int n_chunks = rows / KC;
  d2 ra[D], rw[D];
  // every call loads (past the end the last chunk again), so that the wait
  // for one set leaves the later ones in flight
  auto fetch = [&](int ch, int i) {
    const int64_t at = ch < n_chunks ? ch : n_chunks - 1;
    ra[i] = *reinterpret_cast<const d2 *>(pa + at * stepA);
    rw[i] = *reinterpret_cast<const d2 *>(pw + at * stepW);
  };
  auto stash = [&](int buf, int i) {
    asm volatile("" ::: "memory");
    *reinterpret_cast<d2 *>(&As[buf][sk][sm]) = ra[i];
    *reinterpret_cast<d2 *>(&Ws[buf][sk][sm]) = rw[i];
  };
  d4 acc = d4{0.0, 0.0, 0.0, 0.0};
  double fa[2][KS], fb[2][KS];     // operand fragments of two chunks
  auto read = [&](int buf) {
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      fa[buf][s] = As[buf][4 * s + kk][wq * 16 + ll];
      fb[buf][s] = Ws[buf][4 * s + kk][wc * 16 + ll];
    }
  };
  // Step i: the fragments of chunk i + 1 leave LDS, chunk i + 2 goes into the
  // buffer that held chunk i (its fragments were read before the last
  // barrier), chunk i + 2 + D starts its way from memory, chunk i is multiplied.
  // Register set i % D and LDS buffer i % 2 hold chunk i.
#pragma unroll
  for (int i = 0; i < D; ++i) fetch(i, i);
  stash(0, 0);
  stash(1, 1);
  fetch(D, 0);
  fetch(D + 1, 1);
  __syncthreads();
  read(0);
  __syncthreads();
  auto step = [&](int c, int i) {
    read((i + 1) & 1);
    __builtin_amdgcn_sched_barrier(0);
    stash(i & 1, (i + 2) % D);
    fetch(c + 2 + D, (i + 2) % D);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < KS; ++s)
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(fa[i & 1][s], fb[i & 1][s], acc, 0, 0, 0);
    __syncthreads();
  };
  int c = 0;
  for (; c + D <= n_chunks; c += D) {
#pragma unroll
    for (int i = 0; i < D; ++i) step(c + i, i);
  }
  if (c < n_chunks) {                      // an even count of chunks: two are left
    step(c, 0);
    step(c + 1, 1);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int64_t q = q0 + wq * 16 + kk + 4 * i;
    if (q < nb) Y[q * Kp + c0 + wc * 16 + ll] = acc[i];
  }
}

__global__ void __launch_bounds__(256)
    k_gemm_small_fp64(const double *__restrict__ Bt, int nb, int end, int64_t ldb, int rows,
                      const double *__restrict__ W, int Kp, int n_ct, double *__restrict__ Y) {
  const int64_t tile = xcd_logical_block(blockIdx.x, gridDim.x);
  gemm_small_tile(Bt, nb, end, ldb, rows, W, Kp, Y, (int)(tile / n_ct) * kTinyTile, (int)(tile % n_ct) * kTinyTile);
}

// The small tiles over the work list of a multi-event batch, one workgroup per
// item (events in decreasing row count, so the longest items start first).
__global__ void __launch_bounds__(256) k_ragged_gemm_small_fp64(const EventDesc *__restrict__ ev, int n_ev) {
  const int64_t item = dealt_item(blockIdx.x, gridDim.x);
  const EventDesc &d = ev[work_event(ev, n_ev, item)];
  const int local = (int)(item - d.item0);
  const EvalConsts &c = *d.consts;
  const int rows = (c.N + c.M + 2 * kTinyKC - 1) / (2 * kTinyKC) * (2 * kTinyKC);
  gemm_small_tile(d.Bt, (int)d.n, (int)d.ldb, d.ldb, rows, d.W, d.Kp, d.Y, local / d.tiles_c * kTinyTile,
                  local % d.tiles_c * kTinyTile);
}

// Basis rows that k_rows_fp64 writes: N + M rounded up to its 16-row groups
// (at least gemm_rows for chunks of 8 or 16 rows).
int basis_rows_written(const EvalConsts &hc) { return (hc.N + hc.M + 15) / 16 * 16; }

template <int RT, int CT, int KC, int WQ = 2, int WC = 2>
void launch_gemm(const double *Bt, const Fp64Part &part, int64_t ldb, const EvalConsts &hc, const double *W,
                 double *Y, hipStream_t s) {
  constexpr int QT = WQ * RT * 16, CW = WC * CT * 16;
  static_assert(kColTile % CW == 0 && kRowChunk % KC == 0 && 16 % KC == 0, "K and the rows are padded to whole tiles");
  const int n_ct = col_tiles(hc, CW);
  const int64_t nblk = (part.count + QT - 1) / QT * n_ct;
  hipLaunchKernelGGL((k_gemm_fp64<RT, CT, KC, WQ, WC>), dim3((unsigned)nblk), dim3(64 * WQ * WC), 0, s,
                     Bt + part.first, part.count, part.read_end, ldb, gemm_rows(hc, KC), W, hc.Kp, n_ct,
                     Y + part.first * hc.Kp);
  RBFL_HIP(hipGetLastError());
}

void launch_gemm_small(const double *Bt, const Fp64Part &part, int64_t ldb, const EvalConsts &hc, const double *W,
                       double *Y, hipStream_t s) {
  static_assert(kColTile % kTinyTile == 0 && kRowChunk % (2 * kTinyKC) == 0, "whole tiles and chunk pairs");
  const int n_ct = col_tiles(hc, kTinyTile);
  const int64_t nblk = (part.count + kTinyTile - 1) / kTinyTile * n_ct;
  hipLaunchKernelGGL(k_gemm_small_fp64, dim3((unsigned)nblk), dim3(256), 0, s, Bt + part.first, (int)part.count,
                     (int)part.read_end, ldb, gemm_rows(hc, 2 * kTinyKC), W, hc.Kp, n_ct, Y + part.first * hc.Kp);
  RBFL_HIP(hipGetLastError());
}

}  // namespace

// Rows that a batch's contraction with `variant` (-1: the fused epilogue's) reads
// and the row kernels must write: whole chunk pairs where 32 x 32 tiles take a part.
static int rows_needed(const EvalConsts &hc, int64_t nb, int variant, bool pinned) {
  if (variant < 0) return basis_rows_written(hc);
  const int64_t rest = fp64_parts(hc, nb, variant, pinned).rest.count;
  return rest > 0 && tiles32(hc, rest) < kTinyTiles ? hc.rows : basis_rows_written(hc);
}

// The same for a multi-event batch: 1 = 32 x 32, 2 = 64 x 64 tiles, 0 = the
// plan's variant (64 x 64 / variant: 129 / 145 us for 4 events of 1000 proposals,
// 4096 tiles; 385 / 400 us for 12, 11,440 tiles).
int ragged_small_tile(int64_t tiles) { return tiles < kTinyTiles ? 1 : tiles < kMidTiles ? 2 : 0; }

int gemm_lnl_col_tile() { return kLnlWC * kLnlCT * 16; }

void launch_gemm_lnl_fp64(const double *Bt, int64_t nb, const EvalConsts &hc, const double *W, const EvalConsts *c,
                          const void *setups, const double2 *basis4, const int4 *coldesc, double *part, int64_t ldp,
                          hipStream_t s) {
  constexpr int QT = kLnlWQ * kLnlRT * 16, CW = kLnlWC * kLnlCT * 16;
  static_assert(kColTile % CW == 0 && kRowChunk % kLnlKC == 0, "K and the rows are padded to whole tiles");
  if (nb <= 0) return;
  const int64_t ldb = rows_ld(nb);
  const int64_t nblk = (nb + QT - 1) / QT * (hc.Kp / CW);
  hipLaunchKernelGGL(k_gemm_lnl_fp64, dim3((unsigned)nblk), dim3(64 * kLnlWQ * kLnlWC), 0, s, Bt, nb, ldb,
                     gemm_rows(hc, kLnlKC), W,
                     hc.Kp, c, static_cast<const EpiSetup *>(setups), basis4, coldesc, part, ldp);
  RBFL_HIP(hipGetLastError());
}

int gemm_fp64_variants() { return 7; }

const char *gemm_fp64_variant_name(int v) {
  static const char *names[] = {"rows + gemm 64x128 kc8",  "rows + gemm 128x64 kc8", "rows + gemm 64x128 kc16",
                                "rows + gemm 128x64 kc16", "rows + gemm 64x64 kc8",
                                "rows + gemm 256x128 kc8 (8 waves)", "rows + gemm 128x128 kc8 (8 waves)"};
  return names[v];
}

// Operand reuse of a variant's workgroup tile, QT CW / (QT + CW): the
// algorithmic bytes over the bytes the workgroups read, up to a constant.
double gemm_fp64_reuse(int v) {
  static const double qt[] = {64, 128, 64, 128, 64, 256, 128}, cw[] = {128, 64, 128, 64, 64, 128, 128};
  return qt[v] * cw[v] / (qt[v] + cw[v]);
}

// How many of a batch's first proposals the contraction forms its own rows for
// (k_rows_gemm_fp64).  None with more than one column tile, and none while
// there are fewer than two workgroups per CU, where a workgroup alone waits for
// its exponentials (1536 rows: 188 against 162 us at 16384 proposals, 279
// against 315 us at 32768), unless there are few rows, where the separate
// kernels' start-up counts for more (208 rows: 32 against 39 us at 12288).
// Otherwise all, but for a last partial round of the chip (three workgroups on
// each of the 256 CUs) of less than a sixth: one workgroup alone on a CU takes
// half as long as three together, the small tiles take a quarter of that.
int64_t gemm_own_rows(const EvalConsts &hc, int64_t nb) {
  constexpr int64_t kRound = 3 * 256 * kFormRowsQ;
  if (hc.Kp != 128 || nb < (hc.rows <= 512 ? 12288 : 32768)) return 0;
  const int64_t rest = nb % kRound;
  return nb > kRound && rest < kRound / 6 ? nb - rest : nb;
}

void launch_rows_gemm_fp64(const EvalConsts *c, const EvalConsts &hc, const double *params, int64_t ld, int64_t b0,
                           int64_t nb, const double *nodes, const double *W, double *Y, hipStream_t s) {
  constexpr int KC = 16;
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)((nb + kFormRowsQ - 1) / kFormRowsQ)), dim3(256), 0, s, c, params, ld, b0,
                       nb, nodes, gemm_rows(hc, KC), W, Y);
  };
  switch (col_tiles(hc, 32)) {
    case 1: launch(k_rows_gemm_fp64<KC, 1>); break;
    case 2: launch(k_rows_gemm_fp64<KC, 2>); break;
    case 3: launch(k_rows_gemm_fp64<KC, 3>); break;
    default: launch(k_rows_gemm_fp64<KC, 4>);
  }
  RBFL_HIP(hipGetLastError());
}

bool launch_rows_fp64(const EvalConsts *c, const EvalConsts &hc, const double *params, int64_t ld, int64_t b0,
                      int64_t nb, const double *nodes, double *Bt, hipStream_t s, int variant, void *setups,
                      bool pinned) {
  const int64_t ldb = rows_ld(nb);
  const int n_rows = rows_needed(hc, nb, variant, pinned);
  // one value per thread while that is fewer than four rounds of the chip
  // (1021 proposals of 832 rows: 9.1 against 10.7 us; 2048: no gain)
  if (ldb * n_rows <= (1 << 20)) {
    const unsigned blocks = (unsigned)((ldb * n_rows + 255) / 256);
    const bool with_setups = setups != nullptr && nb <= kSetupMax && hc.n_bands <= 1;
    if (with_setups) {
      const int n_setup = (int)((nb + kSetupGroup - 1) / kSetupGroup);
      hipLaunchKernelGGL(k_rows_setup_fp64, dim3(n_setup + blocks), dim3(256), 0, s, c, params, ld, b0, (int)nb,
                         (int)ldb, n_rows, nodes, Bt, n_setup, static_cast<EpiSetup *>(setups));
    } else {
      hipLaunchKernelGGL(k_rows_small_fp64, dim3(blocks), dim3(256), 0, s, c, params, ld, b0, (int)nb, (int)ldb, n_rows,
                         nodes, Bt);
    }
    RBFL_HIP(hipGetLastError());
    return with_setups;
  }
  dim3 grid((unsigned)((ldb + 255) / 256), (unsigned)(n_rows / 16));
  hipLaunchKernelGGL(k_rows_fp64, grid, dim3(256), 0, s, c, params, ld, b0, nb, ldb, nodes, Bt);
  RBFL_HIP(hipGetLastError());
  return false;
}

void launch_ragged_rows_fp64(const EventDesc *ev, int n_ev, int64_t total_groups, int64_t max_ldb,
                             const double *params, int64_t ld, hipStream_t s) {
  dim3 grid((unsigned)((max_ldb + 255) / 256), (unsigned)total_groups);
  hipLaunchKernelGGL(k_ragged_rows_fp64, grid, dim3(256), 0, s, ev, n_ev, params, ld);
  RBFL_HIP(hipGetLastError());
}

// Multi-event GEMM tiles: variant 0 is 64 x 128 with 8-row chunks (4 waves),
// variant 1 64 x 128 with 16-row chunks (4 waves), variant 2 128 x 128 with
// 8-row chunks (8 waves, the single-event kernel's preferred tile).
void launch_ragged_gemm_fp64(int variant, const EventDesc *ev, int n_ev, int64_t total_items,
                             unsigned long long *counter, int grid, hipStream_t s) {
  hipLaunchKernelGGL(k_zero_item_counter, dim3(1), dim3(64), 0, s, counter);
  RBFL_HIP(hipGetLastError());
  if (variant == 2)
    hipLaunchKernelGGL((k_ragged_gemm_fp64<2, 4, 8, 4, 2>), dim3(grid), dim3(512), 0, s, ev, n_ev, total_items,
                       counter);
  else if (variant == 1)
    hipLaunchKernelGGL((k_ragged_gemm_fp64<2, 4, 16>), dim3(grid), dim3(kGemmThreads), 0, s, ev, n_ev, total_items,
                       counter);
  else
    hipLaunchKernelGGL((k_ragged_gemm_fp64<2, 4, 8>), dim3(grid), dim3(kGemmThreads), 0, s, ev, n_ev, total_items,
                       counter);
  RBFL_HIP(hipGetLastError());
}

void launch_ragged_gemm_small_fp64(int small, const EventDesc *ev, int n_ev, int64_t total_items, hipStream_t s) {
  if (small == 1)
    hipLaunchKernelGGL(k_ragged_gemm_small_fp64, dim3((unsigned)total_items), dim3(256), 0, s, ev, n_ev);
  else
    hipLaunchKernelGGL(k_ragged_gemm_mid_fp64, dim3((unsigned)total_items), dim3(256), 0, s, ev, n_ev);
  RBFL_HIP(hipGetLastError());
}

void launch_gemm_fp64(const double *Bt, int64_t nb, const EvalConsts &hc, const double *W, double *Y, hipStream_t s,
                      int variant, bool pinned) {
  if (variant < 0 || variant >= gemm_fp64_variants()) throw Error(RBFL_E_INVALID_ARG, "unknown FP64 GEMM variant");
  const int64_t ldb = rows_ld(nb);
  const Fp64Parts p = fp64_parts(hc, nb, variant, pinned);
  if (p.main.count > 0) switch (variant) {
      case 0: launch_gemm<2, 4, 8>(Bt, p.main, ldb, hc, W, Y, s); break;
      case 1: launch_gemm<4, 2, 8>(Bt, p.main, ldb, hc, W, Y, s); break;
      case 2: launch_gemm<2, 4, 16>(Bt, p.main, ldb, hc, W, Y, s); break;
      case 3: launch_gemm<4, 2, 16>(Bt, p.main, ldb, hc, W, Y, s); break;
      case 4: launch_gemm<2, 2, 8>(Bt, p.main, ldb, hc, W, Y, s); break;
      case 5: launch_gemm<4, 4, 8, 4, 2>(Bt, p.main, ldb, hc, W, Y, s); break;
      default: launch_gemm<2, 4, 8, 4, 2>(Bt, p.main, ldb, hc, W, Y, s);
    }
  if (p.rest.count <= 0) return;
  if (tiles32(hc, p.rest.count) < kTinyTiles) launch_gemm_small(Bt, p.rest, ldb, hc, W, Y, s);
  else launch_gemm<2, 2, 8>(Bt, p.rest, ldb, hc, W, Y, s);
}

bool launch_product_fp64(const EvalConsts *c, const EvalConsts &hc, const double *params, int64_t ld, int64_t b0,
                         int64_t nb, const double *nodes, const double *W, double *Bt, double *Y, hipStream_t s,
                         int variant, hipEvent_t mid, void *setups, bool pinned) {
  const int64_t own = pinned ? 0 : gemm_own_rows(hc, nb);
  bool ready = false;
  if (own < nb)
    ready = launch_rows_fp64(c, hc, params, ld, b0 + own, nb - own, nodes, Bt, s, variant, own == 0 ? setups : nullptr,
                             pinned);
  if (mid) RBFL_HIP(hipEventRecord(mid, s));
  if (own > 0) launch_rows_gemm_fp64(c, hc, params, ld, b0, own, nodes, W, Y, s);
  if (own < nb) launch_gemm_fp64(Bt, nb - own, hc, W, Y + own * hc.Kp, s, variant, pinned);
  return ready;
}

bool gemm_fp64_variant_runs(const EvalConsts &hc, int64_t nb, int variant) {
  return main_part(hc, nb - gemm_own_rows(hc, nb), variant) > 0;
}

}  // namespace rbfl
