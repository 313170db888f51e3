// FP64 ln L of the smallest batches in one launch (frozen antenna patterns).
#include <algorithm>

#include "basis_rows.h"
#include "epilogue_setup.h"
#include "rbfl_internal.h"

namespace rbfl {

namespace {

typedef double d4 __attribute__((ext_vector_type(4)));

constexpr int kMaxGroup = 16;        // proposals per workgroup: the rows of one tile
constexpr int kMaxRowValues = 6000;  // row values that a workgroup forms (48 KB of LDS)

size_t shared_bytes(const EvalConsts &hc, int slots) {
  return (size_t)slots * (sizeof(double) * hc.rows + sizeof(EpiSetup) + sizeof(EpiTmp));
}

// A row of outputs that other workgroups have written in this launch: read past
// the caches that may hold it as it was.
struct SharedRow {
  const double *p;
  __device__ double operator[](int i) const {
    return __hip_atomic_load(p + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
};
__device__ __forceinline__ double2 load_pair(SharedRow y, int i) { return double2{y[i], y[i + 1]}; }

// Workgroup (x, y) forms the interpolated outputs of columns 64 x .. 64 x + 63 of
// the proposals slots y .. and the last workgroup of a y to finish reduces them
// to ln L.  Waves 0-3 form the proposals' basis rows in LDS and multiply them, 16
// columns each, with W straight from memory into registers (D - 1 chunks of 32
// rows in flight); waves 4-7 form the epilogue's setups meanwhile, in every
// workgroup, since any of them can be the last.
//
// A batch this small waits for launches and for chains of dependent steps, not
// for the chip: rows, product and epilogue in launches of their own take 13.0 us
// for four proposals of 200 nodes, one detector and one mode (this kernel 9.0),
// 24.4 us with 800 nodes, three detectors and five modes (18.5: 5.5 the chain of
// 208 MFMAs, 5 the reduction).  The next chunk's fragments are read from LDS and
// the loads of W issued before a chunk's MFMAs; left to itself the compiler puts
// both right before their use (13.7 -> 20 us for one proposal of 800 nodes).
// Sharing the 16 columns out to four waves, each holding a quarter of the rows'
// W in registers, was slower (15.5 us).  Row values, the order of the products
// and the reduction are those of the staged kernels, so ln L is the same bit for
// bit.
//
// slots (a power of two): the proposals' stride in LDS.  nan->done[y] counts the
// finished workgroups and wraps to zero with the last.
__global__ void __launch_bounds__(512, 2)
    k_eval_small(const EvalConsts *__restrict__ cp, const double *__restrict__ params, int64_t ld, int nb, int slots,
                 const double *__restrict__ nodes, const double *__restrict__ W, double *__restrict__ Y,
                 const double2 *__restrict__ basis4, double *__restrict__ lnl, NanCount *__restrict__ nan) {
  extern __shared__ double As[];     // [rows][slots], then the setups
  __shared__ YlmTerms ylm[2 * RBFL_MAX_MODES];
  __shared__ int coef_off[RBFL_MAX_DET][RBFL_MAX_MODES], sig_off[RBFL_MAX_DET];
  __shared__ int last;
  const EvalConsts &c = *cp;
  const int rows = c.rows, Kp = c.Kp, nm = c.n_modes;
  EpiSetup *su = reinterpret_cast<EpiSetup *>(As + (size_t)rows * slots);
  EpiTmp *tmp = reinterpret_cast<EpiTmp *>(su + slots);
  const int t = threadIdx.x, lane = t & 63, kk = lane >> 4, ll = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const bool multiplies = wave < 4;
  const int first = blockIdx.y * slots, cnt = min(slots, nb - first);
  const int c0 = blockIdx.x * 64 + wave * 16;   // of a multiplying wave
  constexpr int KS = 8, D = 4;                  // steps of four rows per chunk, chunks of W held
  const int n_chunks = rows / (4 * KS);
  const unsigned w_at = (unsigned)(kk * Kp + c0 + ll);
  double w[D][KS];
  auto fetch = [&](int ch, int i) {                       // past the end the last chunk again
    const double *p = W + (int64_t)min(ch, n_chunks - 1) * 4 * KS * Kp;
#pragma unroll
    for (int s = 0; s < KS; ++s, p += 4 * Kp) w[i][s] = p[w_at];
  };
  // every wave meets the others three times: rows formed, outputs and parts of
  // the setups written, setups joined
  if (multiplies) {
#pragma unroll
    for (int i = 0; i < D - 1; ++i) fetch(i, i);
    const int j = t & (slots - 1);
    if (j < cnt) {
      double x[4];
#pragma unroll
      for (int d = 0; d < 4; ++d) x[d] = params[d * ld + first + j] / c.semi[d];
      const int N = c.N, NM = c.N + c.M;
#pragma unroll 4
      for (int r = t / slots; r < rows; r += 256 / slots)
        As[r * slots + j] = basis_row_fp64(r, N, NM, x, nodes + 4 * (int64_t)r, c.eps2, c.poly_idx);
    }
    __syncthreads();
    d4 acc = d4{0.0, 0.0, 0.0, 0.0};
    // rows of the tile past the group multiply whatever LDS holds and are not stored
    const double *a = As + kk * slots + min(ll, slots - 1);
    double av[2][KS];
    auto read = [&](int ch, int i) {
#pragma unroll
      for (int s = 0; s < KS; ++s) av[i][s] = a[(min(ch, n_chunks - 1) * KS + s) * 4 * slots];
    };
    auto step = [&](int ch, int i) {
      fetch(ch + D - 1, (i + D - 1) % D);
      read(ch + 1, (i + 1) & 1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int s = 0; s < KS; ++s)
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(av[i & 1][s], w[i][s], acc, 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    };
    static_assert(D % 2 == 0, "the fragments' sets alternate over the unrolled steps");
    int ch = 0;
    read(ch, 0);
    for (; ch + D <= n_chunks; ch += D) {
#pragma unroll
      for (int i = 0; i < D; ++i) step(ch + i, i);
    }
#pragma unroll
    for (int i = 0; i < D - 1; ++i)
      if (ch + i < n_chunks) step(ch + i, i);
    // written through to where every XCD reads it; the wait orders it before
    // this workgroup is counted
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (kk + 4 * i < cnt)
        __hip_atomic_store(Y + (int64_t)(first + kk + 4 * i) * Kp + c0 + ll, acc[i], __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  } else {
    epi_copy_ylm(t - 256, c, ylm);
    epi_copy_offsets(t - 256, c, coef_off, sig_off);
    __syncthreads();
    epi_setup_parts(t - 256, [&](int) -> const EvalConsts & { return c; },
                    [&](int, int i) -> const YlmTerms & { return ylm[i]; }, c.n_det, nm, params, ld, first, cnt, su,
                    tmp);
  }
  __syncthreads();
  if (!multiplies)
    epi_setup_join(t - 256, [&](int) -> const EvalConsts & { return c; }, c.n_det, nm, cnt, su, tmp);
  else if (t == 0)
    last = atomicInc(nan->done + blockIdx.y, gridDim.x - 1) == gridDim.x - 1;
  __syncthreads();
  if (!last) return;
  if (blockIdx.y == 0 && t == 0) nan->slots = (unsigned long long)nb;
  for (int j = wave; j < cnt; j += 8) {
    const double v = epi_reduce<5>(c, su[j], SharedRow{Y + (int64_t)(first + j) * Kp}, basis4, coef_off, sig_off);
    if (lane != 0) continue;
    lnl[first + j] = v;
    nan->part[first + j] = isnan(v) ? 1ull : 0ull;
  }
}

}  // namespace

// Proposals per workgroup of the one-launch evaluation of n proposals, 0: n is
// too large for it.  The smallest count that leaves at most kSmallBlocks
// workgroups, one per CU (with two per CU they share its matrix cores: 21.3 to
// 27.7 us for 16 proposals of 832 rows and 1280 columns), while a wave forms its
// share of the rows in less time than the launches it saves: us staged / here at
// 832 x 1280 25.8 / 21.3 for 16 proposals (2 per workgroup, 1664 row values),
// 26.6 / 23.9 for 32 (3328), 26.9 / 35 for 64 (6656); at 224 x 128 15.9 / 12.5
// for 1024 (1792); at 1504 x 128 33.8 / 25.6 for 256 (3008); at 3008 x 2560 57 /
// 49 for 6 (3008).
int small_eval_group(const EvalConsts &hc, int64_t n) {
  const int n_ct = col_tiles(hc, 64);
  if (hc.n_bands > 1 || n > (int64_t)kMaxGroup * (kSmallBlocks / n_ct)) return 0;
  for (int slots = 1; slots <= kMaxGroup && slots * hc.rows <= kMaxRowValues; slots *= 2)
    if ((n + slots - 1) / slots * n_ct <= kSmallBlocks) return slots;
  return 0;
}

void launch_eval_small(int slots, const EvalConsts *c, const EvalConsts &hc, const double *params, int64_t ld,
                       int64_t n, const double *nodes, const double *W, double *Y, const double2 *basis4, double *lnl,
                       NanCount *nan, hipStream_t s) {
  const unsigned groups = (unsigned)((n + slots - 1) / slots);
  hipLaunchKernelGGL(k_eval_small, dim3(col_tiles(hc, 64), groups), dim3(512), shared_bytes(hc, slots), s, c, params, ld,
                     (int)n, slots, nodes, W, Y, basis4, lnl, nan);
  RBFL_HIP(hipGetLastError());
}

}  // namespace rbfl
