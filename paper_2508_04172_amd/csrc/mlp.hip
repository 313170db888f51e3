// Surrogate network kernels: a multilayer perceptron in -> H -> H -> out with
// SiLU activations, trained by the project's own forward, backward and Adam
// kernels (FP32 arithmetic on the FP32 matrix cores, FP32 master weights).
//
// Parameter layout: W1 [H][in], b1 [H], W2 [H][H], b2 [H], W3 [out][H],
// b3 [out], weights row-major.  Initialisation from caller-provided standard
// normal deviates z: W = z / sqrt(fan_in), b = 0.
#include "rbfl_internal.h"

namespace rbfl {

namespace {

constexpr int kT = 256;

typedef float f4 __attribute__((ext_vector_type(4)));

// Large forward layers whose operands are both contiguous in k (activations
// A[m][k], weights W[n][k]): 128 x 128 tiles of 8 waves (4 along m x 2 along
// n, each 2 x 4 tiles of 16 x 16), 16-deep k chunks double-buffered through
// LDS with one float4 of each operand per thread and chunk; workgroups are
// dealt to the 8 XCDs in turn, so logical tiles are remapped to give each XCD a
// contiguous range: the column tiles of one row tile share an XCD's L2.  The
// caller guarantees K % 16 == 0 and 16-byte aligned rows.
// ACT 0: linear, 1: SiLU, 2: linear with the output standardisation undone
// in FP64, Y[m][n] = mu[n] + sd[n] v into the interpolant's output layout
// (row stride ldc), as the surrogate form's inference needs it; with Bb set
// (residual form) the FP64 polynomial base sum_j Ub[m][j] Bb[j][n] is added
// (Ub: the proposal's nbase monomials, Bb: the base coefficients [nbase][N]).
template <int ACT>
__global__ void __launch_bounds__(512) k_gemm_f32_nt(int M, int N, int K, const float *__restrict__ A, int64_t lda,
                                                     const float *__restrict__ B, int64_t ldb,
                                                     const float *__restrict__ bias, float *__restrict__ Z,
                                                     float *__restrict__ C, int64_t ldc, const float *__restrict__ mu,
                                                     const float *__restrict__ sd, double *__restrict__ Y64,
                                                     const double *__restrict__ Ub, const double *__restrict__ Bb,
                                                     int nbase) {
  __shared__ float As[2][16][128 + 4];
  __shared__ float Bs[2][16][128 + 4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wq = wave & 3, wc = wave >> 2;
  const int kk = lane >> 4, ll = lane & 15;
  const int n_nt = (N + 127) / 128;
  const int64_t nblk = gridDim.x, bx = blockIdx.x;
  const int64_t xcd = bx & 7, slot = bx >> 3, base = nblk >> 3, extra = nblk & 7;
  const int64_t tile = xcd * base + (xcd < extra ? xcd : extra) + slot;
  const int m0 = (int)(tile / n_nt) * 128, n0 = (int)(tile % n_nt) * 128;
  // staging: thread tid carries row tid / 4 of both tiles, k quad (tid % 4) * 4
  const int sr = tid >> 2, sk = (tid & 3) * 4;
  const int am = m0 + sr, bn = n0 + sr;
  const float *pa = A + (int64_t)(am < M ? am : 0) * lda + sk;
  const float *pb = B + (int64_t)(bn < N ? bn : 0) * ldb + sk;
  f4 ra, rb;
  auto fetch = [&](int k0) {
    ra = am < M ? *reinterpret_cast<const f4 *>(pa + k0) : f4{0.0f, 0.0f, 0.0f, 0.0f};
    rb = bn < N ? *reinterpret_cast<const f4 *>(pb + k0) : f4{0.0f, 0.0f, 0.0f, 0.0f};
  };
  auto stash = [&](int buf) {
    asm volatile("" ::: "memory");
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      As[buf][sk + j][sr] = ra[j];
      Bs[buf][sk + j][sr] = rb[j];
    }
  };
  f4 acc[2][4];
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int u = 0; u < 4; ++u) acc[t][u] = f4{0.0f, 0.0f, 0.0f, 0.0f};
  const int n_chunks = K / 16;
  fetch(0);
  stash(0);
  __syncthreads();
  for (int ch = 0; ch < n_chunks; ++ch) {
    const int cur = ch & 1;
    if (ch + 1 < n_chunks) fetch(16 * (ch + 1));
#pragma unroll
    for (int st = 0; st < 4; ++st) {
      const int k = 4 * st + kk;
      float a[2], b[4];
#pragma unroll
      for (int t = 0; t < 2; ++t) a[t] = As[cur][k][wq * 32 + 16 * t + ll];
#pragma unroll
      for (int u = 0; u < 4; ++u) b[u] = Bs[cur][k][wc * 64 + 16 * u + ll];
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int u = 0; u < 4; ++u) acc[t][u] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[t], b[u], acc[t][u], 0, 0, 0);
    }
    if (ch + 1 < n_chunks) stash(cur ^ 1);
    __syncthreads();
  }
  // residual form: this thread's 2 x 4 rows x 4 columns of the FP64 base
  double bsum[2][4][4] = {};
  if (ACT == 2 && Bb) {
    for (int j = 0; j < nbase; ++j) {
      double uj[2][4], bj[4];
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int m = m0 + wq * 32 + 16 * t + 4 * kk + i;
          uj[t][i] = m < M ? Ub[(int64_t)m * nbase + j] : 0.0;
        }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int n = n0 + wc * 64 + 16 * u + ll;
        bj[u] = n < N ? Bb[(int64_t)j * N + n] : 0.0;
      }
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int u = 0; u < 4; ++u) bsum[t][i][u] = fma(uj[t][i], bj[u], bsum[t][i][u]);
    }
  }
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int m = m0 + wq * 32 + 16 * t + 4 * kk + i;
      if (m >= M) continue;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int n = n0 + wc * 64 + 16 * u + ll;
        if (n >= N) continue;
        float v = acc[t][u][i] + (bias ? bias[n] : 0.0f);
        if (ACT == 2) {
          Y64[(int64_t)m * ldc + n] = (double)mu[n] + (double)sd[n] * (double)v + bsum[t][i][u];
          continue;
        }
        if (Z) Z[(int64_t)m * ldc + n] = v;
        if (ACT == 1) v = v / (1.0f + __expf(-v));
        C[(int64_t)m * ldc + n] = v;
      }
    }
}

// One product of the training step, C[m][n] = sum_k A(m,k) B(k,n), with what
// follows it.  ak: A is A[m * lda + k], else A[k * lda + m]; bk: B is
// B[n * ldb + k], else B[k * ldb + n].
struct Product {
  int M, N, K;
  const float *A, *B;
  int64_t lda, ldb;
  const float *bias;
  int epi;               // kLinear .. kLayer1Back
  float *C, *Z;          // [M][N] outputs (Z: pre-activations of kSilu, may be null)
  const float *aux;      // kSiluBack / kLayer1Back: Z [M][N]; kLoss: targets [M][N]
  float scale;           // kLoss: 1 / count
  double *part;          // kLoss: one partial sum of squares per tile
  float *colsum;         // not null (A given by columns): sum_k A(m,k) [M]
  const float *X;        // kLayer1Back: inputs [M][n_in]
  int n_in;
  float *part1;          // kLayer1Back: per row tile [N][n_in + 1] partial gradients of W1 and b1
};
enum { kLinear = 0, kSilu, kLoss, kSiluBack, kLayer1Back };
constexpr int kMaxIn1 = 7;             // inputs that kLayer1Back takes (n_in + 1 <= 8 sums per column)

// dH silu'(z), silu'(z) = s (1 + z (1 - s)), s = 1 / (1 + e^-z).
__device__ __forceinline__ float silu_back(float dh, float z) {
  const float s = 1.0f / (1.0f + __expf(-z));
  return dh * s * (1.0f + z * (1.0f - s));
}

// LDS of one product's workgroup: two buffers of both operands' chunks, rows
// of 32 k padded to 36 floats (a wave's 16-byte fragment reads then cover the
// banks evenly); the tile of kLayer1Back and the reductions reuse it.
constexpr int kPK = 36;
template <int T>
struct ProductLds {
  float A[2][32 * T][kPK], B[2][32 * T][kPK];
};

// One (32 T) x (32 T) tile of a product by a workgroup of four waves (2 x 2),
// each T x T tiles of 16 x 16 on v_mfma_f32_16x16x4f32.  With 32 x 32 tiles the
// batch of 1024 samples fills the chip (576 workgroups for the output layer's
// two products, 28 us for 1.34 GFLOP) but reads 167 MB through L2, which bounds
// it: four chunks in flight instead of two took the same time.  A fragment read of 16
// bytes is four consecutive k of one row, so MFMA step s of a 16-deep group
// multiplies k = s, 4 + s, 8 + s, 12 + s of it.  The next D chunks of 32 k
// are in flight in registers; the k past the last full chunk are loaded first,
// zeroed beyond the operand, and multiplied last (up to 16 of them as one group:
// 65,536 rows of 8 terms and 1275 outputs, bound by latency, 124 to 108 us for the
// forward pass).
template <int T, bool AK, bool BK, bool VEC>
__device__ __forceinline__ void product_tile(const Product &p, int tile, ProductLds<T> &lds) {
  constexpr int TM = 32 * T;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wq = wave & 1, wc = wave >> 1, kk = lane >> 4, ll = lane & 15;
  const int n_nt = (p.N + TM - 1) / TM;
  const int tm = tile / n_nt, tn = tile - tm * n_nt;
  const int m0 = tm * TM, n0 = tn * TM;
  // this thread's quads of four consecutive k: rows of the tile and first k;
  // rows past the operand read its last row (their outputs are not stored)
  auto row_of = [&](bool k_major, int u) { return k_major ? (tid >> 3) + 32 * u : (tid & 31) + 32 * u; };
  auto quad_of = [&](bool k_major) { return 4 * (k_major ? (tid & 7) : (tid >> 5)); };
  auto start = [&](const float *P, int64_t ld, bool k_major, int R, int r) {
    const int64_t rc = r < R ? r : R - 1;
    return k_major ? P + rc * ld + quad_of(true) : P + quad_of(false) * ld + rc;
  };
  const float *pa[T], *pb[T];
#pragma unroll
  for (int u = 0; u < T; ++u) {
    pa[u] = start(p.A, p.lda, AK, p.M, m0 + row_of(AK, u));
    pb[u] = start(p.B, p.ldb, BK, p.N, n0 + row_of(BK, u));
  }
  const int n_full = p.K / 32, tail = p.K - 32 * n_full;
  auto load = [&](const float *P, int64_t ld, bool k_major, int ch) {
    f4 v;
    if (k_major) {
      const float *q = P + 32 * ch;
      if (VEC) return *reinterpret_cast<const f4 *>(q);
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = q[j];
    } else {
      const float *q = P + 32 * ch * ld;
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = q[j * ld];
    }
    return v;
  };
  // the k past the last full chunk, zero beyond the operand
  auto load_tail = [&](const float *P, int64_t ld, bool k_major) {
    const int k = quad_of(k_major);
    const int64_t step = k_major ? 1 : ld;
    const float *q = P + 32 * n_full * step;
    f4 v;
    if (k_major && VEC) {                // K % 4 == 0: a quad is whole or beyond the end
      v = *reinterpret_cast<const f4 *>(k < tail ? q : q - k);
      return k < tail ? v : f4{0.0f, 0.0f, 0.0f, 0.0f};
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const bool in = k + j < tail;
      const float x = q[in ? j * step : -(int64_t)k * step];
      v[j] = in ? x : 0.0f;
    }
    return v;
  };
  constexpr int D = 2;
  f4 ra[D][T], rb[D][T], ta[T], tb[T];
  auto fetch = [&](int ch, f4 *a, f4 *b) {
    const int cc = ch < n_full ? ch : n_full - 1;      // past the end the last chunk again, not used
#pragma unroll
    for (int u = 0; u < T; ++u) {
      a[u] = load(pa[u], p.lda, AK, cc);
      b[u] = load(pb[u], p.ldb, BK, cc);
    }
  };
  float cs[T] = {};
  auto stash = [&](int buf, const f4 *a, const f4 *b) {
    asm volatile("" ::: "memory");
#pragma unroll
    for (int u = 0; u < T; ++u) {
      *reinterpret_cast<f4 *>(&lds.A[buf][row_of(AK, u)][quad_of(AK)]) = a[u];
      *reinterpret_cast<f4 *>(&lds.B[buf][row_of(BK, u)][quad_of(BK)]) = b[u];
    }
  };
  auto add_columns = [&](const f4 *a) {
    if (!AK)
#pragma unroll
      for (int u = 0; u < T; ++u) cs[u] += (a[u][0] + a[u][1]) + (a[u][2] + a[u][3]);
  };
  f4 acc[2][T][T];
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
      for (int u = 0; u < T; ++u) acc[h][t][u] = f4{0.0f, 0.0f, 0.0f, 0.0f};
  auto multiply = [&](int buf, int halves = 2) {    // groups of 16 k of the chunk
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if (h >= halves) break;
      f4 a[T], b[T];
#pragma unroll
      for (int t = 0; t < T; ++t)
        a[t] = *reinterpret_cast<const f4 *>(&lds.A[buf][wq * 16 * T + 16 * t + ll][16 * h + 4 * kk]);
#pragma unroll
      for (int u = 0; u < T; ++u)
        b[u] = *reinterpret_cast<const f4 *>(&lds.B[buf][wc * 16 * T + 16 * u + ll][16 * h + 4 * kk]);
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
          for (int u = 0; u < T; ++u)
            acc[h][t][u] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[t][s], b[u][s], acc[h][t][u], 0, 0, 0);
    }
  };
  if (tail > 0) {
#pragma unroll
    for (int u = 0; u < T; ++u) {
      ta[u] = load_tail(pa[u], p.lda, AK);
      tb[u] = load_tail(pb[u], p.ldb, BK);
    }
  }
  if (n_full > 0) {
    // register set c % D and LDS buffer c % 2 hold chunk c; chunks c + 1 .. c + D
    // are on their way
#pragma unroll
    for (int i = 0; i < D; ++i) fetch(i, ra[i], rb[i]);
    stash(0, ra[0], rb[0]);
    add_columns(ra[0]);
    fetch(D, ra[0], rb[0]);
    __syncthreads();
    auto step = [&](int c, int i) {
      const int n = (i + 1) % D;
      multiply(i & 1);
      if (c + 1 < n_full) {
        stash((i + 1) & 1, ra[n], rb[n]);
        add_columns(ra[n]);
      }
      fetch(c + 1 + D, ra[n], rb[n]);
      __syncthreads();
    };
    for (int c = 0; c < n_full; c += D) {
#pragma unroll
      for (int i = 0; i < D; ++i)
        if (c + i < n_full) step(c + i, i);
    }
  }
  if (tail > 0) {
    stash(0, ta, tb);
    add_columns(ta);
    __syncthreads();
    multiply(0, tail <= 16 ? 1 : 2);
    __syncthreads();
  }
  if (!AK && p.colsum != nullptr && tn == 0) {
    // eight threads hold partial sums of each row of the tile
    float *red = &lds.A[0][0][0];
#pragma unroll
    for (int u = 0; u < T; ++u) red[(tid >> 5) * TM + row_of(false, u)] = cs[u];
    __syncthreads();
    if (tid < TM && m0 + tid < p.M) {
      float v = 0.0f;
      for (int j = 0; j < 8; ++j) v += red[j * TM + tid];
      p.colsum[m0 + tid] = v;
    }
    __syncthreads();
  }
  // a tile's columns' biases ahead of the stores, which the compiler has to keep
  // them behind otherwise: one load after another for each of the outputs
  const bool biased = p.epi <= kLoss && p.bias != nullptr;
  float bias[T] = {};
  if (biased)
#pragma unroll
    for (int u = 0; u < T; ++u) bias[u] = p.bias[min(n0 + wc * 16 * T + 16 * u + ll, p.N - 1)];
  double sq = 0.0;
  float *ds = &lds.A[0][0][0];           // kLayer1Back: dZ1 of the tile, [TM][TM + 1]
  static_assert(sizeof(ProductLds<T>) >= sizeof(float) * (32 * T) * (32 * T + 1), "the tile fits the chunks' LDS");
#pragma unroll
  for (int t = 0; t < T; ++t)
#pragma unroll
    for (int u = 0; u < T; ++u)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int mr = wq * 16 * T + 16 * t + 4 * kk + i, nc = wc * 16 * T + 16 * u + ll;
        const int m = m0 + mr, n = n0 + nc;
        const bool in = m < p.M && n < p.N;
        const int64_t at = (int64_t)m * p.N + n;
        float v = acc[0][t][u][i] + acc[1][t][u][i];
        if (biased) v += bias[u];
        if (p.epi == kLinear) {
          if (in) p.C[at] = v;
        } else if (p.epi == kSilu) {
          if (in) {
            if (p.Z) p.Z[at] = v;
            p.C[at] = v / (1.0f + __expf(-v));
          }
        } else if (p.epi == kLoss) {
          const float r = in ? v - p.aux[at] : 0.0f;
          if (in) p.C[at] = 2.0f * r * p.scale;
          sq += (double)r * (double)r;
        } else if (p.epi == kSiluBack) {
          if (in) p.C[at] = silu_back(v, p.aux[at]);
        } else {
          ds[mr * (TM + 1) + nc] = in ? silu_back(v, p.aux[at]) : 0.0f;
        }
      }
  if (p.epi == kLoss) {
    double *red = reinterpret_cast<double *>(&lds.A[0][0][0]);
    for (int o = 32; o > 0; o >>= 1) sq += __shfl_xor(sq, o, 64);
    if (lane == 0) red[wave] = sq;
    __syncthreads();
    if (tid == 0) p.part[tile] = (red[0] + red[1]) + (red[2] + red[3]);
  } else if (p.epi == kLayer1Back) {
    __syncthreads();
    const int sums = p.n_in + 1;
    for (int e = tid; e < TM * sums; e += kT) {
      const int nc = e % TM, i = e / TM;
      if (n0 + nc >= p.N) continue;
      float v = 0.0f;
      for (int r = 0; r < TM && m0 + r < p.M; ++r)
        v += ds[r * (TM + 1) + nc] * (i < p.n_in ? p.X[(int64_t)(m0 + r) * p.n_in + i] : 1.0f);
      p.part1[((int64_t)tm * p.N + n0 + nc) * sums + i] = v;
    }
  }
}

template <int T, bool AK, bool BK, bool VEC>
__global__ void __launch_bounds__(kT) k_product(Product p) {
  __shared__ ProductLds<T> lds;
  // workgroups are dealt to the 8 XCDs in turn: a contiguous range of tiles on
  // each, so that the column tiles of a row tile share an XCD's L2 (65,536 rows of
  // 40 terms and 1275 outputs: 209 to 188 us for the whole forward pass)
  const int64_t nblk = gridDim.x, bx = blockIdx.x, xcd = bx & 7, base = nblk >> 3, extra = nblk & 7;
  product_tile<T, AK, BK, VEC>(p, (int)(xcd * base + (xcd < extra ? xcd : extra) + (bx >> 3)), lds);
}

// Two products of one stage of the backward pass in one launch: workgroups
// below n_w take the weight gradient w (both operands by columns), the others
// the input gradient x (VEC: its rows of A in aligned float4s).
// The weight gradient keeps 32 x 32 tiles at any batch: its sums run over the
// batch, so a tile is the longest chain of the launch.
template <int T, bool VEC>
__global__ void __launch_bounds__(kT) k_product_pair(Product w, Product x, int n_w) {
  __shared__ union {
    ProductLds<1> w;
    ProductLds<T> x;
  } lds;
  if ((int)blockIdx.x < n_w) product_tile<1, false, false, false>(w, blockIdx.x, lds.w);
  else product_tile<T, true, false, VEC>(x, blockIdx.x - n_w, lds.x);
}

// First layer for few inputs: Z[b][h] = b1[h] + sum_i W1[h][i] X[b][i], H =
// silu(Z).  A thread keeps one output's weights and goes through the rows
// blockIdx.x R .. + R - 1 (every `par`-th, where the block holds several rows of
// few outputs), so that it is bound by the stores: 65,536 rows of 256 outputs
// 17.6 us, 100 with one output per thread and its index divided out, 26 with the
// input count a variable, whose loads wait one for the other (64 outputs: 12.2
// and 15).
template <int IN>
__global__ void __launch_bounds__(kT) k_layer1(const float *__restrict__ X, int B, int hid, int R, int par,
                                               const float *__restrict__ W1, const float *__restrict__ b1,
                                               float *__restrict__ Z, float *__restrict__ H) {
  const int sub = par > 1 ? (int)threadIdx.x / hid : 0;
  const int h = (int)(blockIdx.y * kT + threadIdx.x) - sub * hid;
  if (h >= hid || sub >= par) return;
  float w[IN];
#pragma unroll
  for (int i = 0; i < IN; ++i) w[i] = W1[(int64_t)h * IN + i];
  const float bias = b1[h];
  const int end = min(B, ((int)blockIdx.x + 1) * R);
#pragma unroll 8
  for (int b = blockIdx.x * R + sub; b < end; b += par) {
    const float *x = X + (int64_t)b * IN;
    float v = 0.0f;
#pragma unroll
    for (int i = 0; i < IN; ++i) v = fmaf(x[i], w[i], v);
    v += bias;
    const int64_t e = (int64_t)b * hid + h;
    if (Z) Z[e] = v;
    H[e] = v / (1.0f + __expf(-v));
  }
}

// Gradients of W1 [hid][n_in] and b1 [hid] from the row tiles' partial sums
// part1[tile][hid][n_in + 1], tiles in order.
__global__ void __launch_bounds__(kT) k_layer1_sum(const float *__restrict__ part1, int tiles, int hid, int n_in,
                                                   float *__restrict__ gw1, float *__restrict__ gb1) {
  const int e = blockIdx.x * kT + threadIdx.x;
  const int sums = n_in + 1;
  if (e >= hid * sums) return;
  float v = 0.0f;
#pragma unroll 8
  for (int t = 0; t < tiles; ++t) v += part1[(int64_t)t * hid * sums + e];
  const int h = e / sums, i = e - h * sums;
  if (i < n_in) gw1[(int64_t)h * n_in + i] = v;
  else gb1[h] = v;
}

// *out = scale * sum of part[0, n) (one workgroup, fixed order); out is pinned host memory.
__global__ void __launch_bounds__(kT) k_sum_parts(const double *__restrict__ part, int n, double scale,
                                                  double *out) {
  __shared__ double red[kT / 64];
  double s = 0.0;
  for (int i = threadIdx.x; i < n; i += kT) s += part[i];
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) *out = ((red[0] + red[1]) + (red[2] + red[3])) * scale;
}

// Y[b][c] = mu[c] + sd[c] y[b][c] in FP64 (row stride ldy) from FP32 y [B][out],
// plus the FP64 base sum_j Ub[b][j] Bb[j][c] of the residual form when Bb is set.
__global__ void __launch_bounds__(kT) k_unstandardise(const float *__restrict__ y, int64_t B, int out,
                                                      const float *__restrict__ mu, const float *__restrict__ sd,
                                                      double *__restrict__ Y, int64_t ldy,
                                                      const double *__restrict__ Ub, const double *__restrict__ Bb,
                                                      int nbase) {
  const int64_t e = (int64_t)blockIdx.x * kT + threadIdx.x;
  if (e >= B * out) return;
  const int64_t b = e / out;
  const int c = (int)(e - b * out);
  double base = 0.0;
  if (Bb)
    for (int j = 0; j < nbase; ++j) base = fma(Ub[b * nbase + j], Bb[(int64_t)j * out + c], base);
  Y[b * ldy + c] = (double)mu[c] + (double)sd[c] * (double)y[e] + base;
}

__global__ void k_adam(float *__restrict__ p, const float *__restrict__ g, float *__restrict__ m,
                       float *__restrict__ v, int64_t n, float lr, float b1, float b2, float eps, float bc1,
                       float bc2) {
  const int64_t e = (int64_t)blockIdx.x * kT + threadIdx.x;
  if (e >= n) return;
  const float ge = g[e];
  const float me = b1 * m[e] + (1.0f - b1) * ge;
  const float ve = b2 * v[e] + (1.0f - b2) * ge * ge;
  m[e] = me;
  v[e] = ve;
  p[e] -= lr * (me / bc1) / (sqrtf(ve / bc2) + eps);
}

inline unsigned blocks(int64_t n) { return (unsigned)((n + kT - 1) / kT); }

}  // namespace

void Mlp::init(int n_in, int hidden, int n_out, const double *normals) {
  in = n_in;
  hid = hidden;
  out = n_out;
  o_w1 = 0;
  o_b1 = o_w1 + (int64_t)hid * in;
  o_w2 = o_b1 + hid;
  o_b2 = o_w2 + (int64_t)hid * hid;
  o_w3 = o_b2 + hid;
  o_b3 = o_w3 + (int64_t)out * hid;
  np = o_b3 + out;
  std::vector<float> h(np, 0.0f);
  for (int64_t i = 0; i < (int64_t)hid * in; ++i) h[o_w1 + i] = (float)(normals[o_w1 + i] / sqrt((double)in));
  for (int64_t i = 0; i < (int64_t)hid * hid; ++i) h[o_w2 + i] = (float)(normals[o_w2 + i] / sqrt((double)hid));
  for (int64_t i = 0; i < (int64_t)out * hid; ++i) h[o_w3 + i] = (float)(normals[o_w3 + i] / sqrt((double)hid));
  p.alloc(np);
  g.alloc(np);
  m.alloc(np);
  v.alloc(np);
  RBFL_HIP(hipMemcpy(p.p, h.data(), sizeof(float) * np, hipMemcpyHostToDevice));
  RBFL_HIP(hipMemset(g.p, 0, sizeof(float) * np));
  RBFL_HIP(hipMemset(m.p, 0, sizeof(float) * np));
  RBFL_HIP(hipMemset(v.p, 0, sizeof(float) * np));
  if (!loss) RBFL_HIP(hipHostMalloc(reinterpret_cast<void **>(&loss), sizeof(double), hipHostMallocDefault));
  *loss = 0.0;
  t = 0;
}

void Mlp::reserve(int64_t B) {
  if (B <= cap) return;
  cap = 0;                 // a failed growth leaves no capacity behind
  Z1.alloc((size_t)B * hid);
  H1.alloc((size_t)B * hid);
  Z2.alloc((size_t)B * hid);
  H2.alloc((size_t)B * hid);
  Yb.alloc((size_t)B * out);
  dY.alloc((size_t)B * out);
  dA.alloc((size_t)B * hid);
  dB.alloc((size_t)B * hid);
  cap = B;
}

// Work space of loss_grad for B samples: the loss tiles' partial sums (fewer
// than 2048 tiles of 32 x 32, else tiles of 64 x 64, see tile_of) and the row
// tiles' partial gradients of the first layer.
void Mlp::reserve_grad(int64_t B) {
  reserve(B);
  if (B <= grad_cap) return;
  grad_cap = 0;
  part.alloc((size_t)std::max<int64_t>(2048, (B + 63) / 64 * ((out + 63) / 64)));
  if (in <= kMaxIn1) part1.alloc((size_t)((B + 31) / 32) * hid * (in + 1));
  grad_cap = B;
}

// Whether k_gemm_f32_nt applies: both operands contiguous in k, K a multiple
// of its 16-deep chunks, rows of 16-byte aligned float4s.
static bool nt_ok(int K, const float *A, int64_t sam, int64_t sak, const float *B, int64_t sbk, int64_t sbn) {
  const bool aligned = ((reinterpret_cast<uintptr_t>(A) | reinterpret_cast<uintptr_t>(B)) & 15) == 0;
  return sak == 1 && sbk == 1 && K % 16 == 0 && sam % 4 == 0 && sbn % 4 == 0 && aligned;
}

// Tile of a product in units of 32: tiles of 64 x 64 once there are two per
// CU, else 32 x 32 (B = 1024, 256 x 1275 outputs of 1024 or 1275 terms: 320 and
// 256 workgroups instead of 80 and 64).
static int64_t tiles(int64_t M, int64_t N, int t) { return (M + 32 * t - 1) / (32 * t) * ((N + 32 * t - 1) / (32 * t)); }
static int tile_of(int64_t tiles64) { return tiles64 >= 512 ? 2 : 1; }

static bool rows16(const float *P, int64_t ld, int K) {
  return K % 4 == 0 && ld % 4 == 0 && (reinterpret_cast<uintptr_t>(P) & 15) == 0;
}

// A forward layer C = act(A B^T + bias): A [M][K] (row stride lda), B [N][K].
static void layer(int epi, int M, int N, int K, const float *A, int64_t lda, const float *B, const float *bias,
                  float *Z, float *C, hipStream_t s, const float *target = nullptr, double *part = nullptr) {
  if (epi != kLoss && tiles(M, N, 4) >= 256 && nt_ok(K, A, lda, 1, B, 1, K)) {
    dim3 g((unsigned)tiles(M, N, 4));
    if (epi == kSilu)
      hipLaunchKernelGGL(k_gemm_f32_nt<1>, g, dim3(512), 0, s, M, N, K, A, lda, B, (int64_t)K, bias, Z, C, (int64_t)N,
                         nullptr, nullptr, nullptr, nullptr, nullptr, 0);
    else
      hipLaunchKernelGGL(k_gemm_f32_nt<0>, g, dim3(512), 0, s, M, N, K, A, lda, B, (int64_t)K, bias, Z, C, (int64_t)N,
                         nullptr, nullptr, nullptr, nullptr, nullptr, 0);
    RBFL_HIP(hipGetLastError());
    return;
  }
  Product p{};
  p.M = M;
  p.N = N;
  p.K = K;
  p.A = A;
  p.lda = lda;
  p.B = B;
  p.ldb = K;
  p.bias = bias;
  p.epi = epi;
  p.Z = Z;
  p.C = C;
  p.aux = target;
  p.part = part;
  p.scale = (float)(1.0 / ((double)M * N));
  const bool vec = rows16(A, lda, K) && rows16(B, K, K);
  const int t = tile_of(tiles(M, N, 2));
  const dim3 g((unsigned)tiles(M, N, t));
  if (t == 2) {
    if (vec) hipLaunchKernelGGL((k_product<2, true, true, true>), g, dim3(kT), 0, s, p);
    else hipLaunchKernelGGL((k_product<2, true, true, false>), g, dim3(kT), 0, s, p);
  } else {
    if (vec) hipLaunchKernelGGL((k_product<1, true, true, true>), g, dim3(kT), 0, s, p);
    else hipLaunchKernelGGL((k_product<1, true, true, false>), g, dim3(kT), 0, s, p);
  }
  RBFL_HIP(hipGetLastError());
}

// One stage of the backward pass: with dZ [B][n] the gradient at a layer's
// pre-activations, H [B][m] its inputs and W [n][m] its weights, dW = dZ^T H,
// db = the column sums of dZ and (epi not kLinear) the gradient at the inputs'
// pre-activations dZ W * silu'(Z), in one launch.
static int backward(int B, int n, int m, const float *dZ, const float *H, float *dW, float *db, const float *W, int epi,
                    const float *Z, float *dZin, const float *X, int n_in, float *part1, hipStream_t s) {
  Product w{}, x{};
  w.M = n;
  w.N = m;
  w.K = B;
  w.A = dZ;
  w.lda = n;
  w.B = H;
  w.ldb = m;
  w.epi = kLinear;
  w.C = dW;
  w.colsum = db;
  x.M = B;
  x.N = m;
  x.K = n;
  x.A = dZ;
  x.lda = n;
  x.B = W;
  x.ldb = m;
  x.epi = epi;
  x.C = dZin;
  x.aux = Z;
  x.X = X;
  x.n_in = n_in;
  x.part1 = part1;
  const bool both = epi != kLinear;
  const int t = tile_of(both ? tiles(B, m, 2) : 0);
  const int n_w = (int)tiles(n, m, 1);
  const dim3 g((unsigned)(n_w + (both ? tiles(B, m, t) : 0)));
  const bool vec = rows16(dZ, n, n);
  if (t == 2) {
    if (vec) hipLaunchKernelGGL((k_product_pair<2, true>), g, dim3(kT), 0, s, w, x, n_w);
    else hipLaunchKernelGGL((k_product_pair<2, false>), g, dim3(kT), 0, s, w, x, n_w);
  } else {
    if (vec) hipLaunchKernelGGL((k_product_pair<1, true>), g, dim3(kT), 0, s, w, x, n_w);
    else hipLaunchKernelGGL((k_product_pair<1, false>), g, dim3(kT), 0, s, w, x, n_w);
  }
  RBFL_HIP(hipGetLastError());
  return (B + 32 * t - 1) / (32 * t);    // row tiles of the input gradient
}

// Z1 (may be null) and H1 of the first layer.
static void layer1(const Mlp &m, const float *X, int B, float *Z1, float *H1, hipStream_t s) {
  if (m.in > kMaxIn1) {
    layer(kSilu, B, m.hid, m.in, X, m.in, m.p.p + m.o_w1, m.p.p + m.o_b1, Z1, H1, s);
    return;
  }
  // rows of a workgroup: several at once while the outputs are few, and enough
  // in turn to leave eight workgroups per CU
  const int par = std::max(1, kT / m.hid), cols = (m.hid + kT - 1) / kT;
  const int R = std::max(1, B * cols / (2048 * par)) * par;
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3((B + R - 1) / R, cols), dim3(kT), 0, s, X, B, m.hid, R, par, m.p.p + m.o_w1,
                       m.p.p + m.o_b1, Z1, H1);
  };
  static_assert(kMaxIn1 == 7, "one kernel per input count");
  switch (m.in) {
    case 1: launch(k_layer1<1>); break;
    case 2: launch(k_layer1<2>); break;
    case 3: launch(k_layer1<3>); break;
    case 4: launch(k_layer1<4>); break;
    case 5: launch(k_layer1<5>); break;
    case 6: launch(k_layer1<6>); break;
    default: launch(k_layer1<7>);
  }
  RBFL_HIP(hipGetLastError());
}

void Mlp::forward(const float *X, int64_t B, float *Y, hipStream_t s) {
  reserve(B);
  const int b = (int)B;
  layer1(*this, X, b, nullptr, H1.p, s);
  layer(kSilu, b, hid, hid, H1.p, hid, p.p + o_w2, p.p + o_b2, nullptr, H2.p, s);
  layer(kLinear, b, out, hid, H2.p, hid, p.p + o_w3, p.p + o_b3, nullptr, Y, s);
}

void Mlp::infer(const float *X, int64_t B, const float *mu, const float *sd, double *Y, int64_t ldy, hipStream_t s,
                const double *Ub, const double *Bb, int nbase) {
  reserve(B);
  const int b = (int)B;
  layer1(*this, X, b, nullptr, H1.p, s);
  layer(kSilu, b, hid, hid, H1.p, hid, p.p + o_w2, p.p + o_b2, nullptr, H2.p, s);
  const float *W3 = p.p + o_w3;
  if (nt_ok(hid, H2.p, hid, 1, W3, 1, hid)) {
    dim3 g((unsigned)((int64_t)((out + 127) / 128) * ((b + 127) / 128)));
    hipLaunchKernelGGL(k_gemm_f32_nt<2>, g, dim3(512), 0, s, b, out, hid, H2.p, (int64_t)hid, W3, (int64_t)hid,
                       p.p + o_b3, nullptr, nullptr, ldy, mu, sd, Y, Ub, Bb, nbase);
    RBFL_HIP(hipGetLastError());
    return;
  }
  layer(kLinear, b, out, hid, H2.p, hid, W3, p.p + o_b3, nullptr, Yb.p, s);
  hipLaunchKernelGGL(k_unstandardise, dim3((unsigned)(((int64_t)b * out + kT - 1) / kT)), dim3(kT), 0, s, Yb.p,
                     (int64_t)b, out, mu, sd, Y, ldy, Ub, Bb, nbase);
  RBFL_HIP(hipGetLastError());
}

// Forward pass, mean-squared error and every gradient.  A batch of about a
// thousand samples is a few microseconds of matrix products each and mostly
// waits for launches and chains, so what is elementwise runs in the products'
// own epilogues: the loss and dY in the output layer's, silu' in the input
// gradients', the bias gradients in the weight gradients', the first layer's
// gradients as partial sums of the tiles of dZ1 (never stored); and each
// stage's two products share a launch: 1024 samples of 4 - 256 - 256 - 1275 take
// 86 us in 8 launches, 1.69 ms in 17 with separate elementwise kernels, 64 x 64
// tiles on 16 to 80 workgroups and one thread per column sum.
void Mlp::loss_grad(const float *X, const float *T, int64_t B, hipStream_t s) {
  reserve_grad(B);
  const int b = (int)B;
  layer1(*this, X, b, Z1.p, H1.p, s);
  layer(kSilu, b, hid, hid, H1.p, hid, p.p + o_w2, p.p + o_b2, Z2.p, H2.p, s);
  layer(kLoss, b, out, hid, H2.p, hid, p.p + o_w3, p.p + o_b3, nullptr, dY.p, s, T, part.p);
  hipLaunchKernelGGL(k_sum_parts, dim3(1), dim3(kT), 0, s, part.p, (int)tiles(b, out, tile_of(tiles(b, out, 2))),
                     1.0 / ((double)B * out), loss);
  RBFL_HIP(hipGetLastError());
  // layer 3: dW3, db3, dZ2; layer 2: dW2, db2 and dZ1 or, for few inputs, the
  // first layer's gradients
  backward(b, out, hid, dY.p, H2.p, g.p + o_w3, g.p + o_b3, p.p + o_w3, kSiluBack, Z2.p, dB.p, nullptr, 0, nullptr, s);
  if (in <= kMaxIn1) {
    const int row_tiles = backward(b, hid, hid, dB.p, H1.p, g.p + o_w2, g.p + o_b2, p.p + o_w2, kLayer1Back, Z1.p,
                                   nullptr, X, in, part1.p, s);
    hipLaunchKernelGGL(k_layer1_sum, dim3(blocks((int64_t)hid * (in + 1))), dim3(kT), 0, s, part1.p, row_tiles, hid, in,
                       g.p + o_w1, g.p + o_b1);
    RBFL_HIP(hipGetLastError());
    return;
  }
  backward(b, hid, hid, dB.p, H1.p, g.p + o_w2, g.p + o_b2, p.p + o_w2, kSiluBack, Z1.p, dA.p, nullptr, 0, nullptr, s);
  backward(b, hid, in, dA.p, X, g.p + o_w1, g.p + o_b1, nullptr, kLinear, nullptr, nullptr, nullptr, 0, nullptr, s);
}

void Mlp::adam(double lr, double b1, double b2, double eps, hipStream_t s) {
  ++t;
  const float bc1 = (float)(1.0 - pow(b1, t)), bc2 = (float)(1.0 - pow(b2, t));
  hipLaunchKernelGGL(k_adam, dim3(blocks(np)), dim3(kT), 0, s, p.p, g.p, m.p, v.p, np, (float)lr, (float)b1,
                     (float)b2, (float)eps, bc1, bc2);
  RBFL_HIP(hipGetLastError());
}

}  // namespace rbfl
