// Per-proposal setup of the online stage's epilogue (Sec. II D): domain
// flags, each detector's arrival-time position in the window and each
// (detector, mode) amplitude of Eq. logl_complete (corrected reading); and the
// reduction of one proposal's interpolated outputs to ln L.
// Shared by the epilogue kernels and the contraction kernels that finish
// ln L in their own epilogues.
#pragma once

#include "rbfl_internal.h"
#include "rbfl_math.h"

namespace rbfl {

struct EpiSetup {
  int status;                       // 0 evaluate, 1 outside the domain (-inf), 2 NaN input
  int event;                        // multi-event batches: the proposal's event
  int n0[RBFL_MAX_DET];             // spline stencil base sample per detector
  double f[RBFL_MAX_DET];           // fractional sample position per detector
  double rr;                        // d_ref / d_L
  double Ar[RBFL_MAX_DET][RBFL_MAX_MODES], Ai[RBFL_MAX_DET][RBFL_MAX_MODES];
};

// a1 for proposal g: loads its 11 parameters into p; 2 for a NaN input, else
// 1 outside the ellipsoid or the physical region, else 0.
__device__ __forceinline__ int epi_prelude(const EvalConsts &c, const double *__restrict__ params, int64_t ld,
                                           int64_t g, double p[11]) {
  bool any_nan = false;
#pragma unroll
  for (int i = 0; i < 11; ++i) {
    p[i] = params[i * ld + g];
    any_nan |= isnan(p[i]);
  }
  if (any_nan) return 2;
  double r2 = 0.0;
  for (int d = 0; d < 4; ++d) {
    const double x = p[d] / c.semi[d];
    r2 += x * x;
  }
  bool valid = r2 <= 1.0;
  {
    double th[4], phys[4];
    for (int i = 0; i < 4; ++i) {
      double t = c.theta_c[i];
      for (int j = 0; j < 4; ++j) t += c.V[4 * i + j] * p[j];
      th[i] = t;
    }
    valid = valid && theta_to_phys(th, c.f0, c.chi_max, phys);
  }
  return valid ? 0 : 1;
}

__device__ __forceinline__ void epi_setup(const EvalConsts &c, const double *__restrict__ params, int64_t ld,
                                          int64_t g, EpiSetup &o) {
  double p[11];
  const int pre = epi_prelude(c, params, ld, g, p);
  if (pre == 2) {
    o.status = 2;
    return;
  }
  bool valid = pre == 0;
  const double alpha = p[4], dec = p[5], psi = p[6], iota = p[7], phi = p[8], tc = p[9], dl = p[10];
  o.rr = c.d_ref / dl;
  double ch, sh;
  sincos(0.5 * iota, &sh, &ch);
  double ynr[RBFL_MAX_MODES], yni[RBFL_MAX_MODES], ypr[RBFL_MAX_MODES], ypi[RBFL_MAX_MODES];
  for (int a = 0; a < c.n_modes; ++a) {
    eval_ylm(c.ylm_neg[a], ch, sh, phi, &ynr[a], &yni[a]);
    eval_ylm(c.ylm_pos[a], ch, sh, phi, &ypr[a], &ypi[a]);
  }
  const int T = c.T;
  for (int k = 0; k < c.n_det; ++k) {
    // a4: detector response, arrival time and spline stencil
    double fp, fc, dt;
    detector_response(c.D[k], c.r[k], alpha, dec, psi, &fp, &fc, &dt);
    const double s = (tc + dt - c.t_trig) * c.fs + (double)c.half_w;
    const double fl = floor(s);
    valid = valid && fl >= 4.0 && fl <= (double)(T - 6);
    o.n0[k] = valid ? (int)fl : 4;
    o.f[k] = s - fl;
    // a6: amplitudes of every mode at this detector
    for (int a = 0; a < c.n_modes; ++a) {
      const double sg = (c.mode_l[a] & 1) ? -1.0 : 1.0;
      o.Ar[k][a] = 0.5 * ((fp * ynr[a] - fc * yni[a]) + sg * (fp * ypr[a] - fc * ypi[a]));
      o.Ai[k][a] = 0.5 * ((fp * yni[a] + fc * ynr[a]) + sg * (-fp * ypi[a] - fc * ypr[a]));
    }
  }
  o.status = valid ? 0 : 1;
}

// Weight of one interpolated output in ln L = sum_c w_c Y[c] (Eq.
// logl_complete, corrected reading, frozen antenna patterns) for a proposal
// with setup o, r = d_ref / d_L, amplitudes A_{k,a} and spline position
// n0 + f at detector k.  d is the output's column descriptor: d.x = 0 / 1 for
// Re / Im of SVD coefficient d.w of mode d.z at detector d.y,
//   w = r Re(conj(A) b) / r (Ai br - Ar bi),  b = sum_p f^p B4[n0][d.w][p];
// d.x = 2 / 3 for Re / Im of the overlap of modes d.z, d.w,
//   w = -r^2 |A_a|^2 / 2 on the diagonal, else -r^2 Re(conj(A_a) A_b) /
//   r^2 Im(conj(A_a) A_b).
__device__ __forceinline__ double lnl_weight(const int4 d, const EpiSetup &o, int n_modes, int T, int q,
                                             const double2 *__restrict__ basis4) {
  const int k = d.y, a = d.z;
  const double rr = o.rr;
  const double ara = o.Ar[k][a], aia = o.Ai[k][a];
  if (d.x <= 1) {
    const double f = o.f[k];
    const double2 *v = basis4 + (((int64_t)(k * n_modes + a) * T + o.n0[k]) * q + d.w) * 4;
    const double2 v0 = v[0], v1 = v[1], v2 = v[2], v3 = v[3];
    const double br = fma(fma(fma(v3.x, f, v2.x), f, v1.x), f, v0.x);
    const double bi = fma(fma(fma(v3.y, f, v2.y), f, v1.y), f, v0.y);
    return d.x == 0 ? rr * (ara * br + aia * bi) : rr * (aia * br - ara * bi);
  }
  const double arb = o.Ar[k][d.w], aib = o.Ai[k][d.w];
  if (d.x == 2 && a == d.w) return -0.5 * rr * rr * (ara * ara + aia * aia);
  if (d.x == 2) return -rr * rr * (ara * arb + aia * aib);
  return rr * rr * (ara * aib - aia * arb);
}

// The setups of `cnt` (at most 64) proposals g0 .. g0 + cnt - 1 by one
// workgroup of four waves, the same arithmetic as epi_setup item by item:
// wave 0 the domain checks (a lane per proposal), wave 1 the detector
// responses and stencils (a lane per proposal and detector), waves 2 and 3
// the harmonics (a lane per proposal, mode and sign), then every thread the
// amplitudes.  A lane of epi_setup walks about 25 sines, cosines and powers in
// a row; split this way the longest chain is one item of each kind, which is
// what a small batch waits for.  consts(j): the constants of the j-th
// proposal's event; ylm(j, i): its harmonic terms, i < n_modes of -m, then of
// +m; nd, nm: bounds of its detector and mode counts.  epi_setup_parts and
// epi_setup_join are the two halves for threads t = 0 .. 255, a block barrier
// apart; epi_setup_block is both, and ends with a block barrier.
struct EpiTmp {
  double fp[RBFL_MAX_DET], fc[RBFL_MAX_DET];
  double yr[2 * RBFL_MAX_MODES], yi[2 * RBFL_MAX_MODES];
  int pre, out[RBFL_MAX_DET];
};

template <class ConstsOf, class YlmOf>
__device__ __forceinline__ void epi_setup_parts(int t, ConstsOf consts, YlmOf ylm, int nd, int nm,
                                                const double *__restrict__ params, int64_t ld, int64_t g0, int cnt,
                                                EpiSetup *su, EpiTmp *tmp) {
  const int wave = t >> 6, lane = t & 63;
  if (wave == 0) {
    if (lane < cnt) {
      const EvalConsts &c = consts(lane);
      double p[11];
      tmp[lane].pre = epi_prelude(c, params, ld, g0 + lane, p);
      su[lane].rr = c.d_ref / p[10];
    }
  } else if (wave == 1) {
    for (int e = lane; e < cnt * nd; e += 64) {
      const int j = e / nd, k = e - j * nd;
      const EvalConsts &c = consts(j);
      if (k >= c.n_det) continue;
      const int64_t g = g0 + j;
      double fp, fc, dt;
      detector_response(c.D[k], c.r[k], params[4 * ld + g], params[5 * ld + g], params[6 * ld + g], &fp, &fc, &dt);
      const double s = (params[9 * ld + g] + dt - c.t_trig) * c.fs + (double)c.half_w;
      const double fl = floor(s);
      const bool in = fl >= 4.0 && fl <= (double)(c.T - 6);
      su[j].n0[k] = in ? (int)fl : 4;
      su[j].f[k] = s - fl;
      tmp[j].fp[k] = fp;
      tmp[j].fc[k] = fc;
      tmp[j].out[k] = in ? 0 : 1;
    }
  } else {
    for (int e = (wave - 2) * 64 + lane; e < cnt * 2 * nm; e += 128) {
      const int j = e / (2 * nm), i = e - j * 2 * nm;
      if (i >= 2 * consts(j).n_modes) continue;
      const int64_t g = g0 + j;
      double ch, sh;
      sincos(0.5 * params[7 * ld + g], &sh, &ch);
      eval_ylm(ylm(j, i), ch, sh, params[8 * ld + g], &tmp[j].yr[i], &tmp[j].yi[i]);
    }
  }
}

template <class ConstsOf>
__device__ __forceinline__ void epi_setup_join(int t, ConstsOf consts, int nd, int nm, int cnt, EpiSetup *su,
                                               const EpiTmp *tmp) {
  for (int e = t; e < cnt * nd * nm; e += 256) {
    const int j = e / (nd * nm), r = e - j * nd * nm, k = r / nm, a = r - k * nm;
    const EvalConsts &c = consts(j);
    const int n = c.n_modes;
    if (k >= c.n_det || a >= n) continue;
    const double fp = tmp[j].fp[k], fc = tmp[j].fc[k];
    const double ynr = tmp[j].yr[a], yni = tmp[j].yi[a], ypr = tmp[j].yr[n + a], ypi = tmp[j].yi[n + a];
    const double sg = (c.mode_l[a] & 1) ? -1.0 : 1.0;
    su[j].Ar[k][a] = 0.5 * ((fp * ynr - fc * yni) + sg * (fp * ypr - fc * ypi));
    su[j].Ai[k][a] = 0.5 * ((fp * yni + fc * ynr) + sg * (-fp * ypi - fc * ypr));
  }
  if (t < cnt) {
    const int j = t;
    int bad = tmp[j].pre;
    if (bad == 0)
      for (int k = 0; k < consts(j).n_det; ++k) bad |= tmp[j].out[k];
    su[j].status = bad;
  }
}

template <class ConstsOf, class YlmOf>
__device__ __forceinline__ void epi_setup_block(ConstsOf consts, YlmOf ylm, int nd, int nm,
                                                const double *__restrict__ params, int64_t ld, int64_t g0, int cnt,
                                                EpiSetup *su, EpiTmp *tmp) {
  epi_setup_parts(threadIdx.x, consts, ylm, nd, nm, params, ld, g0, cnt, su, tmp);
  __syncthreads();
  epi_setup_join(threadIdx.x, consts, nd, nm, cnt, su, tmp);
  __syncthreads();
}

// ln L of one proposal from its setup o and interpolated row y; one whole
// wave per call, result in lane 0.  The loads of each stage
// are issued together before their values are used (kEpiUnroll coefficients
// per lane at a time, the detector's overlap reals one per lane), so a
// proposal waits for a few memory round trips instead of one per coefficient.
constexpr int kEpiUnroll = 2;

__device__ __forceinline__ double2 load_pair(const double *__restrict__ y, int i) {
  return *reinterpret_cast<const double2 *>(y + i);
}

// coef_off / sig_off: the output offsets of the consts (an LDS copy where the
// block has one).
template <int U = kEpiUnroll, class Row = const double *__restrict__>
__device__ __forceinline__ double epi_reduce(const EvalConsts &c, const EpiSetup &o, Row y,
                                             const double2 *__restrict__ basis4,
                                             const int (*coef_off)[RBFL_MAX_MODES], const int *sig_off) {
  const int lane = threadIdx.x & 63;
  if (o.status != 0) return o.status == 2 ? __builtin_nan("") : -__builtin_huge_val();
  const int n_modes = c.n_modes, q = c.q, T = c.T;
  const int P = c.n_det * n_modes;
  const int G = 64 / P;
  const int pair = lane / G;
  const int gl = lane - pair * G;
  const bool active = pair < P;
  const int k = active ? pair / n_modes : 0;
  const int a = active ? pair - k * n_modes : 0;
  const double f = o.f[k];
  const int n0 = o.n0[k];
  const double ar = o.Ar[k][a], ai = o.Ai[k][a];
  const int det_lead = k * n_modes * G;
  // detector k's overlap reals: lane det_lead + t holds term t (t < n_modes:
  // sigma_tt; then (Re, Im) sigma_ab for a < b in lexicographic order).  A
  // detector owns n_modes * G >= n_modes (n_modes + 1) / 2 lanes for up to 4
  // detectors and 5 modes.
  const int n_terms = n_modes * (n_modes + 1) / 2;
  const int t_own = lane - det_lead;
  double sg_a = 0.0, sg_b = 0.0;
  if (active && t_own < n_terms) {
    const int so = sig_off[k];
    if (t_own < n_modes) {
      sg_a = y[so + t_own];
    } else {
      const int pidx = so + n_modes + 2 * (t_own - n_modes);
      sg_a = y[pidx];
      sg_b = y[pidx + 1];
    }
  }
  // a5: partial reconstruction of z_{k,a} over this lane's coefficients; the
  // spline-folded basis gives the interpolated basis value as a cubic in f
  double zr = 0.0, zi = 0.0;
  if (active) {
    const int off = coef_off[k][a];
    const double2 *base = basis4 + ((int64_t)(k * n_modes + a) * T + n0) * q * 4;
    for (int i0 = gl; i0 < q; i0 += U * G) {
      double2 cc[U], v[U][4];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        // past the end: a valid entry is loaded and its coefficient zeroed,
        // so that every load is issued before the first use
        const bool ok = i0 + u * G < q;
        const int i = ok ? i0 + u * G : i0;
        const double2 cv = load_pair(y, off + 2 * i);
        cc[u].x = ok ? cv.x : 0.0;
        cc[u].y = ok ? cv.y : 0.0;
#pragma unroll
        for (int j = 0; j < 4; ++j) v[u][j] = base[4 * i + j];
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const double br = fma(fma(fma(v[u][3].x, f, v[u][2].x), f, v[u][1].x), f, v[u][0].x);
        const double bi = fma(fma(fma(v[u][3].y, f, v[u][2].y), f, v[u][1].y), f, v[u][0].y);
        zr += cc[u].x * br - cc[u].y * bi;
        zi += cc[u].x * bi + cc[u].y * br;
      }
    }
  }
  // combine the G partials of each pair in its first lane (a fixed tree: after
  // the step of distance o, lane g of a pair holds the sum over lanes
  // g .. g + 2 o - 1 of it)
  double tr = zr, ti = zi;
  for (int o = 1; o < G; o <<= 1) {
    const double vr = __shfl(tr, lane + o, 64), vi = __shfl(ti, lane + o, 64);
    if (gl + o < G) {
      tr += vr;
      ti += vi;
    }
  }
  const double zterm = ar * tr + ai * ti;   // Re(conj(A) z), valid in pair leaders
  // overlap term of detector k: every A_{k,b} is in the setup
  double st_s = 0.0, st_c = 0.0, zt_s = 0.0, zt_c = 0.0;
  {
    auto add = [](double &sum, double &comp, double v) {
      const double t = sum + v;
      comp += fabs(sum) >= fabs(v) ? (sum - t) + v : (v - t) + sum;
      sum = t;
    };
    for (int m = 0; m < n_modes; ++m) {
      add(zt_s, zt_c, __shfl(zterm, det_lead + m * G, 64));
      add(st_s, st_c, (o.Ar[k][m] * o.Ar[k][m] + o.Ai[k][m] * o.Ai[k][m]) * __shfl(sg_a, det_lead + m, 64));
    }
    int t = n_modes;
    for (int m = 0; m < n_modes; ++m)
      for (int mm = m + 1; mm < n_modes; ++mm) {
        const double sr = __shfl(sg_a, det_lead + t, 64), si = __shfl(sg_b, det_lead + t, 64);
        ++t;
        const double pr = o.Ar[k][m] * o.Ar[k][mm] + o.Ai[k][m] * o.Ai[k][mm];
        const double pi = o.Ar[k][m] * o.Ai[k][mm] - o.Ai[k][m] * o.Ar[k][mm];
        add(st_s, st_c, 2.0 * (pr * sr - pi * si));
      }
  }
  const double rr = o.rr;
  const double term = rr * (zt_s + zt_c) - 0.5 * rr * rr * (st_s + st_c);   // valid in detector leaders
  double tot = 0.0, comp = 0.0;
  for (int kk = 0; kk < c.n_det; ++kk) {
    const double v = __shfl(term, kk * n_modes * G, 64);
    const double t = tot + v;
    comp += fabs(tot) >= fabs(v) ? (tot - t) + v : (v - t) + tot;
    tot = t;
  }
  return tot + comp;
}

// The harmonics' terms of c, n_modes of -m, then n_modes of +m, into LDS by
// threads t = 0 .. 255, word by word.
__device__ __forceinline__ void epi_copy_ylm(int t, const EvalConsts &c, YlmTerms *ylm) {
  constexpr int kWords = sizeof(YlmTerms) / 4;
  static_assert(sizeof(YlmTerms) % 4 == 0, "copied by words");
  const int words = c.n_modes * kWords;
  for (int e = t; e < 2 * words; e += 256)
    reinterpret_cast<int *>(ylm)[e] =
        e < words ? reinterpret_cast<const int *>(c.ylm_neg)[e] : reinterpret_cast<const int *>(c.ylm_pos)[e - words];
}

// Setups first .. first + cnt - 1 of a batch (cnt <= kSetupGroup) to memory, by a
// workgroup of 256 threads of the launch that forms the basis rows.
constexpr int kSetupGroup = 8;
__device__ __forceinline__ void epi_setups_out(const EvalConsts &c, const double *__restrict__ params, int64_t ld,
                                               int64_t b0, int first, int cnt, EpiSetup *__restrict__ setups) {
  __shared__ EpiSetup su[kSetupGroup];
  __shared__ EpiTmp tmp[kSetupGroup];
  __shared__ YlmTerms ylm[2 * RBFL_MAX_MODES];
  epi_copy_ylm(threadIdx.x, c, ylm);
  __syncthreads();
  epi_setup_block([&](int) -> const EvalConsts & { return c; }, [&](int, int i) -> const YlmTerms & { return ylm[i]; },
                  c.n_det, c.n_modes, params, ld, b0 + first, cnt, su, tmp);
  for (int e = threadIdx.x; e < cnt * (int)(sizeof(EpiSetup) / 8); e += 256)
    reinterpret_cast<double *>(setups + first)[e] = reinterpret_cast<const double *>(su)[e];
}

// c's output offsets likewise.
__device__ __forceinline__ void epi_copy_offsets(int t, const EvalConsts &c, int (*coef_off)[RBFL_MAX_MODES],
                                                 int *sig_off) {
  if (t >= RBFL_MAX_DET * RBFL_MAX_MODES) return;
  coef_off[t / RBFL_MAX_MODES][t % RBFL_MAX_MODES] = c.coef_off[t / RBFL_MAX_MODES][t % RBFL_MAX_MODES];
  if (t < RBFL_MAX_DET) sig_off[t] = c.sig_off[t];
}

}  // namespace rbfl
