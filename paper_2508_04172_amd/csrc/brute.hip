// Exact ln L at each proposal without the interpolant (the reference the
// meshfree method approximates): the templates of every mode are formed on the
// frequency grid at the proposal's own intrinsic parameters, and
//   z_ka(tau_k) = 4 df sum_f conj(h_a) d_k e^{+2 pi i f tau_k} / S_k,
//   sigma_k,ab  = 4 df sum_f conj(h_a) h_b / S_k
// are direct sums over the band, combined as in Eq. logl_complete (corrected
// reading; equal to Eq. logl_basic for the projected signal of
// Eq. projected_h_fd).  tau_k = t_c + dt_k is absolute time in the segment;
// the phase f tau is split into a whole number of samples, reduced exactly in
// integers, plus a remainder, so long segments keep full precision.
//
// One workgroup per proposal; the threads stride over the bins, fixed-order
// reductions.  With A_ka the amplitudes, z and sigma enter only as
//   Re sum_a conj(A_ka) z_ka = <h_k|d_k>, sum_ab conj(A_ka) A_kb sigma_k,ab =
//   <h_k|h_k>,  h_k = sum_a A_ka h_a,
// so h_k is formed per bin and the two products are summed directly: one pass
// over the bins, the templates formed once for every detector.
// With the Earth's rotation switched on the antenna factors and delays vary
// along the band (each mode's frequency at its own stationary-phase time).
#include "rbfl_internal.h"

namespace rbfl {

namespace {

constexpr int kBruteThreads = 256;

// Sums v over the workgroup of BT threads (fixed order); result valid in every
// thread.
template <int BT>
__device__ __forceinline__ double block_sum(double v, double *red) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  __syncthreads();
  if (lane == 0) red[wave] = v;
  __syncthreads();
  double t = 0.0;
  for (int w = 0; w < BT / 64; ++w) t += red[w];
  return t;
}

// Frozen antenna patterns, ND detectors.  Bound by FP64 VALU work, so what the
// modes share is computed once per bin: with v = (pi M f)^(1/3), mode (l, m)
// has (pi M 2f/m)^(1/3) = (2/m)^(1/3) v, its logarithm ln v + ln(2/m)/3 and the
// amplitude f^(-7/6) = (pi M)^(7/6) v^(-7/2): one cube root, logarithm,
// reciprocal and square root per bin instead of one of each per mode and
// detector.  Phases are formed in half turns, so their reduction is exact and
// cheap, and the whole-sample shift j n mod n_s steps by a constant per
// iteration instead of two 64-bit divisions per bin.  What multiplies a phase of
// thousands of radians (v^-5 and its factor) is carried in two parts (4% of the
// time): rounded once each it left ln L of 300 proposals 5.0e-14 of its norm
// from a plain 64-bit evaluation, as the sums per detector and mode were; now
// 4.2e-14.  301 proposals of 32,448
// bins, 5 modes, 3 detectors: 0.18-0.21 ms by the card's clock, 1.04-1.20 ms with
// the templates formed per detector and 20 complex sums per thread.
template <int ND, int BT>
__global__ void __launch_bounds__(BT, 4) k_brute(const EvalConsts *__restrict__ cp, const double *__restrict__ params,
                                              int64_t ld, const double2 *__restrict__ Dd,
                                              const double *__restrict__ wk, int64_t j_lo, int64_t J, int64_t n_s,
                                              double df, double inv_dref_s, double *__restrict__ lnl) {
  __shared__ double red[BT / 64];
  __shared__ Binary bin;
  __shared__ int status;                            // 0 evaluate, 1 unphysical, 2 NaN input
  __shared__ double fpc[ND][2], rem_s[ND];
  __shared__ int64_t nmod_s[ND];
  __shared__ double yr[2 * RBFL_MAX_MODES], yi[2 * RBFL_MAX_MODES];
  struct ModeConsts {
    double cv, lcv, cph, cph_lo, k0, fr, amp;
    int64_t jend;
    double2 A[ND];
  };
  __shared__ ModeConsts mc[RBFL_MAX_MODES];
  const EvalConsts &c = *cp;
  const int64_t g = blockIdx.x;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int nm = c.n_modes;
  const double fs = (double)n_s * df;
  if (wave == 0) {
    double p[11];
    bool any_nan = false;
#pragma unroll
    for (int i = 0; i < 11; ++i) {
      p[i] = params[i * ld + g];
      any_nan |= isnan(p[i]);
    }
    double th[4], phys[4];
    for (int i = 0; i < 4; ++i) {
      double t = c.theta_c[i];
      for (int j = 0; j < 4; ++j) t += c.V[4 * i + j] * p[j];
      th[i] = t;
    }
    const bool ok = !any_nan && theta_to_phys(th, c.f0, c.chi_max, phys);
    if (lane == 0) {
      status = any_nan ? 2 : ok ? 0 : 1;
      if (ok) bin = make_binary(phys[0], phys[1], phys[2], phys[3], c.f_ref);
    }
  } else if (wave == 1) {
    if (lane < ND) {
      double dt;
      detector_response(c.D[lane], c.r[lane], params[4 * ld + g], params[5 * ld + g], params[6 * ld + g],
                        &fpc[lane][0], &fpc[lane][1], &dt);
      const double tau = params[9 * ld + g] + dt;
      const int64_t nsh = (int64_t)llrint(tau * fs);
      rem_s[lane] = tau - (double)nsh / fs;
      nmod_s[lane] = ((nsh % n_s) + n_s) % n_s;
    }
  } else if (wave == 2 && lane < 2 * nm) {
    double ch, sh;
    sincos(0.5 * params[7 * ld + g], &sh, &ch);
    eval_ylm(lane < nm ? c.ylm_neg[lane] : c.ylm_pos[lane - nm], ch, sh, params[8 * ld + g], &yr[lane], &yi[lane]);
  }
  __syncthreads();
  if (status != 0) {
    if (tid == 0) lnl[g] = status == 2 ? __builtin_nan("") : -__builtin_huge_val();
    return;
  }
  if (tid < nm) {
    const int l = c.mode_l[tid], m = c.mode_m[tid];
    const double hm = 0.5 * (double)m;
    ModeConsts &o = mc[tid];
    o.cv = cbrt(1.0 / hm);
    o.lcv = -log(hm) / 3.0;
    // hm pre hm^(5/3) / pi in two parts: its relative error is one of the whole
    // phase, the same in every bin, so it does not average out
    const double cb = cbrt(hm), cb_lo = fma(-cb * cb, cb, hm) / (3.0 * cb * cb);
    const double sq = cb * cb, sq_lo = fma(cb, cb, -sq) + 2.0 * cb * cb_lo;
    const double h2 = hm * hm, x = h2 * bin.pre, x_lo = fma(h2, bin.pre, -x);   // h2 = m^2 / 4 is exact
    const double y = x * sq, y_lo = fma(x, sq, -y) + x * sq_lo + x_lo * sq;
    o.cph = y / kPi;
    o.cph_lo = (fma(-o.cph, kPi, y) + y_lo - o.cph * 1.2246467991473532e-16) / kPi;   // pi past its double
    o.k0 = hm * (0.25 * kPi + bin.psi_ref) / kPi;
    o.fr = hm * bin.f_ref;
    o.amp = mode_amp(l, m, bin.eta, bin.delta) * bin.amp * inv_dref_s * pow(kPi * bin.m_s, 7.0 / 6.0);
    o.jend = std::min<int64_t>(j_lo + J, (int64_t)ceil((double)m * bin.f_isco / df));
  }
  if (tid >= 64 && tid < 64 + ND * nm) {
    const int k = (tid - 64) / nm, a = (tid - 64) - k * nm;
    const double sg = (c.mode_l[a] & 1) ? -1.0 : 1.0;
    const double fp = fpc[k][0], fc = fpc[k][1];
    mc[a].A[k].x = 0.5 * ((fp * yr[a] - fc * yi[a]) + sg * (fp * yr[nm + a] - fc * yi[nm + a]));
    mc[a].A[k].y = 0.5 * ((fp * yi[a] + fc * yr[a]) + sg * (-fp * yi[nm + a] - fc * yr[nm + a]));
  }
  __syncthreads();
  int64_t jmax = j_lo;
  for (int a = 0; a < nm; ++a) jmax = std::max(jmax, mc[a].jend);
  const double inv_ns = 1.0 / (double)n_s, um = kPi * bin.m_s, um_lo = fma(kPi, bin.m_s, -um) + 1.2246467991473532e-16 * bin.m_s,
               c1 = bin.dpsi_ref / kPi;
  const double p2 = bin.p2, p3 = bin.p3, p4 = bin.p4, p5 = bin.p5, p6 = bin.p6 + 1.3862943611198906 * bin.p6l,
               p6l = bin.p6l, p7 = bin.p7;
  int64_t ph[ND], dph[ND];
  double zt[ND] = {}, st[ND] = {};
#pragma unroll
  for (int k = 0; k < ND; ++k) {
    ph[k] = ((j_lo + tid) % n_s * nmod_s[k]) % n_s;     // products below n_s^2 / 2: fit in 64 bits
    dph[k] = (BT % n_s * nmod_s[k]) % n_s;
  }
  for (int64_t j = j_lo + tid; j < jmax; j += BT) {
    const double f = (double)j * df;
    const double t = um * f, t_lo = fma(um, f, -t) + um_lo * f;
    const double v = cbrt(t), lv = log(v), w = 1.0 / v;
    // w^5 in two parts, with w's own error from t w^3 = 1: five times it would
    // be the largest error of a phase of thousands of radians
    const double w2 = w * w, w2l = fma(w, w, -w2), w3 = w2 * w, w3l = fma(w2, w, -w3) + w2l * w;
    const double one = t * w3, off = (1.0 - one) - (fma(t, w3, -one) + t * w3l + t_lo * w3);
    const double w5 = w2 * w3, w5l = fma(w2, w3, -w5) + (w2 * w3l + w2l * w3) + w5 * (5.0 / 3.0) * off;
    const double af = w3 * sqrt(w);
    double Hr[ND] = {}, Hi[ND] = {};                    // h_k = sum_a A_ka h_a
    // one mode at a time, its constants from LDS: unrolled, the constants and
    // the sines' temporaries of five modes take more than 128 registers
#pragma unroll 1
    for (int a = 0; a < nm; ++a) {
      const ModeConsts &o = mc[a];
      const double va = v * o.cv, la = lv + o.lcv, va2 = va * va;
      double s = p7;
      s = s * va + (p6 + p6l * la);
      s = s * va + p5 * (1.0 + 3.0 * la);
      s = s * va + p4;
      s = s * va + p3;
      s = s * va + p2;
      s = s * va2 + 1.0;
      const double ws = w5 * s, wsl = fma(w5, s, -ws) + w5l * s;
      const double turns = (fma(o.cph, ws, fma(o.cph, wsl, o.cph_lo * ws)) - o.k0) - c1 * (f - o.fr);   // phase / pi
      double sn, cs;
      sincospi(turns, &sn, &cs);
      const double am = j < o.jend ? o.amp * af : 0.0;
      const double hr = am * cs, hi = am * sn;          // conj(h_a) = am e^{+i phase}, zero beyond the mode's band
#pragma unroll
      for (int k = 0; k < ND; ++k) {
        const double2 A = o.A[k];
        Hr[k] += A.x * hr + A.y * hi;
        Hi[k] += A.y * hr - A.x * hi;
      }
    }
#pragma unroll
    for (int k = 0; k < ND; ++k) {
      // e^{+2 pi i f tau} with the whole samples reduced exactly
      double se, ce;
      sincospi(2.0 * ((double)ph[k] * inv_ns + f * rem_s[k]), &se, &ce);
      const double2 d = Dd[(int64_t)k * J + j - j_lo];
      zt[k] += Hr[k] * (d.x * ce - d.y * se) + Hi[k] * (d.x * se + d.y * ce);
      st[k] += (Hr[k] * Hr[k] + Hi[k] * Hi[k]) * wk[(int64_t)k * J + j - j_lo];
      ph[k] += dph[k];
      ph[k] -= ph[k] >= n_s ? n_s : 0;
    }
  }
  const double rr = c.d_ref / params[10 * ld + g];
  double total = 0.0, comp = 0.0;
#pragma unroll
  for (int k = 0; k < ND; ++k) {
    const double t1 = rr * block_sum<BT>(zt[k], red) - 0.5 * rr * rr * block_sum<BT>(st[k], red);
    const double t = total + t1;
    comp += fabs(total) >= fabs(t1) ? (total - t) + t1 : (t1 - t) + total;
    total = t;
  }
  if (tid == 0) lnl[g] = total + comp;
}

__global__ void __launch_bounds__(kBruteThreads) k_brute_rotating(const EvalConsts *__restrict__ cp,
                                                         const double *__restrict__ params, int64_t ld,
                                                         const double2 *__restrict__ Dd,
                                                         const double *__restrict__ wk, int64_t j_lo, int64_t J,
                                                         int64_t n_s, double df, double inv_dref_s,
                                                         double *__restrict__ lnl) {
  __shared__ double red[kBruteThreads / 64];
  const EvalConsts &c = *cp;
  const int64_t g = blockIdx.x;
  double p[11];
  bool any_nan = false;
#pragma unroll
  for (int i = 0; i < 11; ++i) {
    p[i] = params[i * ld + g];
    any_nan |= isnan(p[i]);
  }
  if (any_nan) {
    if (threadIdx.x == 0) lnl[g] = __builtin_nan("");
    return;
  }
  double th[4], phys[4];
  for (int i = 0; i < 4; ++i) {
    double t = c.theta_c[i];
    for (int j = 0; j < 4; ++j) t += c.V[4 * i + j] * p[j];
    th[i] = t;
  }
  if (!theta_to_phys(th, c.f0, c.chi_max, phys)) {
    if (threadIdx.x == 0) lnl[g] = -__builtin_huge_val();
    return;
  }
  const Binary b = make_binary(phys[0], phys[1], phys[2], phys[3], c.f_ref);
  const double alpha = p[4], dec = p[5], psi = p[6], iota = p[7], phi = p[8], tc = p[9], dl = p[10];
  const double rr = c.d_ref / dl;
  const int n_modes = c.n_modes;
  // band end of each mode: f < m F_isco
  int64_t jend[RBFL_MAX_MODES];
  int64_t jmax = j_lo;
#pragma unroll
  for (int a = 0; a < RBFL_MAX_MODES; ++a) {
    if (a >= n_modes) break;
    jend[a] = std::min<int64_t>(j_lo + J, (int64_t)ceil((double)c.mode_m[a] * b.f_isco / df));
    jmax = std::max(jmax, jend[a]);
  }
  double ch, sh;
  sincos(0.5 * iota, &sh, &ch);
  const double fs = (double)n_s * df;
  double total = 0.0, comp = 0.0;
  // rotating Earth: A and the delay of every (bin, mode) at the mode's
  // stationary-phase time t_a = t_c + Psi'(2f/m) / (2 pi); <h_k|d_k> and
  // <h_k|h_k> summed directly over the band
  double ynr[RBFL_MAX_MODES], yni[RBFL_MAX_MODES], ypr[RBFL_MAX_MODES], ypi[RBFL_MAX_MODES];
  for (int a = 0; a < n_modes; ++a) {
    eval_ylm(c.ylm_neg[a], ch, sh, phi, &ynr[a], &yni[a]);
    eval_ylm(c.ylm_pos[a], ch, sh, phi, &ypr[a], &ypi[a]);
  }
  for (int k = 0; k < c.n_det; ++k) {
    const double2 *Dk = Dd + (int64_t)k * J;
    const double *wkk = wk + (int64_t)k * J;
    double zr = 0.0, sw = 0.0;
    for (int64_t j = j_lo + threadIdx.x; j < jmax; j += kBruteThreads) {
      const double f = (double)j * df;
      double hr = 0.0, hi = 0.0;
      for (int a = 0; a < n_modes; ++a) {
        if (!(j < jend[a])) continue;
        const int l = c.mode_l[a], m = c.mode_m[a];
        const double x = 2.0 * f / (double)m;
        const double ta = tc + (dphase22_pn(x, b) - b.dpsi_ref) / (2.0 * kPi);
        double fp, fc, dt;
        detector_response(c.D[k], c.r[k], alpha - c.earth_rate * (ta - c.t_trig), dec, psi, &fp, &fc, &dt);
        const double sg = (l & 1) ? -1.0 : 1.0;
        const double Ar = 0.5 * ((fp * ynr[a] - fc * yni[a]) + sg * (fp * ypr[a] - fc * ypi[a]));
        const double Ai = 0.5 * ((fp * yni[a] + fc * ynr[a]) + sg * (-fp * ypi[a] - fc * ypr[a]));
        const double ph = 0.5 * (double)m * phase22(x, b);
        const double amp = mode_amp(l, m, b.eta, b.delta) * b.amp * inv_dref_s * exp(-7.0 / 6.0 * log(f));
        double sn, cs;
        sincos(ph, &sn, &cs);
        const double xr = amp * cs, xi = -amp * sn;   // h_a = amp e^{-i ph}
        const double tau = tc + dt;
        const int64_t nsh = (int64_t)llrint(tau * fs);
        const double rem = tau - (double)nsh / fs;
        const int64_t nm_ = ((nsh % n_s) + n_s) % n_s;
        const int64_t ph_int = ((j % n_s) * nm_) % n_s;
        double se, ce;
        sincospi(-2.0 * ((double)ph_int / (double)n_s + f * rem), &se, &ce);
        const double vr = Ar * xr - Ai * xi, vi = Ar * xi + Ai * xr;
        hr += vr * ce - vi * se;
        hi += vr * se + vi * ce;
      }
      const double2 d = Dk[j - j_lo];
      zr += hr * d.x + hi * d.y;                       // Re(conj(h) d)
      sw += (hr * hr + hi * hi) * wkk[j - j_lo];
    }
    const double v = rr * block_sum<kBruteThreads>(zr, red) - 0.5 * rr * rr * block_sum<kBruteThreads>(sw, red);
    const double t = total + v;
    comp += fabs(total) >= fabs(v) ? (total - t) + v : (v - t) + total;
    total = t;
  }
  if (threadIdx.x == 0) lnl[g] = total + comp;
}

}  // namespace

template <int ND>
static void launch_brute_det(const EvalConsts *c, const double *params, int64_t ld, int64_t n, const double2 *Dd,
                               const double *wk, int64_t j_lo, int64_t J, int64_t n_s, double df, double inv_dref_s,
                               double *lnl, hipStream_t s) {
  // four waves per SIMD from one workgroup while there are at most two
  // workgroups per CU (301 proposals: 180 us against 266 us with workgroups of 4
  // waves, 1 proposal: 127 against 185 us), else workgroups of 4 waves, which
  // leave no CU waiting for the rest of a large one
  if (n <= 512)
    hipLaunchKernelGGL((k_brute<ND, 1024>), dim3((unsigned)n), dim3(1024), 0, s, c, params, ld, Dd, wk, j_lo, J, n_s, df,
                       inv_dref_s, lnl);
  else
    hipLaunchKernelGGL((k_brute<ND, 256>), dim3((unsigned)n), dim3(256), 0, s, c, params, ld, Dd, wk, j_lo, J, n_s, df,
                       inv_dref_s, lnl);
  RBFL_HIP(hipGetLastError());
}

void launch_brute(const EvalConsts *c, const EvalConsts &hc, const double *params, int64_t ld, int64_t n,
                  const double2 *Dd, const double *wk, int64_t j_lo, int64_t J, int64_t n_s, double df,
                  double inv_dref_s, double *lnl, hipStream_t s) {
  if (n <= 0) return;
  if (hc.earth_rate != 0.0) {
    hipLaunchKernelGGL(k_brute_rotating, dim3((unsigned)n), dim3(kBruteThreads), 0, s, c, params, ld, Dd, wk, j_lo, J,
                       n_s, df, inv_dref_s, lnl);
    RBFL_HIP(hipGetLastError());
    return;
  }
  static_assert(RBFL_MAX_DET == 4, "one kernel per detector count");
  switch (hc.n_det) {
    case 1: launch_brute_det<1>(c, params, ld, n, Dd, wk, j_lo, J, n_s, df, inv_dref_s, lnl, s); break;
    case 2: launch_brute_det<2>(c, params, ld, n, Dd, wk, j_lo, J, n_s, df, inv_dref_s, lnl, s); break;
    case 3: launch_brute_det<3>(c, params, ld, n, Dd, wk, j_lo, J, n_s, df, inv_dref_s, lnl, s); break;
    default: launch_brute_det<4>(c, params, ld, n, Dd, wk, j_lo, J, n_s, df, inv_dref_s, lnl, s);
  }
}

}  // namespace rbfl
