// Reverse-mode derivative of the log-likelihood recursion with respect to
// theta, and of the log prior.
//
// The forward sweep stores the exponents w_k of the observation that opens
// every segment of SEG observations (a checkpoint) in the workspace.  The
// reverse sweep visits the segments last to first: it recomputes the
// segment forward from its checkpoint, keeping each observation's exponents
// in a per-lane LDS buffer, then propagates the adjoints back through the
// segment.  Parameter adjoints are summed per segment in the recursion's
// precision and added to FP64 totals.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "model.h"

namespace smc {

// psi(x) by upward recurrence to x >= 8 and the asymptotic series in 1/x^2.
__device__ inline double digamma_dev(double x) {
  double acc = 0.0;
  while (x < 8.0) {
    acc -= 1.0 / x;
    x += 1.0;
  }
  const double r = 1.0 / x, r2 = r * r;
  const double series =
      r2 * (1.0 / 12 - r2 * (1.0 / 120 - r2 * (1.0 / 252 - r2 * (1.0 / 240 - r2 * (1.0 / 132)))));
  return acc + log(x) - 0.5 * r - series;
}

// d log p(theta) / d theta.
template <class M>
__device__ inline void logprior_grad(const double *th, double *g);

// (Within the support of the truncated theta_8i the truncation only adds a
// constant, so every term is Gaussian.)
template <int K, int SH, typename R, int I>
struct PriorGrad {
  __device__ static void run(const double *th, double *g) {
    using E = Egarch<K, SH, R, I>;
#pragma unroll
    for (int i = 0; i < E::D; ++i) {
      double m, sd, lsd;
      E::prior_moments(i, m, sd, lsd);
      g[i] = -(th[i] - m) / (sd * sd);
    }
  }
};

// Segment lengths: checkpoints every 64 observations in FP32, every 32 in
// FP64 (the per-lane LDS buffer holds SEG x K values).
template <typename R>
struct SegLen {
  static constexpr int value = sizeof(R) == 4 ? 64 : 32;
};

template <class M>
struct Adjoint;

template <int K, int SH, typename R, int I>
struct Adjoint<Egarch<K, SH, R, I>> {
  using Md = Egarch<K, SH, R, I>;
  using Y = typename Md::Y;
  using Par = typename Md::Par;
  static constexpr int D = Md::D;
  static constexpr int SEG = SegLen<R>::value;
  static constexpr bool kT = Md::kT;
  static constexpr bool kMix = Md::kMix;
  static constexpr int kNM = Md::kNM;
  static constexpr int kLdsPerLane = SEG * K;  // values of type R

  __device__ static int64_t nseg(int64_t t) { return (t + SEG - 1) / SEG; }

  // Chain rule from the adjoints of the components' constants (lw_i =
  // log2(p_i / sigma_i), nb_i = -log2(e) / (2 sigma_i^2), mu_i) back through
  // eqs EGARCH_tran1/2 to theta_6i, theta_7i, theta_8i.
  __device__ static void mixture_chain(const double *th, const double *lwb, const double *nbb,
                                       const double *mub, double scale, double *g) {
#pragma clang fp contract(off)
    constexpr int b = 2 + 3 * K;
    double ps[kNM], pw[kNM], mss[kNM], ss[kNM], S = 0.0, mbar = 0.0, q = 0.0;
#pragma unroll
    for (int i = 0; i < I; ++i) {
      ps[i] = tanh(th[b + i]) + 1.0;
      S += ps[i];
    }
#pragma unroll
    for (int i = 0; i < I; ++i) {
      pw[i] = ps[i] / S;
      mbar += pw[i] * th[b + I + i];
    }
#pragma unroll
    for (int i = 0; i < I; ++i) {
      mss[i] = th[b + I + i] - mbar;  // mu**
      ss[i] = exp(th[b + 2 * I + i]);  // sigma*
      q += pw[i] * (mss[i] * mss[i] + ss[i] * ss[i]);
    }
    const double c = 1.0 / sqrt(q);
    // adjoints of the normalised p_i, mu_i, sigma_i
    double pb[kNM], mb[kNM], sb[kNM], cb = 0.0;
#pragma unroll
    for (int i = 0; i < I; ++i) {
      const double si = c * ss[i];
      pb[i] = lwb[i] / (pw[i] * kLn2);
      sb[i] = -lwb[i] / (si * kLn2) + nbb[i] * kLog2e / (si * si * si);
      mb[i] = mub[i];
      cb += mb[i] * mss[i] + sb[i] * ss[i];
    }
    const double qb = cb * (-0.5 * c * c * c);
    double mbarb = 0.0, pdot = 0.0;
    double mssb[kNM], pbt[kNM];
#pragma unroll
    for (int i = 0; i < I; ++i) {
      mssb[i] = c * mb[i] + qb * 2.0 * pw[i] * mss[i];
      mbarb -= mssb[i];
    }
#pragma unroll
    for (int i = 0; i < I; ++i) {
      pbt[i] = pb[i] + qb * (mss[i] * mss[i] + ss[i] * ss[i]) + mbarb * th[b + I + i];
      pdot += pbt[i] * pw[i];
    }
#pragma unroll
    for (int i = 0; i < I; ++i) {
      const double ssb = c * sb[i] + qb * 2.0 * pw[i] * ss[i];
      const double psb = (pbt[i] - pdot) / S;
      const double tn = tanh(th[b + i]);
      g[b + i] += scale * psb * (1.0 - tn * tn);
      g[b + I + i] += scale * (mssb[i] + mbarb * pw[i]);
      g[b + 2 * I + i] += scale * ssb * ss[i];
    }
  }

  // Values of one observation that its density's adjoint leaves behind, beside
  // E and the adjoint eb of the shock: FP32 Student-t e^2/q1 and log2 q1 with
  // q1 = 1 + e^2/(nu - 2); FP64 Student-t e^2/q1 (the logarithms' sum is the
  // forward sweep's); mixtures 2^(x_i - m) and ln2 / sum_j 2^(x_j - m), whose
  // products are ln2 pi_i.
  static constexpr int NX = kT ? (sizeof(R) == 4 ? 2 : 1) : (kMix ? kNM + 1 : 0);
  static constexpr int NXA = NX > 0 ? NX : 1;

  // The reverse step of an observation in parts, so that a block can give
  // them to different waves (GradBlock) and one wave can run them in turn
  // with the same operations.  Contractions are written out, so both forms
  // round alike.
  //
  // local: from the exponents w and y alone, z, E = 2^(sum w), the adjoint eb of
  // the shock e = z E in the observation's log density (ln2 sw - e^2/2, or
  // - hnu1 log(1 + e^2/(nu-2)), or the mixture's ln2 log2 sum_i 2^x_i, x_i =
  // lw_i + nb_i (e - mu_i)^2, whose d/dx_i is ln2 pi_i with pi_i = 2^(x_i - m) /
  // sum_j 2^(x_j - m)).
  __device__ __forceinline__ static void local(const Par &p, const R (&w)[K], R yv, R &z, R &E,
                                               R &eb, R (&x)[NXA]) {
#pragma clang fp contract(off)
    R sw = (R)0;
#pragma unroll
    for (int k = 0; k < K; ++k) sw += w[k];
    E = exp2_fast(sw);
    z = fma(yv, p.isig, -p.mus);
    if constexpr (kT) {
      const R e = z * E;
      const R q1 = fma(e * e, p.inu2, (R)1);
      eb = -(R)p.hnu1 * (R)2 * e * p.inu2 / q1;
      x[0] = e * e / q1;
      if constexpr (sizeof(R) == 4) x[1] = __builtin_amdgcn_logf(q1);
    } else if constexpr (kMix) {
      R dm[kNM], xi[kNM];
#pragma unroll
      for (int i = 0; i < kNM; ++i) {
        dm[i] = fma(z, E, -p.mu[i]);
        xi[i] = fma(p.nb[i] * dm[i], dm[i], p.lw[i]);
      }
      R mx = xi[0];
#pragma unroll
      for (int i = 1; i < kNM; ++i) mx = fmax(mx, xi[i]);
      R sm = (R)0;
#pragma unroll
      for (int i = 0; i < kNM; ++i) {
        x[i] = exp2_lean(xi[i] - mx);
        sm += x[i];
      }
      x[kNM] = (R)kLn2 / sm;
      eb = (R)0;
#pragma unroll
      for (int i = 0; i < kNM; ++i)
        eb = fma((R)2 * (x[i] * x[kNM]) * p.nb[i], dm[i], eb);
    } else {
      eb = -(z * E);
    }
  }

  // chain: the adjoints wb of the next observation's exponents become those of
  // this one's (w_k,s+1 = kz_k E + a_k w_k + c0_k).
  __device__ __forceinline__ static void chain(const Par &p, R z, R E, R eb, R (&wb)[K]) {
#pragma clang fp contract(off)
    R Eb = (R)0;
#pragma unroll
    for (int k = 0; k < K; ++k) Eb = fma(wb[k], fma(p.kb[k], fabs(z), p.kg[k] * z), Eb);
    Eb = fma(eb, z, Eb);
    const R swb = fma(Eb * E, (R)kLn2, (R)kLn2);
#pragma unroll
    for (int k = 0; k < K; ++k) wb[k] = fma(wb[k], p.a[k], swb);
  }

  // Parameter adjoints, summed over a segment in R (Sums), then in FP64.
  template <typename V>
  struct Sums {
    V a[K], c0[K], kb[K], kg[K];       // the factors' coefficients
    V isig, mus, inu2, hnu1;           // location, scale, degrees of freedom
    V lw[kNM], nb[kNM], mu[kNM];       // mixture components
  };
  template <typename V>
  __device__ __forceinline__ static void clear(Sums<V> &s) {
#pragma unroll
    for (int k = 0; k < K; ++k) s.a[k] = s.c0[k] = s.kb[k] = s.kg[k] = (V)0;
    s.isig = s.mus = s.inu2 = s.hnu1 = (V)0;
#pragma unroll
    for (int i = 0; i < kNM; ++i) s.lw[i] = s.nb[i] = s.mu[i] = (V)0;
  }
  // wb: the adjoints before chain() of the same observation
  __device__ __forceinline__ static void sum_exponents(const R (&w)[K], const R (&wb)[K],
                                                       Sums<R> &s) {
#pragma unroll
    for (int k = 0; k < K; ++k) s.a[k] = fma(wb[k], w[k], s.a[k]);
  }
  __device__ __forceinline__ static void sum_factors(R z, R E, const R (&wb)[K], Sums<R> &s) {
#pragma clang fp contract(off)
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const R kzb = wb[k] * E;
      s.kb[k] = fma(kzb, fabs(z), s.kb[k]);
      s.kg[k] = fma(kzb, z, s.kg[k]);
      s.c0[k] += wb[k];
    }
  }
  __device__ __forceinline__ static void sum_shock(const Par &p, R yv, R z, R E, R eb,
                                                   const R (&x)[NXA], const R (&wb)[K],
                                                   Sums<R> &s) {
#pragma clang fp contract(off)
    const R sgn = z > (R)0 ? (R)1 : (z < (R)0 ? (R)-1 : (R)0);
    R zb = (R)0;
#pragma unroll
    for (int k = 0; k < K; ++k) zb = fma(wb[k] * E, fma(p.kb[k], sgn, p.kg[k]), zb);
    zb = fma(eb, E, zb);
    s.isig = fma(zb, yv, s.isig);
    s.mus -= zb;
    if constexpr (kT) {
      s.inu2 = fma(-(R)p.hnu1, x[0], s.inu2);
      if constexpr (NX > 1) s.hnu1 -= x[1];
    }
  }
  __device__ __forceinline__ static void sum_mixture(const Par &p, R z, R E, const R (&x)[NXA],
                                                     Sums<R> &s) {
#pragma clang fp contract(off)
    if constexpr (kMix) {
#pragma unroll
      for (int i = 0; i < kNM; ++i) {
        const R dm = fma(z, E, -p.mu[i]), pi = x[i] * x[kNM];
        s.lw[i] = fma(x[i], x[kNM], s.lw[i]);
        s.nb[i] = fma(pi * dm, dm, s.nb[i]);
        s.mu[i] = fma(-((R)2 * pi * p.nb[i]), dm, s.mu[i]);
      }
    }
  }
  __device__ __forceinline__ static void flush_exponents(Sums<R> &s, Sums<double> &tot) {
#pragma unroll
    for (int k = 0; k < K; ++k) {
      tot.a[k] += (double)s.a[k];
      s.a[k] = (R)0;
    }
  }
  __device__ __forceinline__ static void flush_factors(Sums<R> &s, Sums<double> &tot) {
#pragma unroll
    for (int k = 0; k < K; ++k) {
      tot.c0[k] += (double)s.c0[k];
      tot.kb[k] += (double)s.kb[k];
      tot.kg[k] += (double)s.kg[k];
      s.c0[k] = s.kb[k] = s.kg[k] = (R)0;
    }
  }
  __device__ __forceinline__ static void flush_shock(Sums<R> &s, Sums<double> &tot) {
    tot.isig += (double)s.isig;
    tot.mus += (double)s.mus;
    tot.inu2 += (double)s.inu2;
    tot.hnu1 += (double)s.hnu1;
    s.isig = s.mus = s.inu2 = s.hnu1 = (R)0;
  }
  __device__ __forceinline__ static void flush_mixture(Sums<R> &s, Sums<double> &tot) {
#pragma unroll
    for (int i = 0; i < kNM; ++i) {
      tot.lw[i] += (double)s.lw[i];
      tot.nb[i] += (double)s.nb[i];
      tot.mu[i] += (double)s.mu[i];
      s.lw[i] = s.nb[i] = s.mu[i] = (R)0;
    }
  }

  // Forward sweep over 1..t: the log likelihood, the state at t and the
  // checkpoints ckpt[nseg][K][P] (not written by lanes that are not live).
  // hold, when given, receives the last segment's exponents ([SEG * K][64],
  // this lane's column).  Observations come eight at a time, the next eight's
  // loads issued before the current ones are used.
  static constexpr int kFwd = 8;
  __device__ static double forward(const Par &p, int64_t t, const Y *__restrict__ y, R *ckpt,
                                   int64_t P, int64_t pidx, bool live, R *hold, R (&st)[Md::S],
                                   double &se_out) {
#pragma clang fp contract(off)
    typename Md::Run r;
#pragma unroll
    for (int k = 0; k < K; ++k) r.w[k] = (R)0;
    r.sw = (R)0;
    double sv = 0.0, se = 0.0;
    const int64_t ns = nseg(t);
    R wl[K];
    R lastE = (R)1, lastz = (R)0;
    auto segment = [&](int64_t sg, auto keep) {
      if (live)
#pragma unroll
        for (int k = 0; k < K; ++k) ckpt[(sg * K + k) * P + pidx] = r.w[k];
      open_segment(r);  // as the replay will open it
      // 32-bit counters and a segment pointer keep the loop's bookkeeping
      // off the scalar unit
      const int64_t s0 = sg * SEG;
      const int len = (int)(min(t, s0 + SEG) - s0);
      const Y *__restrict__ ys = y + s0;
      R av = (R)0, ae = (R)0, pm = (R)1;
      R tx[kFwd];  // FP64 Student-t: x_i of a group (Egarch::kTLog)
      // observation j of the segment; at: its place among eight, known at
      // compile time in the unrolled loop
      auto one = [&](int j, int at, R yv) {
#pragma unroll
        for (int k = 0; k < K; ++k) {
          wl[k] = r.w[k];
          if constexpr (decltype(keep)::value) hold[(j * K + k) * 64] = r.w[k];
        }
        av += Md::step(p, yv, r, ae, pm, lastE, lastz);
        if constexpr (kMix) {
          // the mixture sums' product, folded into log2 every 8 observations
          if (at == 7) {
            se += (double)log2_fast(pm);
            pm = (R)1;
          }
        } else if constexpr (Md::kTProd) {
          // FP32 Student-t factors, multiplied in groups (Egarch::kTProd)
          if (at % Md::kTGroup == Md::kTGroup - 1) {
            ae += log2_fast(pm);
            pm = (R)1;
          }
        }
      };
      int j = 0;
      if (len >= kFwd) {
        Y yn[kFwd];
#pragma unroll
        for (int u = 0; u < kFwd; ++u) yn[u] = ys[u];
        for (; j + kFwd <= len; j += kFwd) {
          Y yb[kFwd];
#pragma unroll
          for (int u = 0; u < kFwd; ++u) yb[u] = yn[u];
          const Y *__restrict__ pn = ys + (j + 2 * kFwd <= len ? j + kFwd : j);
#pragma unroll
          for (int u = 0; u < kFwd; ++u) yn[u] = pn[u];
#pragma unroll
          for (int u = 0; u < kFwd; ++u) {
            one(j + u, u, yb[u]);
            if constexpr (Md::kTLog) {
              tx[u] = Md::t_x(p, lastz, lastE);
              if (u == kFwd - 1) ae += Md::t_group_log(tx);
            }
          }
        }
      }
      for (; j < len; ++j) {
        one(j, j % kFwd, ys[j]);
        if constexpr (Md::kTLog) ae += log1p_pos<true>(Md::t_x(p, lastz, lastE));
      }
      if constexpr (Md::kTProd) ae += log2_fast(pm);
      sv += (double)av;
      se += (double)ae;
      if constexpr (kMix) se += (double)log2_fast(pm);
    };
    for (int64_t sg = 0; sg < ns - 1; ++sg) segment(sg, std::false_type());
    if (hold) segment(ns - 1, std::true_type());
    else segment(ns - 1, std::false_type());
    const R kap = (R)Md::kKappa;
#pragma unroll
    for (int k = 0; k < K; ++k) st[k] = wl[k] / kap;
    st[K] = Md::shock(p, lastz, lastE);
    se_out = se;
    const double n = (double)t;
    if constexpr (kT) return n * (p.cst - p.lsig) + kLn2 * sv - p.hnu1 * t_scale<R>() * se;
    else if constexpr (kMix) return n * (p.cst - p.lsig) + kLn2 * (sv + se);
    else return n * (p.cst - p.lsig) + kLn2 * sv - 0.5 * se;
  }

  // The checkpoints through the likelihood's own forward recursion (advance(),
  // advance_split()), and the density terms' sum, which FP64 Student-t
  // gradients need (se).
  struct Mark {
    static constexpr bool on = true;
    R *ckpt;
    int64_t P, pidx;
    bool live;
    double se = 0.0;
    __device__ __forceinline__ void operator()(int i, const typename Md::Run &r) {
      if (i % SEG == 0 && live)
#pragma unroll
        for (int k = 0; k < K; ++k) ckpt[((int64_t)(i / SEG) * K + k) * P + pidx] = r.w[k];
    }
    __device__ __forceinline__ void done(double s) { se = s; }
  };
  static constexpr bool kNeedsSe = Md::kTLog;

  // Log-likelihood over 1..t from s0 and its gradient g[D] (accumulated into
  // g, times `scale`), one particle per lane.  ckpt: [nseg][K][P] of R; lds:
  // this lane's column base of a [SEG*K][64] buffer of R; st receives the
  // state at t.  kFwd = false: the checkpoints are there (Mark), with their se;
  // the gradient alone (0 is returned, st is not written).
  template <bool kFwd = true>
  __device__ static double value_and_grad(const Par &p, const double *th, int64_t t,
                                          const Y *__restrict__ y, R *ckpt, int64_t P, int64_t pidx,
                                          R *lds, double scale, double *g, R (&st)[Md::S],
                                          double se = 0.0) {
    if (t <= 0) {
#pragma unroll
      for (int k = 0; k < Md::S; ++k) st[k] = (R)0;
      return 0.0;
    }
    double ll = 0.0;
    if constexpr (kFwd) ll = forward(p, t, y, ckpt, P, pidx, true, nullptr, st, se);
    Sums<double> tot;
    Sums<R> sum;
    clear(tot);
    clear(sum);
    if constexpr (Md::kTLog) tot.hnu1 = -se;  // sum of -log(1 + e^2/(nu - 2))
    R wb[K];  // adjoint of the exponents of the observation after the current one
#pragma unroll
    for (int k = 0; k < K; ++k) wb[k] = (R)0;
    typename Md::Run r;
    for (int64_t sg = nseg(t) - 1; sg >= 0; --sg) {
      const int64_t s0 = sg * SEG;
      const int len = (int)(min(t, s0 + SEG) - s0);
      const Y *__restrict__ ys = y + s0;
      // recompute the segment, keeping each observation's exponents
      load_ckpt(ckpt, sg, P, pidx, r);
      for (int j = 0; j < len; ++j) {
#pragma unroll
        for (int k = 0; k < K; ++k) lds[(j * K + k) * 64] = r.w[k];
        R ae = (R)0, pm = (R)1, Ed, zd;
        (void)Md::step(p, ys[j], r, ae, pm, Ed, zd);
      }
      for (int j = len - 1; j >= 0; --j) {
        R w[K], z, E, eb, x[NXA];
#pragma unroll
        for (int k = 0; k < K; ++k) w[k] = lds[(j * K + k) * 64];
        local(p, w, ys[j], z, E, eb, x);
        sum_exponents(w, wb, sum);
        sum_factors(z, E, wb, sum);
        sum_shock(p, ys[j], z, E, eb, x, wb, sum);
        sum_mixture(p, z, E, x, sum);
        chain(p, z, E, eb, wb);
      }
      flush_exponents(sum, tot);
      flush_factors(sum, tot);
      flush_shock(sum, tot);
      flush_mixture(sum, tot);
    }
    to_theta(th, t, tot, scale, g);
    return ll;
  }

  // A segment starts from its exponents alone: their sum is formed anew (FP64
  // recursions otherwise carry it by an fma of its own), so that the forward
  // sweep and the replays give the same bits.
  __device__ __forceinline__ static void open_segment(typename Md::Run &r) {
    R sw0 = r.w[0];
#pragma unroll
    for (int k = 1; k < K; ++k) sw0 += r.w[k];
    r.sw = sw0;
  }
  __device__ __forceinline__ static void load_ckpt(const R *ckpt, int64_t sg, int64_t P,
                                                   int64_t pidx, typename Md::Run &r) {
#pragma unroll
    for (int k = 0; k < K; ++k) r.w[k] = ckpt[(sg * K + k) * P + pidx];
    open_segment(r);
  }

  // The same by a block of eight waves for one wave of particles, for
  // populations that leave compute units idle.  A wave issues one instruction
  // in four to five cycles however much of the chip is free, and the reverse
  // sweep's 85 to 150 instructions per observation hang on a chain of fewer
  // than ten (chain()).  So after the forward sweep (wave 0) the block runs the
  // sub-blocks of B observations, last to first, through a pipeline with one
  // barrier per stage, each wave at its own place:
  //   waves 4-7  local() of sub-block b, an observation each in turn (FP64:
  //              waves 5-7, as wave 0's replay needs all of its SIMD)
  //   wave 1     chain() of sub-block b + 1, and its product with the exponents
  //   waves 2, 3 the other parameter sums of sub-block b + 2
  //   wave 0     the replay of the segment before b's, spread over b's stages
  // handing over in LDS: the exponents of two segments (the last one's come
  // from the forward sweep), three sub-blocks of local()'s values and two of
  // chain()'s.  Every sum and recursion keeps its operations and order, so
  // the results are value_and_grad()'s to the bit.  A stage takes its busiest
  // wave's issue slots and the latency of its LDS reads (FP32: 170 cycles per
  // observation with B = 16; FP64: 165 for EGARCH(1) Gaussian).  Langevin step
  // of EGARCH(2)-t FP32, 16,384 particles at t = 2,500: 706 us by one wave per
  // 64 particles, 293 by blocks; gradient of EGARCH(1) Gaussian FP64, 4,096
  // vectors over 5,000 observations: 1,313 and 572.
  static constexpr int kBlkWaves = 8;
  // Values per observation from local(): z, E, eb, x, and in FP64 the exponents
  // too, so that the replay may overwrite theirs at once (in FP32, where LDS
  // holds longer sub-blocks instead, it starts a stage later).
  static constexpr bool kRingW = sizeof(R) == 8;
  static constexpr int kLocal = kRingW ? 3 : 4;  // waves of local()
  static constexpr int NF = 3 + NX + (kRingW ? K : 0);
  static constexpr size_t blk_lds(int b) {
    return (size_t)64 * sizeof(R) * (2 * SEG * K + 3 * b * NF + 2 * b * K);
  }
  static constexpr size_t kBlkLdsMax = 156 * 1024;  // of a compute unit's 160 KB
  static constexpr int B = blk_lds(16) <= kBlkLdsMax ? 16 : blk_lds(8) <= kBlkLdsMax ? 8 : 4;
  static constexpr size_t kBlkLds = blk_lds(B);
  static constexpr bool kBlk = kBlkLds <= kBlkLdsMax;  // not the widest families

  // A barrier that orders the block's LDS accesses only: global loads and
  // stores in flight (observations, checkpoints) stay in flight.
  __device__ __forceinline__ static void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
  }
  // Lane u's value, the same in every lane.
  __device__ __forceinline__ static Y lane_value(Y v, int u) {
    if constexpr (sizeof(Y) == 4) {
      return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), u));
    } else {
      const uint64_t x = __builtin_bit_cast(uint64_t, v);
      const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)x, u);
      const uint32_t hi = __builtin_amdgcn_readlane((int)(uint32_t)(x >> 32), u);
      return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
    }
  }

  // Called by all threads of a 512-thread block whose waves hold the same
  // particles (lanes that are not live repeat a live one and write nothing).
  // The value, st and g are valid in wave 0.  kFwd as for value_and_grad().
  template <bool kFwd = true>
  __device__ static double block_value_and_grad(const Par &p, const double *th, int64_t t,
                                                const Y *__restrict__ y, R *ckpt, int64_t P,
                                                int64_t pidx, bool live, void *lds, double scale,
                                                double *g, R (&st)[Md::S], double se = 0.0) {
    if (t <= 0) {
#pragma unroll
      for (int k = 0; k < Md::S; ++k) st[k] = (R)0;
      return 0.0;
    }
    const int lane = threadIdx.x & 63;
    const int role = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    R *wbuf = static_cast<R *>(lds) + lane;   // [2][SEG * K][64]
    R *ring = wbuf + 2 * SEG * K * 64;        // [3][B * NF][64]
    R *wring = ring + 3 * B * NF * 64;        // [2][B * K][64]
    constexpr int Q = SEG / B;                // sub-blocks of a segment
    const int ns = (int)nseg(t), nb = (int)((t + B - 1) / B);
    // Observations of sub-block b, one per lane (repeated; beyond t the last
    // one): loaded a stage ahead by a vector load, so that no wait for LDS
    // waits for them, and read lane by lane.
    auto fetch = [&](int b) {
      const int64_t s = (int64_t)b * B + (lane & (B - 1));
      return y[min(s, t - 1)];
    };
    // Replays sub-block c of a segment into its buffer dst.
    auto replay = [&](R *dst, int c, Y yv, typename Md::Run &r) {
      R *d = dst + c * (B * K * 64);
#pragma unroll
      for (int u = 0; u < B; ++u) {
#pragma unroll
        for (int k = 0; k < K; ++k) d[(u * K + k) * 64] = r.w[k];
        R ae = (R)0, pm = (R)1, Ed, zd;
        (void)Md::step(p, lane_value(yv, u), r, ae, pm, Ed, zd);
      }
    };
    const int top = nb - (ns - 1) * Q;  // sub-blocks of the last segment
    double ll = 0.0;
    if (role == 0) {
      R *last = wbuf + ((ns - 1) & 1) * SEG * K * 64;
      if constexpr (kFwd) {
        ll = forward(p, t, y, ckpt, P, pidx, live, last, st, se);
      } else {  // the last segment's exponents by a replay
        typename Md::Run r;
        load_ckpt(ckpt, ns - 1, P, pidx, r);
        Y yv = fetch((ns - 1) * Q);
        for (int c = 0; c < top; ++c) {
          const Y yn = fetch(min((ns - 1) * Q + c + 1, nb - 1));
          replay(last, c, yv, r);
          yv = yn;
        }
      }
    }
    lds_barrier();
    Sums<double> tot;
    Sums<R> sum;
    clear(tot);
    clear(sum);
    auto count = [&](int b) { return b < nb - 1 ? B : (int)(t - (int64_t)b * B); };
    // f(u) for a sub-block's observations, last to first, unrolled when it is
    // whole
    auto reverse = [&](int b, auto &&f) {
      if (count(b) == B) {
#pragma unroll
        for (int u = B - 1; u >= 0; --u) f(u);
      } else {
        for (int u = count(b) - 1; u >= 0; --u) f(u);
      }
    };
    // One loop per role, each with the same nb + 2 stages and barriers.
    if (role == 0) {
      typename Md::Run r;
      R ck[K];  // the next segment's checkpoint
#pragma unroll
      for (int k = 0; k < K; ++k) ck[k] = r.w[k] = (R)0;
      r.sw = (R)0;
      Y yv = (Y)0;
      if (ns >= 2) {
#pragma unroll
        for (int k = 0; k < K; ++k) ck[k] = ckpt[((int64_t)(ns - 2) * K + k) * P + pidx];
        yv = fetch((ns - 2) * Q);
      }
      // While segment sg is in the first stage, replay sg - 1 into the other
      // buffer: a sub-block a stage; in FP32 from the second of sg's stages on
      // (chain() still reads sg + 1's exponents there in the first), two in
      // that one.  The last segment may have fewer stages than Q: then more.
      const int per = (Q + top - 1) / top;
      int k0 = 0;
      for (int i = 0; i < nb + 2; ++i) {
        const int bl = nb - 1 - i, sg = bl >= 0 ? bl / Q : 0;
        if (sg > 0) {
          int c0 = k0, c1 = k0 + 1;
          if (sg == ns - 1) {
            c0 = min(k0 * per, Q);
            c1 = min(c0 + per, Q);
          } else if (!kRingW) {
            c1 = k0 == 0 ? 0 : k0 + 1;
            c0 = k0 <= 1 ? 0 : k0;
          }
          k0 = bl % Q == 0 ? 0 : k0 + 1;
          R *dst = wbuf + ((sg - 1) & 1) * SEG * K * 64;
          for (int c = c0; c < c1; ++c) {
            if (c == 0) {
#pragma unroll
              for (int k = 0; k < K; ++k) r.w[k] = ck[k];
              open_segment(r);
              if (sg > 1)
#pragma unroll
                for (int k = 0; k < K; ++k)
                  ck[k] = ckpt[((int64_t)(sg - 2) * K + k) * P + pidx];
            }
            const Y yn = fetch(c + 1 < Q ? (sg - 1) * Q + c + 1 : max(sg - 2, 0) * Q);
            replay(dst, c, yv, r);
            yv = yn;
          }
        }
        lds_barrier();
      }
    } else if (role == 1) {
      R wb[K];  // adjoint of the exponents of the observation after the current one
#pragma unroll
      for (int k = 0; k < K; ++k) wb[k] = (R)0;
      lds_barrier();
      for (int b = nb - 1; b >= 0; --b) {
        const R *rg = ring + (b % 3) * (B * NF * 64);
        R *wr = wring + (b & 1) * (B * K * 64);
        const R *src = wbuf + ((b / Q) & 1) * SEG * K * 64 + (b % Q) * (B * K * 64);
        reverse(b, [&](int u) {
          const R *o = rg + u * (NF * 64);
          R w[K];
#pragma unroll
          for (int k = 0; k < K; ++k) {
            w[k] = kRingW ? o[(3 + NX + k) * 64] : src[(u * K + k) * 64];
            wr[(u * K + k) * 64] = wb[k];
          }
          sum_exponents(w, wb, sum);
          chain(p, o[0], o[64], o[128], wb);
        });
        if (b % Q == 0) flush_exponents(sum, tot);
        lds_barrier();
      }
      lds_barrier();
    } else if (role < 4) {
      lds_barrier();
      lds_barrier();
      Y yv = fetch(nb - 1);
      auto stages = [&](auto factors, auto shock, auto mixture) {
        for (int b = nb - 1; b >= 0; --b) {
          const Y yn = fetch(max(b - 1, 0));
          const R *rg = ring + (b % 3) * (B * NF * 64);
          const R *wr = wring + (b & 1) * (B * K * 64);
          reverse(b, [&](int u) {
            const R *o = rg + u * (NF * 64);
            R wbu[K], x[NXA];
            const R z = o[0], E = o[64], eb = o[128];
#pragma unroll
            for (int k = 0; k < K; ++k) wbu[k] = wr[(u * K + k) * 64];
#pragma unroll
            for (int q = 0; q < NX; ++q) x[q] = o[(3 + q) * 64];
            if constexpr (decltype(factors)::value) sum_factors(z, E, wbu, sum);
            if constexpr (decltype(shock)::value)
              sum_shock(p, lane_value(yv, u), z, E, eb, x, wbu, sum);
            if constexpr (decltype(mixture)::value) sum_mixture(p, z, E, x, sum);
          });
          if (b % Q == 0) {  // the segment's sums, as value_and_grad adds them
            flush_factors(sum, tot);
            flush_shock(sum, tot);
            flush_mixture(sum, tot);
          }
          yv = yn;
          lds_barrier();
        }
      };
      using yes = std::true_type;
      using no = std::false_type;
      if constexpr (kMix) {
        if (role == 2) stages(yes(), yes(), no());
        else stages(no(), no(), yes());
      } else {
        if (role == 2) stages(yes(), no(), no());
        else stages(no(), yes(), no());
      }
    } else {
      Y yv = fetch(nb - 1);
      for (int b = nb - 1; b >= 0; --b) {
        const Y yn = fetch(max(b - 1, 0));
        const R *src = wbuf + ((b / Q) & 1) * SEG * K * 64 + (b % Q) * (B * K * 64);
        R *rg = ring + (b % 3) * (B * NF * 64);
        auto one = [&](int u) {
          R w[K], z, E, eb, x[NXA];
#pragma unroll
          for (int k = 0; k < K; ++k) w[k] = src[(u * K + k) * 64];
          local(p, w, lane_value(yv, u), z, E, eb, x);
          R *o = rg + u * (NF * 64);
          o[0] = z;
          o[64] = E;
          o[128] = eb;
#pragma unroll
          for (int q = 0; q < NX; ++q) o[(3 + q) * 64] = x[q];
          if constexpr (kRingW)
#pragma unroll
            for (int k = 0; k < K; ++k) o[(3 + NX + k) * 64] = w[k];
        };
        const int n = count(b), r0 = role - (kBlkWaves - kLocal);
        if (r0 >= 0) {
          if (n == B) {
#pragma unroll
            for (int q = 0; q < B / kLocal; ++q) one(q * kLocal + r0);
            if (B % kLocal != 0 && B / kLocal * kLocal + r0 < B) one(B / kLocal * kLocal + r0);
          } else {
            for (int u = r0; u < n; u += kLocal) one(u);
          }
        }
        yv = yn;
        lds_barrier();
      }
      lds_barrier();
      lds_barrier();
    }
    // totals to wave 0
    double *td = reinterpret_cast<double *>(lds) + lane;
    auto each = [&](auto &&f) {
      constexpr int shock = kMix ? 2 : 3;
      int n = 0;
#pragma unroll
      for (int k = 0; k < K; ++k) {
        f(n++, tot.a[k], 1);
        f(n++, tot.c0[k], 2);
        f(n++, tot.kb[k], 2);
        f(n++, tot.kg[k], 2);
      }
      f(n++, tot.isig, shock);
      f(n++, tot.mus, shock);
      f(n++, tot.inu2, shock);
      f(n++, tot.hnu1, shock);
      if constexpr (kMix) {
#pragma unroll
        for (int q = 0; q < kNM; ++q) {
          f(n++, tot.lw[q], 3);
          f(n++, tot.nb[q], 3);
          f(n++, tot.mu[q], 3);
        }
      }
    };
    each([&](int n, double &v, int owner) {
      if (role == owner) td[n * 64] = v;
    });
    lds_barrier();
    if (role == 0) {
      each([&](int n, double &v, int) { v = td[n * 64]; });
      if constexpr (Md::kTLog) tot.hnu1 = -se;
      to_theta(th, t, tot, scale, g);
    }
    return ll;
  }

  // Chain rule from the totals to theta (Table 1 transforms), added to g.
  __device__ static void to_theta(const double *th, int64_t t, const Sums<double> &tot,
                                  double scale, double *g) {
#pragma clang fp contract(off)
    const double n = (double)t;
    const double isigb = tot.isig, musb = tot.mus, inu2b = tot.inu2, hnu1b = tot.hnu1;
    const double (&ab)[K] = tot.a, (&c0b)[K] = tot.c0, (&kbb)[K] = tot.kb, (&kgb)[K] = tot.kg;
    const double (&lwb)[kNM] = tot.lw, (&nbb)[kNM] = tot.nb, (&mub)[kNM] = tot.mu;
    const double isig = exp(-th[1]);
    const double mus = th[0] * 1e-3 * isig;
    g[0] += scale * (musb * 1e-3 * isig);
    g[1] += scale * (-isigb * isig - musb * mus - n);
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const double a = tanh(th[2 + k]);
      const double b = exp(th[2 + K + k]);
      g[2 + k] += scale * ab[k] * (1.0 - a * a);
      g[2 + K + k] += scale * (c0b[k] * (-Md::kKappa * b * kSqrt2OverPi) + kbb[k] * Md::kKappa * b);
      g[2 + 2 * K + k] += scale * kgb[k] * Md::kKappa;
    }
    if constexpr (kT) {
      const double en = exp(th[2 + 3 * K]);
      const double nu = 2.0 + en;
      const double dcst = en * 0.5 * (digamma_dev(0.5 * (nu + 1.0)) - digamma_dev(0.5 * nu)) - 0.5;
      const double hb = hnu1b * t_scale<R>();
      g[2 + 3 * K] += scale * (inu2b * (-1.0 / en) + hb * 0.5 * en + n * dcst);
    }
    if constexpr (kMix) mixture_chain(th, lwb, nbb, mub, scale, g);
  }
};

// The regression needs no recursion: one pass gives the value and gradient.
template <int NREG>
struct Adjoint<Linreg<NREG>> {
  using Md = Linreg<NREG>;
  static constexpr int kLdsPerLane = 0;
  __device__ static int64_t nseg(int64_t) { return 0; }
  __device__ static double value_and_grad(const DevModel &dm, const double *th, int64_t t,
                                          double scale, double *g) {
    double acc = 0.0, gb[NREG];
#pragma unroll
    for (int i = 0; i < NREG; ++i) gb[i] = 0.0;
    for (int64_t s = 0; s < t; ++s) {
      double r = dm.y[s];
#pragma unroll
      for (int i = 0; i < NREG; ++i) r = fma(-dm.X[s * NREG + i], th[i], r);
      acc = fma(r, r, acc);
#pragma unroll
      for (int i = 0; i < NREG; ++i) gb[i] = fma(r, dm.X[s * NREG + i], gb[i]);
    }
    const double iv = exp(-th[NREG]), n = (double)t;
#pragma unroll
    for (int i = 0; i < NREG; ++i) g[i] += scale * gb[i] * iv;
    g[NREG] += scale * (-0.5 * n + 0.5 * iv * acc);
    return n * (-0.5 * kLog2Pi - 0.5 * th[NREG]) - 0.5 * iv * acc;
  }
};

template <int NREG>
struct PriorGradLin {
  __device__ static void run(const double *th, double *g) {
    const double eta = th[NREG], iv = exp(-eta);
    double sb = 0.0;
#pragma unroll
    for (int i = 0; i < NREG; ++i) {
      g[i] = -th[i] * iv / Linreg<NREG>::kC0;
      sb += th[i] * th[i];
    }
    g[NREG] = -Linreg<NREG>::kA0 + Linreg<NREG>::kB0 * iv - 0.5 * NREG +
              0.5 * sb * iv / Linreg<NREG>::kC0;
  }
};

template <class M>
struct PriorGradOf;
template <int K, int SH, typename R, int I>
struct PriorGradOf<Egarch<K, SH, R, I>> {
  __device__ static void run(const double *th, double *g) { PriorGrad<K, SH, R, I>::run(th, g); }
};
template <int NREG>
struct PriorGradOf<Linreg<NREG>> {
  __device__ static void run(const double *th, double *g) { PriorGradLin<NREG>::run(th, g); }
};

}  // namespace smc
