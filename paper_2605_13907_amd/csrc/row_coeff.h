// What one row contributes to the loss of Eq. 19 and to its gradient, in fp64: shared by the kernel that writes the
// coefficients of a batch and by the gradient sweep of small batches, which forms its own.
#pragma once

#include <hip/hip_runtime.h>

#include "ais.h"

namespace ais {

// The arrays and parameters behind a row's coefficient, as the entry points take them.
struct CoeffInputs {
  const float *logp_train, *logp_roll, *logp_old, *logp_ref;
  const unsigned char* valid;
  const long long* cu_rows;
  int n_resp;
  const float* adv;
  const int* count;
  const ais_diag* diag;
  ais_params p;
  double lnC;
};

namespace dev {

// e^x to about an ulp: x = n ln 2 + r with |r| <= ln(2) / 2, e^r by its Taylor series, whose remainder after the 13th power is
// below 2^-57.  Half the instructions of the library's exp.  x neither NaN nor infinite.
__device__ __forceinline__ double exp64_finite(double clamped) {
  const double n = rint(clamped * 1.4426950408889634);
  const double r = fma(n, -0x1.abc9e3b39803fp-56, fma(n, -0x1.62e42fefa39efp-1, clamped));
  double p = 1.0 / 6227020800.0;
  p = fma(p, r, 1.0 / 479001600.0);
  p = fma(p, r, 1.0 / 39916800.0);
  p = fma(p, r, 1.0 / 3628800.0);
  p = fma(p, r, 1.0 / 362880.0);
  p = fma(p, r, 1.0 / 40320.0);
  p = fma(p, r, 1.0 / 5040.0);
  p = fma(p, r, 1.0 / 720.0);
  p = fma(p, r, 1.0 / 120.0);
  p = fma(p, r, 1.0 / 24.0);
  p = fma(p, r, 1.0 / 6.0);
  p = fma(p, r, 0.5);
  p = fma(p, r, 1.0);
  p = fma(p, r, 1.0);
  return ldexp(p, (int)n);
}
// For any x: infinity and 0 at the ends, NaN stays NaN.
__device__ __forceinline__ double exp64(double x) {
  const double e = exp64_finite(fmin(fmax(x, -800.0), 800.0));
  return x != x ? x : e;
}

struct CoeffRule {
  double alpha, lnC, lo_clip, hi_clip, beta_kl;
  bool has_old, kl;
  __device__ __forceinline__ CoeffRule(const ais_params& p, double alpha_, double lnC_, bool old, bool ref)
      : alpha(alpha_), lnC(lnC_), lo_clip(1.0 - (double)p.clip_eps), hi_clip(1.0 + (double)p.clip_eps),
        beta_kl((double)p.beta_kl), has_old(old), kl(ref && p.beta_kl > 0.f) {}
};

// Weight of a response's rows: 1/G and 1/|o_i| of Eq. 19 over all prompts.
__device__ __forceinline__ double response_weight(int n_resp, int count) {
  return count > 0 ? 1.0 / ((double)n_resp * (double)count) : 0.0;
}

struct RowTerm {
  double wtilde;    // rectification weight
  double obj;       // the row's term of the objective
  double dobj;      // its derivative by the row's log-prob
};

// a: the response's advantage.
__device__ __forceinline__ RowTerm row_term(const CoeffRule& c, float lt_f, float roll_f, float old_f, float ref_f,
                                            double a) {
  const double lt = (double)lt_f;
  // the sampler-trainer ratio is taken at the checkpoint that generated the rollout (Alg. 1, "Sampler-Trainer
  // ratio"; Sec. 3.2: the two ratios are orthogonal), the old-new ratio between that checkpoint and theta
  const double l_old = c.has_old ? (double)old_f : lt;
  const double wbar = exp64(fmin(l_old - (double)roll_f, c.lnC));
  RowTerm r;
  r.wtilde = 1.0 + c.alpha * (wbar - 1.0);                                  // Eq. 18 / Alg. 1 rectification weight
  const double rho_on = c.has_old ? exp64(lt - l_old) : 1.0;
  const double clipped = fmin(fmax(rho_on, c.lo_clip), c.hi_clip);
  // the unclipped branch is the minimum (ties included) iff the ratio has not left the trust
  // region on the side the advantage pushes towards
  const bool active = (a >= 0.0) ? (rho_on <= c.hi_clip) : (rho_on >= c.lo_clip);
  const double s = active ? rho_on * a : clipped * a;
  r.obj = r.wtilde * s;
  r.dobj = active ? r.wtilde * a * rho_on : 0.0;
  if (c.kl) {
    const double q = (double)ref_f - lt;
    const double eq = exp64(q);
    r.obj -= c.beta_kl * (eq - q - 1.0);
    r.dobj -= c.beta_kl * (1.0 - eq);
  }
  return r;
}

}  // namespace dev
}  // namespace ais
