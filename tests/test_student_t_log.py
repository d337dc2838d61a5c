"""The FP64 Student-t density's logarithm (model.h, log1p_pos and the product
of a group's factors): its arithmetic replayed on the CPU against long double,
and the GPU likelihood against the oracle at the edges of the groups of 8
observations, for large nu and for shocks whose product of factors leaves the
double range (the group then takes its logarithms one by one)."""
import os
import re
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
MODEL_H = os.path.join(ROOT, "paper_1304_4334_amd", "csrc", "model.h")


def test_log1p_pos_error_within_two_ulp(tmp_path):
    """p in (0, 1e300), the hardware reciprocals replaced by ones with a
    relative error of 2^-22; 0 and inf exact.  The last subtraction rounds to
    half an ulp, the terms before it are at most half the result and carry
    one ulp each, so the sum stays under 2 ulp."""
    if shutil.which("gcc") is None:
        pytest.skip("gcc not available")
    src = open(MODEL_H).read()
    coef = re.search(r"kLog1pCoef\[7\]\s*=\s*\{([^}]*)\}", src).group(1)
    hi, lo = re.search(r"kLn2Hi\s*=\s*([0-9a-fA-Fx.p+-]+)\s*,\s*kLn2Lo\s*=\s*([0-9a-fA-Fx.p+-]+);",
                       src).groups()
    rt = re.search(r"kSqrtHalf\s*=\s*([0-9a-fA-Fx.p+-]+);", src).group(1)
    c_file = tmp_path / "l.c"
    c_file.write_text(f"""
#include <math.h>
#include <stdio.h>
static const double C[7] = {{{coef}}};
static double rcp(double x) {{ return (1.0 / x) * (1.0 + 0x1p-22); }}
static double lg(double p) {{
  double u = 1.0 + p, c = p - (u - 1.0);
  int e;
  double m = frexp(u, &e);
  int up = m < {rt};
  m = ldexp(m, up);
  double k = e - up, f = m - 1.0, d = 2.0 + f, r = rcp(d);
  r = fma(r, fma(-d, r, 1.0), r);
  double s = f * r;
  s = fma(fma(-d, s, f), r, s);
  double z = s * s, q = C[6];
  for (int j = 5; j >= 0; --j) q = fma(q, z, C[j]);
  double l = fma(k, {lo}, ldexp(c, -(e - up)));
  double v = fma(k, {hi}, f - fma(s, fma(-z, q, f), -l));
  return p < INFINITY ? v : p;
}}
int main(void) {{
  double worst = 0.0;
  unsigned long long s = 12345;
  for (int i = 0; i < 3000000; ++i) {{
    s = s * 6364136223846793005ull + 1442695040888963407ull;
    double u = (double)(s >> 11) * 0x1.0p-53;
    double p = (i % 3 == 0) ? 4.0 * u : (i % 3 == 1 ? exp(-40.0 * u) : exp(690.0 * u));
    long double ref = log1pl((long double)p);
    double ulp = nextafter((double)ref, INFINITY) - (double)ref;
    double err = fabs((double)((long double)lg(p) - ref)) / ulp;
    if (err > worst) worst = err;
  }}
  printf("%.6f %.17g %.17g\\n", worst, lg(INFINITY), lg(0.0));
  return 0;
}}
""")
    exe = tmp_path / "l"
    subprocess.run(["gcc", "-O2", "-o", str(exe), str(c_file), "-lm"], check=True)
    worst, at_inf, at_zero = map(float, subprocess.run(
        [str(exe)], check=True, capture_output=True, text=True).stdout.split())
    assert worst < 2.0, worst
    assert at_inf == np.inf and at_zero == 0.0


@pytest.mark.gpu
@pytest.mark.parametrize("K", [1, 2])
@pytest.mark.parametrize("t", [1, 2, 7, 8, 9, 10, 16, 17, 24, 25, 33])
def test_likelihood_and_cphase_at_group_edges(K, t):
    """Log likelihood and C-phase weights over 1..t, nu from near 2 to 1e4
    (beyond it both sides' constants cancel above the bar):
    1e-10 relative, the bar of every FP64 likelihood test."""
    import oracle as O
    import paper_1304_4334_amd as S
    import synthdata as SD
    import torch
    from tests.gpu_helpers import gpu_model, ora_model, pop_to_gpu
    th = SD.egarch2t_truth()
    th = th if K == 2 else th[[0, 1, 2, 4, 6, 8]]
    y = SD.egarch_series(th, 40, K, SD.STUDENT_T, 7)
    w = SD.Workload("t", SD.EGARCH, K=K, shock=SD.STUDENT_T, T=40, J=2, N=64, y=y, theta_true=th)
    gm, om = gpu_model(w), ora_model(w)
    opop = O.Pop(om, 2, 64)
    opop.theta[:] = SD.random_thetas(w, 128, 5, spread=0.05)
    opop.theta[:, -1] = np.linspace(-6.0, np.log(1e4), 128)
    want, _ = O.loglik_batch(om, opop.theta, t)
    g = pop_to_gpu(gm, opop)
    got = S.smc_loglik(gm, g.theta, t).cpu().numpy()
    assert np.allclose(got, want, rtol=1e-10, atol=0.0)
    S.smc_correct(gm, g, 0, t, rss_min=0.0, want_rss=False)
    assert np.allclose(g.logw.cpu().numpy(), want, rtol=1e-10, atol=0.0)
    torch.cuda.synchronize()


@pytest.mark.gpu
@pytest.mark.parametrize("scale", [1e12, 1e40, 1e120])
def test_products_beyond_the_double_range(scale):
    """Shocks of 1e12 to 1e120 standard deviations (loadings of 1e-130, so the
    volatility stays put): products of eight factors up to 1e1920."""
    import oracle as O
    import paper_1304_4334_amd as S
    import synthdata as SD
    from tests.gpu_helpers import gpu_model, ora_model
    import torch
    th = SD.egarch2t_truth()
    th[4:6] = -300.0
    th[6:8] = 0.0
    y = 0.01 * np.random.default_rng(3).standard_normal(37)
    y[3:19] *= scale
    w = SD.Workload("t", SD.EGARCH, K=2, shock=SD.STUDENT_T, T=37, J=2, N=32, y=y, theta_true=th)
    gm, om = gpu_model(w), ora_model(w)
    theta = np.tile(th, (64, 1))
    theta[:, -1] = np.linspace(-3.0, 6.0, 64)
    for t in (3, 5, 8, 16, 37):
        want, _ = O.loglik_batch(om, theta, t)
        got = S.smc_loglik(gm, torch.from_numpy(theta.T.copy()).cuda(), t).cpu().numpy()
        assert np.isfinite(want).all()
        assert np.allclose(got, want, rtol=1e-10, atol=0.0)
