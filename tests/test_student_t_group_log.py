"""The logarithm of a group of eight FP64 Student-t factors (model.h:
log1p_pos, t_join and t_group_log): the functions' own text compiled for the
CPU and compared with long double, beside the sum of eight logarithms of the C
library."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
MODEL_H = os.path.join(ROOT, "paper_1304_4334_amd", "csrc", "model.h")

HARNESS = r"""
#include <math.h>
#include <stdio.h>
#define __device__
#define __forceinline__ inline
using std::fma;
// the hardware's frexp pair, and a reciprocal with a relative error of 2^-22
static double frexp_mant(double x) { int e; return frexp(x, &e); }
static int frexp_exp(double x) { int e; frexp(x, &e); return e; }
#define __builtin_amdgcn_frexp_mant frexp_mant
#define __builtin_amdgcn_frexp_exp frexp_exp
#define __builtin_amdgcn_rcp(x) ((1.0 / (x)) * (1.0 + 0x1p-22))
typedef double R;
constexpr int kAcc = 8;
%s
static unsigned long long seed = 12345;
static double uniform() {
  seed = seed * 6364136223846793005ull + 1442695040888963407ull;
  return ((double)(seed >> 11) + 0.5) * 0x1p-53;
}
int main() {
  double worst = 0.0, alone = 0.0;
  for (int i = 0; i < 3000000; ++i) {
    const double u = uniform();
    const double p = i %% 3 == 0 ? 4.0 * u : (i %% 3 == 1 ? exp(-40.0 * u) : exp(690.0 * u));
    const long double ref = log1pl((long double)p);
    const double ulp = nextafter((double)ref, INFINITY) - (double)ref;
    worst = fmax(worst, fabs((double)((long double)log1p_pos(p) - ref)) / ulp);
    alone = fmax(alone, fabs((double)((long double)log1p_pos<true>(p) - ref)) / ulp);
  }
  printf("%%.6f %%.6f %%.17g %%.17g %%.17g %%.17g\n", worst, alone, log1p_pos(INFINITY),
         log1p_pos(0.0), log1p_pos<true>(INFINITY), log1p_pos<true>(0.0));
  const double scales[] = {1e-8, 1e-6, 1e-4, 1e-3, 1e-2, 0.03, 0.1, 0.3, 1, 3, 10, 100, 1e6};
  for (double sc : scales) {
    double mx[2] = {0, 0}, mean[2] = {0, 0};
    const int n = 40000;
    for (int i = 0; i < n; ++i) {
      double x[8], sum = 0.0;
      long double ref = 0;
      for (int j = 0; j < 8; ++j) {
        const double g = sqrt(-2.0 * log(uniform())) * cos(6.283185307179586 * uniform());
        x[j] = sc * g * g;
        ref += log1pl((long double)x[j]);
        sum += log1p(x[j]);
      }
      const double v[2] = {t_group_log(x), sum};
      for (int k = 0; k < 2; ++k) {
        const double e = fabs((double)(((long double)v[k] - ref) / ref));
        mean[k] += e / n;
        mx[k] = fmax(mx[k], e);
      }
    }
    printf("%%g %%.4e %%.4e %%.4e %%.4e\n", sc, mx[0], mx[1], mean[0], mean[1]);
  }
  // a product beyond the range, a factor that is infinite or not a number
  double big[8] = {1e300, 1e300, 1e300, 3.0, 0.0, 1e300, 1e-9, 1e300};
  double want = 0.0;
  for (double q : big) want += log1p(q);
  printf("%%.17g %%.17g ", t_group_log(big), want);
  big[2] = INFINITY;
  printf("%%g ", t_group_log(big));
  big[2] = NAN;
  printf("%%g ", t_group_log(big));
  double zero[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  printf("%%g\n", t_group_log(zero));
  return 0;
}
"""


def _function(src, head):
    """The text of the function whose definition starts with `head`."""
    a = src.index(head)
    i = src.index("{", a)
    depth = 0
    for j in range(i, len(src)):
        depth += {"{": 1, "}": -1}.get(src[j], 0)
        if depth == 0:
            return src[a:j + 1]
    raise AssertionError(head)


def test_group_logarithm_is_as_close_as_the_eight_logarithms_it_replaces(tmp_path):
    """log1p_pos standing alone: the last addition rounds to half an ulp, the
    terms before it are at most a quarter of the result and those that round lie
    three binades below it (two of them, a sixteenth each), the second-order form of
    c / u adds less than a fortieth: 0.65 ulp; as part of a group 2 ulp, as
    the last subtraction and the one before it round at the result's size with
    an ulp each for the terms before.  A group's error, largest and mean over
    shocks of each size, is no larger than that of the eight logarithms added
    one by one."""
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    src = open(MODEL_H).read()
    parts = re.findall(r"^constexpr double kSqrtHalf = [^;]*;", src, re.M)
    parts += re.findall(r"^constexpr double kLn2Hi = [^;]*;", src, re.M)
    parts += re.findall(r"^constexpr double kLn2Lead = [^;]*;", src, re.M)
    parts += re.findall(r"constexpr double kLog1pCoef\[7\] = \{[^}]*\};", src)
    parts += [_function(src, "template <bool kAlone = false>\n__device__ __forceinline__ double log1p_pos("),
              _function(src, "__device__ __forceinline__ static R t_join("),
              _function(src, "__device__ __forceinline__ static R t_group_log(")]
    cpp, exe = tmp_path / "t.cpp", tmp_path / "t"
    cpp.write_text(HARNESS % "\n".join(parts))
    subprocess.run(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-o", str(exe), str(cpp)],
                   check=True)
    lines = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split("\n")
    worst, alone, *ends = map(float, lines[0].split())
    assert worst < 2.0 and alone < 0.65
    assert ends == [float("inf"), 0.0, float("inf"), 0.0]
    rows = [list(map(float, x.split())) for x in lines[1:14]]
    assert len(rows) == 13
    for scale, mx, mx_lib, mean, mean_lib in rows:
        assert mx <= mx_lib and mean <= mean_lib, scale
    got, want, inf, nan, zero = map(float, lines[14].split())
    assert abs(got - want) <= 1e-15 * want
    assert inf == float("inf") and nan != nan and zero == 0.0
