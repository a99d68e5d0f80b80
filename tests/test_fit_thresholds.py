"""The two ways the fit decides an encoding threshold (smallest float32 t with t >= b^(k + 1/2 - s)):
an interval in long double, and exact integers where the interval leaves two float32 values. Ties,
where b^(k + 1/2 - s) is itself a float32, are the thresholds that only the integers decide."""
import subprocess
from fractions import Fraction

import numpy as np
import pytest

from oracle import logbq_oracle as O
from paper_2607_01127_amd import build
from paper_2607_01127_amd import logbq as L


@pytest.mark.parametrize("bits,root,w,eps", [
    (4, Fraction(3, 2), [1.0, 4782969 * 2.0 ** -14, 0.0], 1e-9),         # b = 9/4, s = 0
    (8, Fraction(2), [2.0 ** -127, 2.0 ** 127, 0.0], 1e-160),            # b = 4, s = 64
], ids=["4-bit", "8-bit"])
def test_fit_thresholds_ties(bits, root, w, eps):
    """w_max / w_min is a power of a base b = root^2 that float64 gives exactly, so the thresholds
    are root^n, n odd: on 8 bits n = -127 .. 125, every one a float32, so both of the exact path's
    sweeps run; one representable too high or too low would show."""
    w = np.array(w, dtype=np.float32)
    r = O.fit_exact(w, bits, eps)
    for fit in (L.fit, L.fit_exact):
        p = fit(w, bits, eps)
        assert p.base == r.base == float(root * root) and p.shift == r.shift
        th = p.thresholds_array()[:p.qmax]
        assert [Fraction(float(t)) for t in th] == \
            [root ** (2 * k + 1 - 2 * p.shift) for k in range(p.qmax)]
        assert th.view(np.uint32).tolist() == \
            O.magnitude_thresholds(r.base, r.shift, bits).view(np.uint32).tolist()


HARNESS = r"""
#include "fit.cpp"
#include <cstdio>
#include <random>
int main() {
  auto exact = [](double b, int32_t s, int k) {
    uint64_t B; int64_t eb;
    split_f64(b, B, eb);
    const int64_t n = 2 * int64_t(k) + 1 - 2 * int64_t(s);
    return exact_threshold(b, s, k, pow_big(B, n < 0 ? -n : n));
  };
  int bad = 0;
  // Random bases of both widths, thresholds over the whole float32 range, |n| to some thousands.
  std::mt19937_64 rng(5);
  std::uniform_real_distribution<double> u(0.0, 1.0);
  long decided = 0, open = 0;
  for (int i = 0; i < 3000; ++i) {
    const bool wide = i % 2 == 0, big = i % 50 == 0;
    const double b = 1.0 + (wide ? 0.3 + 5.0 * u(rng) : (big ? 0.05 : 0.4) * (0.3 + 0.7 * u(rng)));
    const double e = (-102.0 + 190.0 * u(rng)) / std::log(b);    // threshold near exp(-102 .. 88)
    const int k = int(u(rng) * (wide ? 7 : 127));
    const int32_t s = int32_t(std::floor(k + 0.5 - e));
    float t = -1.0f;
    if (!interval_threshold(b, s, k, &t)) { ++open; continue; }
    ++decided;
    if (f2u(t) != f2u(exact(b, s, k))) { std::printf("differs: b %.17g s %d k %d\n", b, s, k); ++bad; }
  }
  if (decided < 2900) { std::printf("decided only %ld, left open %ld\n", decided, open); ++bad; }
  // Ties, thresholds past the largest float32: left open, and right by the integers.
  auto tie = [&](double b, int32_t s, int k, float want) {
    float t = -1.0f;
    if (interval_threshold(b, s, k, &t)) { std::printf("decides a tie: b %g s %d k %d\n", b, s, k); ++bad; }
    if (exact(b, s, k) != want) { std::printf("exact: b %g s %d k %d\n", b, s, k); ++bad; }
  };
  for (int n = -149; n <= 127; n += 2) tie(4.0, (7 - n) / 2, 3, std::ldexp(1.0f, n));
  for (int n = 1; n <= 15; n += 2) tie(2.25, (7 - n) / 2, 3, (float)std::pow(1.5, n));
  tie((1.0 + 0x1p-10) * (1.0 + 0x1p-10), 126, 126, 1.0f + 0x1p-10f);
  tie(4.0, -150, 3, std::numeric_limits<float>::infinity());
  std::printf("%s\n", bad ? "FAILED" : "ok");
  return bad != 0;
}
"""


def test_threshold_interval_against_integers(tmp_path):
    """interval_threshold decides nearly every threshold, always as the exact integers do, and
    refuses ties and overflow."""
    (tmp_path / "harness.cpp").write_text(HARNESS)
    exe = str(tmp_path / "harness")
    subprocess.run(["g++", *build.HOST_FLAGS, "-Wno-unused-function", "-pthread", "-I", build.CSRC,
                    str(tmp_path / "harness.cpp"), "-o", exe], check=True)
    out = subprocess.run([exe], capture_output=True, text=True, timeout=100)
    assert out.returncode == 0 and out.stdout.endswith("ok\n"), out.stdout[-2000:]
