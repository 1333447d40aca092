// Standard normal numbers of a seed (host code, plain C++).
#pragma once
#include <cmath>
#include <random>

// Marsaglia's polar method on mt19937_64: the same numbers in the same order, bit for bit, as
// std::normal_distribution<double>(0, 1) draws from it, which made the weights of every seed so far.
// That one's uniform numbers go through long double on the x87 stack here, at 36 or 66 ns a number
// as the linker happens to place the code (the 1.9 million weights of the training net: 69 or
// 127 ms; 13 ms this way).
class NormalStream {
 public:
  explicit NormalStream(unsigned long long seed) : rng_(seed) {}
  double operator()() {
    if (have_) {
      have_ = false;
      return kept_;
    }
    double x, y, r2;
    do {
      x = 2.0 * unit() - 1.0;
      y = 2.0 * unit() - 1.0;
      r2 = x * x + y * y;
    } while (r2 > 1.0 || r2 == 0.0);
    const double m = std::sqrt(-2.0 * std::log(r2) / r2);
    kept_ = x * m;
    have_ = true;
    return y * m;
  }

 private:
  // uniform in [0, 1)
  double unit() {
    const double u = (double)rng_() * 0x1p-64;
    return u < 1.0 ? u : 1.0 - 0x1p-53;
  }
  std::mt19937_64 rng_;
  double kept_ = 0.0;
  bool have_ = false;
};
