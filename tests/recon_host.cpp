// The reconstruction of csrc/recon.h compiled for the CPU: the forward pass's bound
// (bound_F) against the adjoint's (canon_at) on seeded measures, each a mixture of one
// to six normals. Prints, per number of atoms and kind of measure, the queries and how
// many of them differ in any bit.
#include <cstdio>
#include <random>

#define __builtin_amdgcn_rcpf(x) (1.0f / (x))
#define __builtin_amdgcn_rsqf(x) (1.0f / sqrtf(x))
#define __builtin_amdgcn_sqrtf(x) sqrtf(x)
#define __builtin_amdgcn_exp2f(x) exp2f(x)
// the median of three; with a NaN among them the least of the others
static inline float median3(float a, float b, float c) {
  if (a != a || b != b || c != c) return fminf(fminf(a, b), c);
  return fmaxf(fminf(a, b), fminf(fmaxf(a, b), c));
}
#define __builtin_amdgcn_fmed3f(a, b, c) median3(a, b, c)
#include "recon.h"

struct Kind {
  const char* name;
  double spread, offset, narrow, uneven;  // log range of the scale, offset, log range of the widths, log weights
};
static const Kind kKinds[] = {
    {"centred", 1.0, 0.0, 3.0, 0.0},
    {"off-centre", 2.5, 1.0, 3.0, 0.0},
    {"coincident", 6.0, 2.0, 8.0, 4.0},
};

template <int NH>
static void compare(const Kind& kind, int n_measures) {
  constexpr int NK = 2 * NH + 1;
  std::mt19937_64 rng(10 * NH + (&kind - kKinds));
  std::uniform_real_distribution<double> uni(0.0, 1.0);
  std::normal_distribution<double> nor;
  long queries = 0, differ = 0;
  for (int i = 0; i < n_measures; ++i) {
    const int n = 1 + (int)(6 * uni(rng));
    const double scale = std::exp(-kind.spread * uni(rng)), offset = kind.offset * nor(rng);
    double c[6], s[6], w[6], sum = 0.0, b[NK] = {}, mix[NK];
    for (int j = 0; j < n; ++j) {
      c[j] = offset + scale * nor(rng);
      s[j] = scale * std::exp(-kind.narrow * uni(rng));
      w[j] = std::exp(kind.uneven * nor(rng)) * (0.05 + uni(rng));
      sum += w[j];
    }
    for (int j = 0; j < n; ++j) {
      double m[NK];
      mb::normal_moments<NK>(c[j], s[j] * s[j], m);
      for (int k = 0; k < NK; ++k) b[k] += w[j] / sum * m[k];
    }
    b[0] = 1.0;
    mb::LInv<NH> L;
    mb::hankel_factor<NH>(b, L, mix);
    for (int q = 0; q < 16; ++q) {
      const int j = (int)(n * uni(rng));
      const float y = (float)(c[j] + 1.5 * s[j] * nor(rng));
      float x[NH], w0;
      bool below[NH];
      const float f = mb::bound_F<NH>(L, y, 0.25f);
      const float g = mb::canon_at<NH>(L, y, 0.25f, x, below, w0);
      ++queries;
      differ += memcmp(&f, &g, sizeof f) != 0 && !(f != f && g != g);
    }
  }
  std::printf("%d %s %ld %ld\n", NH, kind.name, queries, differ);
}

int main() {
  for (const Kind& k : kKinds) {
    compare<2>(k, 40000);
    compare<3>(k, 40000);
    compare<4>(k, 40000);
  }
  return 0;
}
