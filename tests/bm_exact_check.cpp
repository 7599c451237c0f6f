// Host check of both Box-Muller generators against extended-precision libm:
// root mean square and worst error in units of 2^-52 (relative for -2 ln u,
// absolute for sine, cosine and the normals), over pseudo-random arguments, the
// ends of the range and both sides of every row and quadrant.
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "lbl_math.hpp"

struct Err {
  double worst = 0, sum2 = 0;
  long n = 0;
  void add(long double got, long double ref, long double scale) {
    const double e = static_cast<double>((got - ref) / scale) * 0x1p52;
    worst = std::fmax(worst, std::fabs(e));
    sum2 += e * e;
    ++n;
  }
  void print(const char* gen, const char* what) const {
    std::printf("%s_%s_rms %.4f\n%s_%s_max %.4f\n", gen, what, std::sqrt(sum2 / n), gen, what, worst);
  }
};

int main(int argc, char** argv) {
  const long n = argc > 1 ? std::atol(argv[1]) : 1000000;
  const long double two_pi = 6.283185307179586476925286766559005768L;
  std::vector<uint32_t> edges;
  for (uint32_t j = 0; j < 128; ++j)
    for (int d = -2; d < 2; ++d) {
      edges.push_back((j << 25) + static_cast<uint32_t>(d));      // rows of the angle
      for (int o = 0; o < 25; o += 4)                             // rows of the mantissa
        edges.push_back(((128u + j) << (24 - o)) + static_cast<uint32_t>(d));
    }
  for (uint32_t k = 0; k < 1024; ++k) {
    edges.push_back(k);
    edges.push_back(0xffffffffu - k);
  }
  const char* name[2] = {"rows", "poly"};
  Err ln[2], sn[2], cs[2], z[2], edge[2];
  uint64_t lcg = 0x9e3779b97f4a7c15ULL;
  auto next = [&] {
    lcg = lcg * 6364136223846793005ULL + 1442695040888963407ULL;
    return static_cast<uint32_t>(lcg >> 32);
  };
  const long ne = static_cast<long>(edges.size());
  for (long i = 0; i < n + ne; ++i) {
    const bool at = i < ne;
    const uint32_t ka = at ? edges[i] : next(), kb = at ? edges[i] : next();
    const long double ua = (static_cast<long double>(ka) + 0.5L) / 4294967296.0L;
    const long double ub = (static_cast<long double>(kb) + 0.5L) / 4294967296.0L;
    const long double l = -2.0L * logl(ua), s = sinl(two_pi * ub), c = cosl(two_pi * ub);
    const double x = static_cast<double>(ka) + 0.5;
    for (int g = 0; g < 2; ++g) {
      const double lg = g ? lbl::bm::neg2_log_poly(x) : lbl::bm::neg2_log(x, lbl::bm::kTables.log);
      double sg, cg;
      if (g)
        lbl::bm::sincos_poly(kb, &sg, &cg);
      else
        lbl::bm::sincos_turn(kb, &sg, &cg);
      if (at) {
        edge[g].add(lg, l, l);
        edge[g].add(sg, s, 1.0L);
        edge[g].add(cg, c, 1.0L);
        continue;
      }
      ln[g].add(lg, l, l);
      sn[g].add(sg, s, 1.0L);
      cs[g].add(cg, c, 1.0L);
      z[g].add(std::sqrt(lg) * cg, sqrtl(l) * c, 1.0L);
      z[g].add(std::sqrt(lg) * sg, sqrtl(l) * s, 1.0L);
    }
  }
  for (int g = 0; g < 2; ++g) {
    ln[g].print(name[g], "log");
    sn[g].print(name[g], "sin");
    cs[g].print(name[g], "cos");
    z[g].print(name[g], "z");
    edge[g].print(name[g], "edge");
  }
  return 0;
}
