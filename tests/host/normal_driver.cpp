// fill_normal against std::normal_distribution, bit for bit (built by tests/test_host_normal.py with g++).
#include <cstdio>
#include <cstring>

#include "hostla.hpp"

int main() {
  for (unsigned long long seed : {0ull, 1ull, 7ull, 12345ull, ~0ull})
    for (std::size_t n : {0ul, 1ul, 2ul, 3ul, 311ul, 312ul, 313ul, 100001ul}) {
      std::mt19937_64 a(seed), b(seed);
      std::vector<double> x(n), y(n);
      stern::fill_normal(a, x.data(), n);
      std::normal_distribution<double> nd;
      for (double& v : y) v = nd(b);
      if (std::memcmp(x.data(), y.data(), n * sizeof(double)) != 0 || a != b) {
        std::printf("seed %llu, %zu values differ\n", seed, n);
        return 1;
      }
    }
  return 0;
}
