// The rule for rows used in place over memory kinds, devices and addresses (built by tests/test_rows_in_place.py with g++).
#include <cstdio>

#include "rows.hpp"

int main() {
  const std::uintptr_t p = 1u << 20;
  int bad = 0;
  auto check = [&](bool want, bool device_memory, int mem, int sys, std::uintptr_t at) {
    if (stern::rows_in_place(device_memory, mem, sys, at) != want) {
      std::printf("device_memory %d, device %d of %d, address %% 16 = %d: not %d\n", device_memory, mem, sys, (int)(at % 16), want);
      ++bad;
    }
  };
  for (int sys = 0; sys < 8; ++sys)
    for (int mem = 0; mem < 8; ++mem)
      for (int off = 0; off < 32; off += 8) {
        check(mem == sys && off % 16 == 0, true, mem, sys, p + off);
        check(false, false, mem, sys, p + off);
      }
  check(false, true, -1, 0, p);  // a place the runtime does not name
  return bad != 0;
}
