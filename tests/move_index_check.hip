// Host check of the division by multiplication in csrc/kernels_basic.h (built and run by tests/test_move_index.py).
#include <cstdio>
#include <cstdint>

#include "../paper_2105_04663_amd/csrc/kernels_basic.h"

int main() {
  using namespace gspmd;
  uint64_t x = 88172645463325252ull;
  auto rnd = [&] { x ^= x << 13; x ^= x >> 7; x ^= x << 17; return x; };
  auto check = [](uint32_t n, uint32_t d) { if (div_by(n, fast_div(d)) != n / d) { std::printf("%u / %u\n", n, d); return false; } return true; };
  const uint32_t top = 0x7fffffffu;
  for (int i = 0; i < 400000; ++i) {
    const uint32_t d = i < 5000 ? i + 1 : i < 5100 ? top - (i - 5000) : 1u + static_cast<uint32_t>(rnd() % (uint64_t(1) << (1 + rnd() % 31))) % top;
    for (int j = 0; j < 8; ++j) {
      const uint32_t q = static_cast<uint32_t>(rnd() % (top / d + 1));      // around multiples of d, where a quotient changes
      const uint64_t n = static_cast<uint64_t>(q) * d;
      if (n <= top && !check(static_cast<uint32_t>(n), d)) return 1;
      if (n >= 1 && n - 1 <= top && !check(static_cast<uint32_t>(n - 1), d)) return 1;
    }
    if (!check(top, d) || !check(0, d) || !check(static_cast<uint32_t>(rnd() & top), d)) return 1;
  }
  for (int b = 0; b < 31; ++b)
    for (uint32_t d : {1u << b, (1u << b) + 1, (1u << b) - 1})
      if (d >= 1 && d <= top && (!check(top, d) || !check(top - 1, d) || !check(top - (top % d), d))) return 1;
  std::printf("move index ok\n");
  return 0;
}
