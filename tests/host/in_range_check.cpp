// The wrapping range test at the limits of the integer tests, as constant
// expressions: a signed overflow in one does not compile.
#include "../../paper_2107_11810_amd/csrc/gv_device.h"

constexpr int32_t LIM = (1 << 30) - 1;
constexpr bool nowhere_passes() {
  const int32_t xs[] = {-LIM, -4097, -1, 0, 1, 4097, LIM};
  const uint32_t Rs[] = {0u, 1u, 8190u, (uint32_t)LIM};
  for (int32_t x : xs)
    for (uint32_t R : Rs)
      if (in_range(x, GV_NOWHERE, R)) return true;
  return false;
}
static_assert(!nowhere_passes(), "a shift to nowhere passes nothing");
static_assert(in_range(-5, 5u, 0u) && in_range(-5, 6u, 1u) && !in_range(-5, 4u, (uint32_t)LIM), "lower end");
static_assert(in_range(3, (uint32_t)-3, 0u) && in_range(-2, 9u, 7u) && !in_range(-1, 9u, 7u), "upper end");
