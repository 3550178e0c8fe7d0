// Host checks of the panel kernel's planning (csrc/host_plan.h), built by
// tests/test_panel_plan.py with the host compiler under AddressSanitizer and
// UndefinedBehaviorSanitizer.  Returns non-zero when a check failed.
#include <algorithm>
#include <cstdio>

#include "../../paper_2606_28952_amd/csrc/host_plan.h"

using namespace pbs;

static int g_fail = 0;
#define CHECK(cond, ...)                                        \
  do {                                                          \
    if (!(cond)) {                                              \
      std::fprintf(stderr, "FAIL %s:%d: ", __FILE__, __LINE__); \
      std::fprintf(stderr, __VA_ARGS__);                        \
      std::fprintf(stderr, "\n");                               \
      ++g_fail;                                                 \
    }                                                           \
  } while (0)

// A group of n >= 1 slots that ends with slot `end` of a full tile is read
// kPanelPullRead slots at a time from its first one: every read lies in the
// region, which lies in the LDS of a compute unit.
static void check_pull_region() {
  constexpr uint32_t slot = 64u * 2u;  // two-byte entries of 64 lanes
  for (uint32_t end = 1; end <= kPanelPullSlots; ++end)
    for (uint32_t n = 1; n <= end; ++n)
      for (uint32_t i = 0; i < n; i += kPanelPullRead) {
        const uint32_t past = (end - n + i + kPanelPullRead) * slot;
        CHECK(past <= kPanelPullBytes, "slots %u..%u read up to byte %u of %u", end - n, end - 1, past,
              kPanelPullBytes);
        if (past > kPanelPullBytes) return;
      }
  CHECK(kPanelMixBytes + kPanelPullBytes <= 163840u, "panel kernel needs %u bytes of LDS",
        kPanelMixBytes + kPanelPullBytes);
}

int main() {
  check_pull_region();
  if (g_fail) return 1;
  std::printf("all panel plan checks passed\n");
  return 0;
}
