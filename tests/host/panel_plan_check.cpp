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

// Rows per workgroup of a batch: between one and the variant's most; one where
// every row finds a free compute unit, the most where many rounds follow, more
// than one where single rows would take many rounds, and no more than leaves
// whole rounds.
static void check_batch_rows() {
  using Jobs = std::vector<std::pair<uint32_t, uint32_t>>;
  CHECK(panel_batch_rows(Jobs(3, {70, 70}), 4, 256) == 1, "210 rows on 256 units");
  CHECK(panel_batch_rows(Jobs(16, {252, 252}), 4, 256) == 4, "4,032 rows in one round of four");
  CHECK(panel_batch_rows(Jobs(64, {924, 924}), 4, 256) == 4, "59,136 rows");
  CHECK(panel_batch_rows(Jobs(1, {3432, 3432}), 2, 256) == 2, "3,432 long rows, two at most");
  CHECK(panel_batch_rows(Jobs(3, {252, 252}), 4, 256) == 3, "756 rows in one round of three");
  for (uint32_t n = 1; n <= 40; n += 3)
    for (uint32_t most : {2u, 4u}) {
      Jobs jobs;
      for (uint32_t i = 0; i < n; ++i) jobs.push_back({10 + 37 * i % 200, 20 + 53 * i % 400});
      const uint32_t r = panel_batch_rows(jobs, most, 256);
      CHECK(r >= 1 && r <= most, "%u jobs: %u rows of %u", n, r, most);
    }
}

int main() {
  check_pull_region();
  check_batch_rows();
  if (g_fail) return 1;
  std::printf("all panel plan checks passed\n");
  return 0;
}
