// Host checks of the panel kernel's planning (csrc/host_plan.h), built by
// tests/test_panel_plan.py with the host compiler under AddressSanitizer and
// UndefinedBehaviorSanitizer.  Returns non-zero when a check failed.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <utility>
#include <vector>

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

static uint64_t binomial(uint32_t n, uint32_t k) {
  uint64_t c = 1;
  for (uint32_t i = 1; i <= k; ++i) c = c * (n - k + i) / i;
  return c;
}

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

// Sectors of n orbitals, a alpha and b beta, that one launch gives to the panel
// kernel (1) or leaves to the sector kernel (0), complex64 and complex128: the
// sizes on both sides of every line of panel_pays, 256 compute units.
static void check_panel_pays() {
  struct Case {
    uint32_t n, a, b, jobs;
    int c64, c128;
  };
  const Case cases[] = {
      {4, 2, 2, 1, 1, 1},   {11, 2, 5, 1, 1, 1},  {11, 5, 6, 1, 1, 1},  {12, 2, 3, 1, 1, 1},  {12, 3, 3, 1, 1, 1},
      {13, 3, 3, 1, 0, 1},  {14, 3, 3, 1, 0, 1},  {14, 1, 3, 1, 1, 1},  {12, 1, 4, 1, 0, 0},  {12, 3, 4, 1, 0, 1},
      {12, 4, 4, 1, 0, 0},  {12, 1, 6, 1, 0, 0},  {12, 2, 6, 1, 0, 0},  {12, 3, 6, 1, 0, 1},  {12, 4, 6, 1, 1, 1},
      {12, 6, 6, 1, 1, 1},  {13, 1, 6, 1, 0, 0},  {13, 2, 6, 1, 0, 0},  {13, 3, 5, 1, 0, 1},  {13, 3, 6, 1, 1, 1},
      {13, 4, 4, 1, 1, 1},  {14, 1, 7, 1, 0, 0},  {14, 2, 7, 1, 0, 0},  {14, 3, 4, 1, 0, 1},  {14, 3, 7, 1, 1, 1},
      {14, 7, 7, 1, 1, 1},  {14, 1, 7, 6, 0, 0},  {14, 1, 7, 24, 0, 1}, {14, 2, 7, 6, 0, 1},  {12, 3, 6, 6, 1, 1},
      {12, 4, 4, 8, 0, 1},  {12, 3, 4, 8, 0, 1},  {14, 3, 3, 6, 1, 1},  {12, 2, 3, 12, 1, 1}, {13, 3, 5, 6, 1, 1},
      {12, 4, 3, 1, 0, 0},  {12, 4, 2, 1, 0, 0},  {12, 4, 3, 4, 1, 1},  {11, 6, 7, 1, 0, 1},  {11, 6, 8, 1, 0, 1},
      {11, 6, 9, 1, 1, 0},  {11, 5, 5, 1, 1, 1},  {11, 4, 3, 1, 1, 1},  {11, 6, 7, 2, 1, 1},  {13, 3, 2, 1, 0, 1},
  };
  for (const Case& c : cases) {
    const uint64_t rows = binomial(c.n, c.a), cols = binomial(c.n, c.b);
    const int v = panel_variant_for(rows, cols, c.n * (c.n - 1) / 2, c.a * (c.n - c.a) + 1);
    CHECK(v >= 0, "(%u; %u, %u) has no variant", c.n, c.a, c.b);
    if (v < 0) continue;
    const double fill = panel_fill(v, c.a * (c.n - c.a), c.b * (c.n - c.b));
    CHECK(fill > 0.0 && fill < 1.0, "(%u; %u, %u) fill %g", c.n, c.a, c.b, fill);
    for (uint32_t elem : {8u, 16u}) {
      const int want = elem == 8 ? c.c64 : c.c128;
      CHECK(panel_pays(v, rows * c.jobs, rows, cols, fill, elem, 256) == (want != 0), "%u x (%u; %u, %u), %u bytes: want %d",
            c.jobs, c.n, c.a, c.b, elem, want);
    }
  }
}

// n a b jobs -> variant and rows of a workgroup: of a single launch (jobs 0) or
// of a batch of `jobs` equal jobs, 256 compute units.
static int print_split(char** v) {
  const uint32_t n = std::atoi(v[1]), a = std::atoi(v[2]), b = std::atoi(v[3]), jobs = std::atoi(v[4]);
  const uint32_t rows = static_cast<uint32_t>(binomial(n, a)), cols = static_cast<uint32_t>(binomial(n, b));
  const int variant = panel_variant_for(rows, cols, n * (n - 1) / 2, a * (n - a) + 1);
  if (variant < 0) return 1;
  const uint32_t most = kPanelVariants[variant].rows;
  uint32_t per;
  if (jobs) {
    per = panel_batch_rows(std::vector<std::pair<uint32_t, uint32_t>>(jobs, {rows, cols}), most, 256);
  } else {
    const uint32_t blocks = panel_blocks(rows, most, 256);
    per = (rows + blocks - 1) / blocks;
  }
  const double fill = panel_fill(variant, a * (n - a), b * (n - b));
  const uint64_t all = static_cast<uint64_t>(rows) * (jobs ? jobs : 1);
  std::printf("%d %u %d %d\n", variant, per, panel_pays(variant, all, rows, cols, fill, 8, 256),
              panel_pays(variant, all, rows, cols, fill, 16, 256));
  return 0;
}

// Targets per lane of the full-space kernels on both sides of every line of
// full_tile (256 compute units); tiles are whole wherever they are used.
static void check_full_tile() {
  struct Case {
    uint32_t sites, groups, with_signs, c64, c128;
  };
  const Case cases[] = {{0, 1, 1, 1, 1},     {6, 7, 1, 1, 1},     {16, 17, 1, 1, 1},   {17, 18, 1, 2, 2},
                        {17, 40, 40, 1, 1},  {18, 19, 1, 4, 4},   {18, 16, 4, 4, 4},   {18, 16, 5, 1, 1},
                        {19, 20, 1, 8, 4},   {19, 20, 20, 1, 1},  {20, 500, 500, 8, 4}, {22, 23, 1, 8, 4}};
  for (const Case& c : cases)
    for (uint32_t elem : {8u, 16u}) {
      const uint32_t r = full_tile(1ull << c.sites, c.groups, c.with_signs, elem, 256);
      CHECK(r == (elem == 8 ? c.c64 : c.c128), "%u sites, %u of %u groups with signs, %u bytes: %u", c.sites,
            c.with_signs, c.groups, elem, r);
    }
  for (uint32_t cus : {32u, 64u, 128u, 256u, 304u})
    for (uint32_t sites = 0; sites < 30; ++sites)
      for (uint32_t elem : {8u, 16u}) {
        const uint32_t r = full_tile(1ull << sites, 4, 1, elem, cus);
        CHECK(r == 1 || (1ull << sites) % (kFullLanes * r) == 0, "%u sites, %u units: %u", sites, cus, r);
      }
}

// Lists or rows kernel, on both sides of the line.
static void check_lists_pays() {
  CHECK(lists_pays(true, 64) && lists_pays(true, 16) && lists_pays(false, 60) && !lists_pays(false, 61) &&
            !lists_pays(false, 64),
        "lists kernel's line");
}

int main(int argc, char** argv) {
  if (argc == 5) return print_split(argv);
  check_pull_region();
  check_full_tile();
  check_lists_pays();
  check_panel_pays();
  check_batch_rows();
  if (g_fail) return 1;
  std::printf("all panel plan checks passed\n");
  return 0;
}
