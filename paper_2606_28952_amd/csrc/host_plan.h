// Host-side planning that needs no device: the sector kernel's LDS layout,
// the rank-revealing factorization of a group's sector-form coefficients
// (Section 2.4, Eq. svd_weights) and the work list of a batched launch.
// Plain C++17 with no HIP header, so that the same code also builds with the
// host compiler under AddressSanitizer and UndefinedBehaviorSanitizer.
#pragma once

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <functional>
#include <utility>
#include <vector>

namespace pbs {

// ------------------------------------------------------ sector LDS layout
constexpr int kMaxMoves = 56;         // pair moves cached per lane (N_beta (n_orb - N_beta) <= 56)
constexpr uint32_t kListSlotsAhead = 6;  // lists kernel: slots of column entries in flight
constexpr uint32_t kListRowsAhead = 20;  // and gathers of the simple classes at most
constexpr uint32_t kRowCapBytes = 64u * 1024u;
constexpr uint32_t kListMinBytes = 4096u;  // simple-class row list when no row is staged
// LDS copy of the uint16 rank tables (n_orb <= 16): chunk 0 with no ones
// below it, then chunk 1 for 0..8 ones below it (zeros when n_orb <= 8)
constexpr uint32_t kRank16Lds = 10u * 256u;
// Fixed LDS placement (the kernel declares no static LDS, so these are
// absolute addresses): workgroup scratch at byte 0, the pair map at kPuOff
// (an 8-byte slot per orbital pair, at most C(32, 2) + 1 entries) and the
// staged row at kRowOff, so per-move addresses need no base register.
constexpr uint32_t kMiscBytes = 256;  // ballot counts and the energy reduction
constexpr uint32_t kPuOff = kMiscBytes;
constexpr uint32_t kPuBytes = 4096;
constexpr uint32_t kRowOff = kPuOff + kPuBytes;
constexpr uint32_t kZeroSlots = 4;     // zero entries after the folded uniques (absent groups, padding)
constexpr uint32_t kFCapMin = 1024;    // folded uniques: smallest LDS capacity planned for
constexpr uint32_t kFCapMax = 4096;    // and the largest (offsets are packed in 16 bits)
constexpr uint32_t kMaxR1 = 32;        // largest factored rank of an X_beta = 0 group
constexpr uint32_t kFactZeroSlots = 4;  // zero factors at the start of the class-0 fold

// Panel kernel (panel.h): lanes per workgroup, most beta columns (seven
// target columns per lane), columns per V tile, most classes per row (13 K
// steps of four, the X_alpha = 0 class among them) and orbital pairs (six
// 16-row tiles), and the V tile's zero entry.
constexpr uint32_t kPanelLanes = 512;
constexpr uint32_t kPanelCols = 7 * kPanelLanes;
constexpr uint32_t kPanelTile = 64;
constexpr uint32_t kPanelClasses = 52;
constexpr uint32_t kPanelPairs = 96;
constexpr uint32_t kPanelZero = kPanelPairs * kPanelTile;
constexpr uint32_t kPanelPullSlots = 128;  // gather entries of a V tile: slots of 64 lanes
constexpr uint32_t kPanelVBytes = (kPanelZero + 1u) * 16u;
// LDS: the V tile, the image matrix and the classes' records; before them the
// staged rows, then the list coefficients and sources, in the same place
constexpr uint32_t kPanelMixBytes = kPanelVBytes + kPanelPairs * kPanelClasses * 8u + kPanelClasses * 32u;
// after the classes' records; slots are read kPanelPullRead at a time, past the last one too
constexpr uint32_t kPanelPullRead = 4;
constexpr uint32_t kPanelPullBytes = (kPanelPullSlots + kPanelPullRead - 1u) * 128u;

// The panel kernel's variants: beta columns (512 per target column of a
// lane), orbital pairs (32 per 16-pair tile of a wave), classes per row (four
// per K step, the X_alpha = 0 class included) and target rows per workgroup
// that each one is built for.  Fixed counts keep the products free of
// branches, so a row's loads stay in flight across them; the narrow ones
// save the padding (at 11 orbitals 8 K steps instead of 13).  Two rows with
// seven columns per lane: four need 112 registers for the sums alone and
// spill (28 qubits, complex64: 14.9 ms against 11.6).
struct PanelVariant {
  uint32_t cols, pairs, classes, rows;
};
constexpr PanelVariant kPanelVariants[] = {{512, 64, 32, 4},   {512, 96, 52, 4},  {1024, 96, 40, 4}, {1024, 96, 52, 4},
                                           {2048, 96, 44, 4}, {2048, 96, 52, 4}, {3584, 96, 52, 2}};
constexpr int kPanelWide = 4;  // first variant for more than 1,024 columns

// The first variant that holds the sector, or -1.  Sectors of at most 512
// beta and more than 512 alpha strings are left to the sector kernel: a row
// is then too short to fill a workgroup's lanes and matrix tiles, while its
// image matrix loads in full (7 of 14 alpha and 3 beta orbitals, complex64:
// 1.98 ms against 1.64; 462 strings each: 0.148 ms against 0.152).
inline int panel_variant_for(uint64_t rows, uint64_t cols, uint32_t pairs, uint32_t classes) {
  if (rows > kPanelCols || (cols <= kPanelLanes && rows > kPanelLanes)) return -1;
  int v = 0;
  for (const PanelVariant& p : kPanelVariants) {
    if (cols <= p.cols && pairs <= p.pairs && classes <= p.classes) return v;
    ++v;
  }
  return -1;
}

// Share of a variant's padded products (classes x pairs) that a target row's
// image classes and a target's single beta moves use.
inline double panel_fill(int variant, uint32_t alpha_hops, uint32_t beta_hops) {
  const PanelVariant& p = kPanelVariants[variant];
  return static_cast<double>(alpha_hops) * beta_hops / (static_cast<double>(p.classes) * p.pairs);
}

// Whether the panel kernel is the faster one for a sector of `cols` beta strings
// in a launch of `rows` rows, all jobs of the variant together; elem: bytes of an
// amplitude.  It takes one workgroup per row, or a few rows, and pays for the
// padding of its products; the sector kernel takes 512 columns per workgroup, so
// it fills the device with fewer rows, and its work follows the moves that exist.
// Sector kernel against panel kernel, one launch, us:
//  * narrow rows, one per workgroup, are short either way: (12; 3, 3) complex64
//    87 against 77, (11; 2, 5) 75 against 66.  A second row for some workgroups
//    doubles the panel kernel's time: (14; 3, 3), 364 rows, complex64 175 / 180,
//    complex128 211 / 189.  495 columns of 12 orbitals: (12; 3, 4) complex64
//    101 / 111, complex128 118 / 116; (12; 4, 4), two rows, 167 / 210 and 216 / 220, and
//    eight jobs of it 1,329 / 1,475 and 1,846 / 1,544
//  * long rows, fewer than compute units: (14; 1, 7) complex64 117 / 600, (14; 2, 7)
//    complex64 355 / 642, complex128 472 / 648; (12; 3, 6), 220 rows, complex64
//    166 / 181, complex128 214 / 171
//  * and more of them: (13; 3, 5), fill 0.28, complex64 390 / 424, (13; 3, 6), 0.30,
//    518 / 506, (14; 3, 4), 1,001 columns, 330 / 349; with 495 and more rows at 0.29
//    to 0.38 1.03 to 1.8 times as fast ((13; 5, 4) alone 0.99); 24 jobs of (14; 1, 7),
//    0.13, 1,027 / 1,190, six of (14; 2, 7), 0.24, 1,749 / 2,048, six of (12; 3, 6),
//    0.25, 894 / 849; complex128 faster throughout (gathers of 16 bytes)
//  * one sector of up to 512 columns whose rows need a second row in most
//    workgroups: (12; 4, 3) complex64 140 / 156, complex128 158 / 164, (12; 4, 2) 112 / 123
//    and 112 / 131; (11; 6, 7) 137 / 143 and 165 / 152, (11; 6, 8) 120 / 121 and 129 / 129,
//    (11; 6, 9) 103 / 101 and 104 / 110, (11; 5, 5) 153 / 153 and 198 / 160
// job_rows: the sector's own rows.
inline bool panel_pays(int variant, uint64_t rows, uint64_t job_rows, uint64_t cols, double fill, uint32_t elem,
                       uint32_t cus) {
  if (rows == job_rows && cols <= kPanelLanes && 2 * rows >= 3ull * cus) {
    if (variant != 0) return false;
    return elem > 8 ? cols >= 128 : cols >= rows || cols <= 64;
  }
  if (variant == 0) return true;
  const bool narrow = cols <= 400;
  if (elem > 8)
    return narrow || (4 * rows >= 3ull * cus && (cols > kPanelLanes || rows <= cus || rows >= 4ull * cus));
  const bool many = 2 * rows >= 3ull * cus;
  if (cols <= kPanelLanes) return narrow && (many || rows <= cus);
  if (many) return fill >= 0.25;
  return rows > cus && cols > 2 * kPanelLanes && fill >= 0.29;
}

// Row blocks that split dim_alpha rows evenly into at most `rows` each:
// as few as that allows, rounded up to whole rounds of one workgroup per
// compute unit (one row each when there are fewer rows than units).
inline uint32_t panel_blocks(uint32_t dim_alpha, uint32_t rows, uint32_t cus) {
  if (dim_alpha <= cus) return dim_alpha;
  const uint32_t least = (dim_alpha + rows - 1u) / rows;
  return std::min(dim_alpha, (least + cus - 1u) / cus * cus);
}

// Workgroups per row of a launch of few rows of `groups` times 512 columns: one
// per group, or per two groups, while all of them fit on the device at once.
inline uint32_t panel_parts(uint64_t rows, uint32_t groups, uint32_t cus) {
  for (uint32_t per : {1u, 2u}) {
    const uint32_t parts = (groups + per - 1u) / per;
    if (rows * parts <= cus) return parts;
  }
  return 1;
}

// Target rows per workgroup (at most `most`) of a launch that takes whole jobs
// of rows x cols configurations: the number whose workgroups, dealt to the
// compute units one at a time as these get free (longest first), end first.
// r rows of a workgroup share tables and take about 0.4 + 0.6 r of one row's time
// (28 qubits: 0.82, 1.34 ms; 12 orbitals: 0.23, 0.36, 0.63 for one, two, four
// rows), and a row's time grows with its columns.  Sixteen complex64 jobs of 10
// orbitals (4,032 rows): 0.93 ms with one row each, 0.65 with four; ten uneven
// jobs of 6 to 9 orbitals (about 560 rows): 0.075 ms with one, 0.087 with three.
inline uint32_t panel_batch_rows(std::vector<std::pair<uint32_t, uint32_t>> jobs, uint32_t most, uint32_t cus) {
  uint64_t rows = 0;
  for (const auto& j : jobs) rows += j.first;
  if (rows >= 16ull * most * cus) return most;  // many rounds: the last one does not matter
  std::sort(jobs.begin(), jobs.end(), [](const auto& a, const auto& b) { return a.second > b.second; });
  uint32_t best = 1;
  double best_time = 0.0;
  for (uint32_t r = 1; r <= most; ++r) {
    std::vector<double> busy(cus, 0.0);  // a heap, the first free unit on top
    double end = 0.0;
    for (const auto& j : jobs) {
      const uint32_t blocks = (j.first + r - 1u) / r;
      for (uint64_t b = 0; b < blocks; ++b) {
        const uint64_t n = (b + 1) * j.first / blocks - b * j.first / blocks;
        std::pop_heap(busy.begin(), busy.end(), std::greater<double>());
        busy.back() += (20.0 + j.second) * (0.4 + 0.6 * static_cast<double>(n));
        end = std::max(end, busy.back());
        std::push_heap(busy.begin(), busy.end(), std::greater<double>());
      }
    }
    if (r == 1 || end < best_time) {
      best = r;
      best_time = end;
    }
  }
  return best;
}

// Whether the lists kernel is the faster one for rows too long for the sector
// kernel's staging (shorter rows were not compared): its gathers of other rows
// beyond the first kListRowsAhead wait one by one, which shows when the rows have
// many and the columns' entries look up their magnitudes.  Rows kernel against
// lists kernel, 16 orbitals, complex64, hops between all pairs: 60 gathers a row,
// 120 magnitudes 13.5 / 13.0 ms, 64 gathers 21.5 / 22.1; one magnitude, 64
// gathers, 19.1 / 15.5.
inline bool lists_pays(bool one_magnitude, uint32_t longest_list) { return one_magnitude || longest_list <= 60; }

// Targets per lane of the full-space kernel: as many as leave a workgroup of 256
// lanes per compute unit; eight of 16 bytes cost too many registers (102 us at 22
// sites, 83 with four).  1: the kernel without tiles.  Tiles share a group's loads
// among targets, but one workgroup per unit waits for each of them in turn, and a
// group with signs takes twice as long there as a run of groups without: so few
// lanes take tiles only for operators that are mostly such runs.  Without and
// with tiles, us: 18 sites complex64, Ising chain (1 of 19 groups signed) 10.6 / 9.6,
// 40 random strings 17.9 / 25.3, 2,000 659 / 1,094; 17 sites, chain, complex128 9.2 /
// 8.3; 20 sites, 500 random strings 500 / 500 and 562 / 465, 10 orbitals 6,360 /
// 4,470; one target per lane in tiles: 14 sites, 300 random strings 71 / 104, 6
// orbitals 197 / 209, chains of up to 16 sites equal.
constexpr uint32_t kFullLanes = 256;
inline uint32_t full_tile(uint64_t dim, uint64_t groups, uint64_t with_signs, uint32_t elem, uint32_t cus) {
  const uint64_t lanes = dim / kFullLanes;
  if (lanes < 2ull * cus || (lanes < 16ull * cus && 4 * with_signs > groups)) return 1;
  if (elem == 8 && lanes >= 8ull * cus) return 8;
  return lanes >= 4ull * cus ? 4 : 2;
}

inline uint32_t align16(uint32_t v) { return (v + 15u) & ~15u; }

// What the layout depends on: the device's LDS per workgroup (less the
// static arrays), the sector, the amplitude size and the operator's table
// sizes.
struct SectorLayoutIn {
  uint32_t lds_limit = 0;
  uint32_t n_orb = 0, n_beta = 0;
  uint64_t dim_beta = 0;
  uint32_t elem_bytes = 8;
  bool realc = true;      // real coefficients (8-byte folded uniques)
  bool allow_row = true;  // a source row may be staged whole
  bool allow_enum = true, allow_qenum = true;
  uint64_t n_pmap = 0, n_qmap = 0;  // pair and quad map entries (0: no map)
  uint32_t n_pairs = 0, n_quads = 0, max_quad_uniques = 0;
  bool a_region = false;  // folded factors of an X_beta = 0 group need a place
};

// Byte offsets of every region and the choices that decide them.  Regions:
// [0, kMiscBytes) scratch, [kPuOff, kPuOff + kPuBytes) pair map (the X_beta
// = 0 factors at off_a inside it when they fit), [kRowOff, kRowOff +
// row_region) staged row or row list, then rank tables, folded uniques,
// their Z-masks, the quad map and, when not in the pair map, the X_beta = 0
// factors; lds is the end of the last region.
struct SectorLayout {
  bool r16 = false, enum_ok = false, qenum_ok = false, row_lds = false;
  uint32_t n_moves = 0, n_qmoves = 0, list_cap = 0, f_cap = 0;
  uint32_t row_region = 0, rank_bytes = 0, off_rank = 0, off_f = 0, f_bytes = 0, off_fz = 0, fz_bytes = 0;
  uint32_t off_qu = 0, qu_bytes = 0, off_a = 0, a_bytes = 0, lds = 0;
  bool a_in_pair_map = false;
};

// Returns false when the operator's orbital pairs do not fit the pair map.
// The folded uniques get what is left of half the LDS, so that two
// workgroups share a compute unit, unless the fixed parts alone need more.
inline bool sector_layout(const SectorLayoutIn& in, SectorLayout* out) {
  SectorLayout L;
  if (in.n_pairs + 1u > kPuBytes / 8u) return false;
  const uint32_t limit = in.lds_limit;
  const uint32_t half = limit / 2u - 512u;
  L.r16 = in.n_orb <= 16;
  L.rank_bytes = L.r16 ? align16(kRank16Lds * 2u) : 0u;
  const uint32_t per_unique = (in.realc ? 8u : 16u) + 4u;
  const uint32_t f_min = (kFCapMin + kZeroSlots) * per_unique + 64u;
  L.n_moves = in.n_beta * (in.n_orb - in.n_beta);
  L.enum_ok = in.allow_enum && in.n_pmap > 0 && L.n_moves <= static_cast<uint32_t>(kMaxMoves) &&
              in.dim_beta < 65536 && in.n_pairs < 65536;
  const uint32_t pu_bytes = kMiscBytes + kPuBytes;
  auto pairs = [](uint64_t m) { return m < 2 ? uint64_t{0} : m * (m - 1) / 2; };
  const uint64_t n_ep = pairs(in.n_orb - in.n_beta), n_op = pairs(in.n_beta);
  L.qenum_ok = in.allow_qenum && L.r16 && L.enum_ok && in.n_qmap > 0 && in.n_quads > 0 && n_op * n_ep > 0;
  L.n_qmoves = static_cast<uint32_t>(n_op * n_ep);
  const uint64_t row_bytes = in.dim_beta * in.elem_bytes;
  const uint64_t row_space = row_bytes > kListMinBytes ? row_bytes : kListMinBytes;
  L.row_lds = in.allow_row && row_bytes <= kRowCapBytes && L.rank_bytes + f_min + pu_bytes + row_space <= limit;
  L.row_region = align16(static_cast<uint32_t>(L.row_lds ? row_space : kListMinBytes));
  L.list_cap = L.row_region / 8u;
  // The double-move phase needs its quad map and every quad unique of a
  // class in LDS at once; it is kept only if that still lets two workgroups
  // share a compute unit (or if two never fit anyway).
  const uint32_t base_fixed = L.rank_bytes + L.row_region + pu_bytes;
  const uint32_t qu_need = align16(in.n_quads * 4u);
  const uint32_t q_need = (in.max_quad_uniques + kZeroSlots) * per_unique + 64u;
  if (L.qenum_ok) {
    const bool two_without = base_fixed + f_min <= half;
    const uint32_t cap = two_without ? half : limit;
    if (base_fixed + qu_need + std::max(q_need, f_min) > cap || in.max_quad_uniques >= kFCapMax) L.qenum_ok = false;
  }
  L.qu_bytes = L.qenum_ok ? qu_need : 0u;
  // the folded factors of an X_beta = 0 group sit after the pair map when
  // its fixed region has room (n_orb <= 16), else in a region of their own
  const uint32_t a_in_pu = align16((in.n_pairs + 1u) * 8u);
  L.a_in_pair_map = a_in_pu + kMaxR1 * 8u <= kPuBytes;
  L.a_bytes = (in.a_region && !L.a_in_pair_map) ? align16(kMaxR1 * 8u) : 0u;
  const uint32_t fixed = base_fixed + L.qu_bytes + L.a_bytes;
  const uint32_t budget = fixed + f_min <= half ? half : limit;
  L.f_cap = std::min(kFCapMax, (budget - fixed - 64u) / per_unique - kZeroSlots);
  uint32_t off = kRowOff + L.row_region;
  L.off_rank = off;
  off += L.rank_bytes;
  L.off_f = off;
  L.f_bytes = align16((L.f_cap + kZeroSlots) * (per_unique - 4u));
  off += L.f_bytes;
  L.off_fz = off;
  L.fz_bytes = align16((L.f_cap + kZeroSlots) * 4u);
  off += L.fz_bytes;
  L.off_qu = off;
  off += L.qu_bytes;
  L.off_a = L.a_in_pair_map ? kPuOff + a_in_pu : off;
  off += L.a_bytes;
  L.lds = off;
  *out = L;
  return true;
}

// ------------------------------------------- spin-factorized coefficients
// M = P Q by pivoted Gram-Schmidt on the rows of M (rows x cols, row-major):
// the next basis vector is the remaining row of largest norm, orthogonalised
// twice against the basis; stops when every remaining row is below
// rtol * (largest row norm of M).  Q (rank x cols, orthonormal rows) is
// returned through the argument, the rank as the result.
inline uint32_t factor_rows(const std::vector<double>& M, uint32_t rows, uint32_t cols, double rtol,
                            std::vector<double>& Q) {
  std::vector<double> res = M;
  Q.clear();
  double scale = 0.0;
  for (uint32_t i = 0; i < rows; ++i) {
    double s = 0.0;
    for (uint32_t j = 0; j < cols; ++j) s += M[static_cast<size_t>(i) * cols + j] * M[static_cast<size_t>(i) * cols + j];
    scale = std::max(scale, std::sqrt(s));
  }
  if (scale == 0.0) return 0;
  uint32_t r = 0;
  std::vector<double> q(cols);
  while (r < rows && r < cols) {
    uint32_t best = 0;
    double bn = -1.0;
    for (uint32_t i = 0; i < rows; ++i) {
      double s = 0.0;
      for (uint32_t j = 0; j < cols; ++j)
        s += res[static_cast<size_t>(i) * cols + j] * res[static_cast<size_t>(i) * cols + j];
      if (s > bn) {
        bn = s;
        best = i;
      }
    }
    if (std::sqrt(bn) <= rtol * scale) break;
    for (uint32_t j = 0; j < cols; ++j) q[j] = res[static_cast<size_t>(best) * cols + j];
    for (int pass = 0; pass < 2; ++pass) {
      for (uint32_t k = 0; k < r; ++k) {
        double d = 0.0;
        for (uint32_t j = 0; j < cols; ++j) d += q[j] * Q[static_cast<size_t>(k) * cols + j];
        for (uint32_t j = 0; j < cols; ++j) q[j] -= d * Q[static_cast<size_t>(k) * cols + j];
      }
      double nn = 0.0;
      for (uint32_t j = 0; j < cols; ++j) nn += q[j] * q[j];
      nn = std::sqrt(nn);
      for (uint32_t j = 0; j < cols; ++j) q[j] /= nn;
    }
    Q.insert(Q.end(), q.begin(), q.end());
    ++r;
    for (uint32_t i = 0; i < rows; ++i) {
      double d = 0.0;
      for (uint32_t j = 0; j < cols; ++j) d += res[static_cast<size_t>(i) * cols + j] * q[j];
      for (uint32_t j = 0; j < cols; ++j) res[static_cast<size_t>(i) * cols + j] -= d * q[j];
    }
  }
  return r;
}

// The sector-form tables of the groups on the host: group g's uniques are
// [pg_u0[g], pg_u0[g + 1]); unique u has beta Z-mask u_zb[u] and terms
// [u_t0[u], u_t0[u + 1]) with alpha Z-masks pt_za and real coefficients pt_c.
struct HostTables {
  std::vector<uint32_t> pg_u0, u_zb, u_t0, pt_za, pg_xb;
  std::vector<double> pt_c;
};

// One group's factors: for each r, the alpha terms (Za, P[mu][r]) and the
// beta list (Zb, Q[r][nu]); exact zeros are left out.
struct GroupFactors {
  uint32_t rank = 0;
  uint32_t n_uniques = 0;
  std::vector<std::vector<std::pair<uint32_t, double>>> a, b;
};

inline GroupFactors factor_group(const HostTables& T, uint32_t g, double rtol = 1e-14) {
  GroupFactors F;
  const uint32_t u0 = T.pg_u0[g], u1 = T.pg_u0[g + 1];
  F.n_uniques = u1 - u0;
  // rows: the distinct alpha Z-masks, ascending
  std::vector<uint32_t> za(T.pt_za.begin() + T.u_t0[u0], T.pt_za.begin() + T.u_t0[u1]);
  std::sort(za.begin(), za.end());
  za.erase(std::unique(za.begin(), za.end()), za.end());
  auto row_of = [&](uint32_t z) {
    return static_cast<uint32_t>(std::lower_bound(za.begin(), za.end(), z) - za.begin());
  };
  const uint32_t nr = static_cast<uint32_t>(za.size()), nc = u1 - u0;
  std::vector<double> M(static_cast<size_t>(nr) * nc, 0.0);
  for (uint32_t u = u0; u < u1; ++u)
    // terms whose beta Z-masks differ by X_beta share one unique in sector
    // form and may share an alpha Z-mask too: their coefficients add
    for (uint32_t t = T.u_t0[u]; t < T.u_t0[u + 1]; ++t)
      M[static_cast<size_t>(row_of(T.pt_za[t])) * nc + (u - u0)] += T.pt_c[t];
  std::vector<double> Q;
  F.rank = factor_rows(M, nr, nc, rtol, Q);
  F.a.resize(F.rank);
  F.b.resize(F.rank);
  for (uint32_t r = 0; r < F.rank; ++r) {
    for (uint32_t mu = 0; mu < nr; ++mu) {
      double p = 0.0;
      for (uint32_t nu = 0; nu < nc; ++nu) p += M[static_cast<size_t>(mu) * nc + nu] * Q[static_cast<size_t>(r) * nc + nu];
      if (p != 0.0) F.a[r].emplace_back(za[mu], p);
    }
    for (uint32_t nu = 0; nu < nc; ++nu)
      if (Q[static_cast<size_t>(r) * nc + nu] != 0.0) F.b[r].emplace_back(T.u_zb[u0 + nu], Q[static_cast<size_t>(r) * nc + nu]);
  }
  return F;
}

// ------------------------------------------------- batched launch work list
// Jobs in launch order (largest cost first, ties in the caller's order,
// unless the caller fixed the order) and each job's first work item in that
// order; total = all items.
struct BatchPlan {
  std::vector<uint32_t> order;
  std::vector<uint64_t> base;  // indexed by launch position
  uint64_t total = 0;
};

inline BatchPlan batch_plan(const std::vector<double>& cost, const std::vector<uint64_t>& items, bool keep_order) {
  BatchPlan B;
  const size_t n = cost.size();
  B.order.resize(n);
  for (size_t i = 0; i < n; ++i) B.order[i] = static_cast<uint32_t>(i);
  if (!keep_order)
    std::stable_sort(B.order.begin(), B.order.end(), [&](uint32_t a, uint32_t b) { return cost[a] > cost[b]; });
  B.base.resize(n);
  uint64_t base = 0;
  for (size_t k = 0; k < n; ++k) {
    B.base[k] = base;
    base += items[B.order[k]];
  }
  B.total = base;
  return B;
}

}  // namespace pbs
