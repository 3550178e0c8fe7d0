// Spin-factorized phase evaluation (Section 2.4: Eqs. svd_weights,
// precomp_alpha, precomp_beta, svd_sreverse_sum and dot_product; Algorithm
// grouped_hvec; the rank distribution of Table svd_rank_dist).
//
// In a spin sector every group's phase sum separates into alpha and beta
// parities: with its sector-form coefficients arranged as a matrix
// M[mu][nu] (rows: the group's distinct alpha Z-masks, columns: its uniques,
// i.e. distinct beta Z-masks),
//   sum_k C_k (-1)^popcount(Z_k & t) = sum_{mu,nu} M[mu][nu] a_mu(t_a) b_nu(t_b),
// a_mu = (-1)^popcount(Za_mu & t_a), b_nu = (-1)^popcount(Zb_nu & t_b).  A
// rank-R factorization M = P Q turns this into sum_r A_r(t_a) F_r(t_b).  The
// sector kernel folds the A_r once per workgroup (all its lanes share t_a);
// this file factors the groups on the host and precomputes F_r for every
// beta string of a sector on the device, laid out per target move so that
// the kernel's loads are coalesced.  The paper computes the factors by an
// SVD; here a rank-revealing Gram-Schmidt factorization (Q with orthonormal
// rows, P = M Q^T, columns chosen by largest remaining norm) gives the same
// exact ranks on these matrices with the same rounding-level residual.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <map>
#include <mutex>
#include <vector>

#include "handles.h"
#include "staging.h"

namespace pbs {
namespace {

// colexicographic rank of a spin string among the n-bit words of its
// popcount (ascending integer order): sum_i C(pos_i, i + 1)
__device__ inline uint32_t colex_rank(uint32_t s) {
  uint32_t r = 0, i = 1;
  while (s) {
    const uint32_t b = __ffs(s) - 1;
    s &= s - 1;
    uint32_t c = 1;  // C(b, i)
    for (uint32_t k = 1; k <= i; ++k) c = c * (b - i + k) / k;
    r += b >= i ? c : 0u;
    ++i;
  }
  return r;
}

// k-th set bit (k from 0) of w
__device__ inline uint32_t kth_bit(uint32_t w, uint32_t k) {
  for (uint32_t i = 0; i < k; ++i) w &= w - 1;
  return __ffs(w) - 1;
}

// i-th pair (a < b) of n items in the order (0,1), (0,2), ..., (1,2), ...
__device__ inline void pair_at(uint32_t i, uint32_t n, uint32_t& a, uint32_t& b) {
  a = 0;
  while (i >= n - 1 - a) {
    i -= n - 1 - a;
    ++a;
  }
  b = a + 1 + i;
}

__device__ inline double eval_rows(const uint32_t* q_zb, const double* q_c, uint32_t lo, uint32_t hi, uint32_t tb) {
  double f = 0.0;
  for (uint32_t k = lo; k < hi; ++k) f += (__popc(q_zb[k] & tb) & 1u) ? -q_c[k] : q_c[k];
  return f;
}

// F rows of the X_beta = 0 groups: f[i * db + j] = sum over row i's list.
__global__ void k_fact_rows(uint32_t n_rows, uint64_t db, const uint32_t* str_b, const uint32_t* q_lo,
                            const uint32_t* q_zb, const double* q_c, double* f) {
  const uint64_t n = static_cast<uint64_t>(n_rows) * db;
  for (uint64_t i = blockIdx.x * static_cast<uint64_t>(blockDim.x) + threadIdx.x; i < n;
       i += static_cast<uint64_t>(gridDim.x) * blockDim.x) {
    const uint32_t row = static_cast<uint32_t>(i / db);
    f[i] = eval_rows(q_zb, q_c, q_lo[row], q_lo[row + 1], str_b[i % db]);
  }
}

// Single moves (occupied p -> empty q, p outer, both ascending):
// em[m * db + j] = source column | (factor slot << 16), fp[(m * r2 + r) * db + j].
__global__ void k_fact_moves(uint64_t db, uint32_t n_orb, uint32_t n_beta, uint32_t r2, const uint32_t* str_b,
                             const int32_t* pk, const uint32_t* q_lo, const uint32_t* q_zb, const double* q_c,
                             uint32_t* em, double* fp) {
  const uint32_t ne = n_orb - n_beta, n_moves = n_beta * ne;
  const uint32_t full = (n_orb == 32) ? 0xffffffffu : ((1u << n_orb) - 1u);
  const uint64_t n = static_cast<uint64_t>(n_moves) * db;
  for (uint64_t i = blockIdx.x * static_cast<uint64_t>(blockDim.x) + threadIdx.x; i < n;
       i += static_cast<uint64_t>(gridDim.x) * blockDim.x) {
    const uint32_t m = static_cast<uint32_t>(i / db);
    const uint64_t j = i % db;
    const uint32_t tb = str_b[j];
    const uint32_t p = kth_bit(tb, m / ne), q = kth_bit(~tb & full, m % ne);
    const uint32_t lo = p < q ? p : q, hi = p < q ? q : p;
    const int32_t k = pk[hi * (hi - 1) / 2 + lo];
    em[static_cast<uint64_t>(m) * db + j] =
        colex_rank(tb ^ (1u << p) ^ (1u << q)) | ((k >= 0 ? kFactZeroSlots + static_cast<uint32_t>(k) * r2 : 0u) << 16);
    for (uint32_t r = 0; r < r2; ++r) {
      const uint32_t row = static_cast<uint32_t>(k) * r2 + r;
      fp[(static_cast<uint64_t>(m) * r2 + r) * db + j] = k >= 0 ? eval_rows(q_zb, q_c, q_lo[row], q_lo[row + 1], tb)
                                                                : 0.0;
    }
  }
}

// Double moves: occupied pair (a < b) outer, empty pair (c < d) inner, each
// in the order of pair_at over the target's occupied / empty orbitals.
// eq[qm * db + j] = source column | (factor slot << 16); fq[(qm * r3 + r) * db + j].
__global__ void k_fact_quads(uint64_t db, uint32_t n_orb, uint32_t n_beta, uint32_t r3, uint32_t slot0,
                             const uint32_t* str_b, const int32_t* qk, const uint32_t* q_lo, const uint32_t* q_zb,
                             const double* q_c, uint32_t* eq, double* fq) {
  const uint32_t ne = n_orb - n_beta;
  const uint32_t n_op = n_beta * (n_beta - 1) / 2, n_ep = ne * (ne - 1) / 2, n_q = n_op * n_ep;
  const uint32_t full = (n_orb == 32) ? 0xffffffffu : ((1u << n_orb) - 1u);
  const uint64_t n = static_cast<uint64_t>(n_q) * db;
  for (uint64_t i = blockIdx.x * static_cast<uint64_t>(blockDim.x) + threadIdx.x; i < n;
       i += static_cast<uint64_t>(gridDim.x) * blockDim.x) {
    const uint32_t qm = static_cast<uint32_t>(i / db);
    const uint64_t j = i % db;
    const uint32_t tb = str_b[j], emp = ~tb & full;
    uint32_t a, b, c, d;
    pair_at(qm / n_ep, n_beta, a, b);
    pair_at(qm % n_ep, ne, c, d);
    const uint32_t X = (1u << kth_bit(tb, a)) | (1u << kth_bit(tb, b)) | (1u << kth_bit(emp, c)) |
                       (1u << kth_bit(emp, d));
    const int32_t k = qk[colex_rank(X)];
    eq[static_cast<uint64_t>(qm) * db + j] =
        colex_rank(tb ^ X) | ((k >= 0 ? slot0 + static_cast<uint32_t>(k) * r3 : 0u) << 16);
    for (uint32_t r = 0; r < r3; ++r) {
      const uint32_t row = static_cast<uint32_t>(k) * r3 + r;
      fq[(static_cast<uint64_t>(qm) * r3 + r) * db + j] = k >= 0 ? eval_rows(q_zb, q_c, q_lo[row], q_lo[row + 1], tb)
                                                                 : 0.0;
    }
  }
}

// Position of this thread's flag among the workgroup's set flags (in thread
// order) and their total; 256 threads.
__device__ inline void block_compact(bool flag, uint32_t* s_cnt, uint32_t& pos, uint32_t& total) {
  const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
  const uint64_t bal = __ballot(flag);
  if (lane == 0) s_cnt[wave] = static_cast<uint32_t>(__popcll(bal));
  __syncthreads();
  pos = static_cast<uint32_t>(__popcll(bal & ((1ull << lane) - 1ull)));
  total = 0;
  for (uint32_t w = 0; w < 4; ++w) {
    pos += w < wave ? s_cnt[w] : 0u;
    total += s_cnt[w];
  }
  __syncthreads();
}

// Alpha lists (Eq. precomp_alpha for the simple classes): one workgroup per
// alpha row, its threads over the simple classes in class order; pass 0
// counts the classes whose source row lies in the sector, pass 1 writes
// their source rank and folded coefficient sum_t c_t (-1)^popcount(za_t & t_alpha)
// in class order.
__global__ __launch_bounds__(256) void k_alpha_list(uint32_t pass, uint64_t da, uint32_t n_alpha,
                                                    const uint32_t* str_a, const uint32_t* simple, uint32_t n_simple,
                                                    const ClassMeta* meta, const uint32_t* u_t0,
                                                    const uint32_t* pt_za, const double* pt_c, const uint32_t* off,
                                                    uint32_t* count, uint32_t* src, double* coef) {
  __shared__ uint32_t s_cnt[4];
  for (uint64_t i = blockIdx.x; i < da; i += gridDim.x) {
    const uint32_t ta = str_a[i];
    uint32_t n = pass ? off[i] : 0u;
    for (uint32_t k0 = 0; k0 < n_simple; k0 += 256) {
      const uint32_t k = k0 + threadIdx.x;
      const ClassMeta* m = k < n_simple ? meta + simple[k] : nullptr;
      const uint32_t sa = m ? ta ^ m->xa : 0u;
      const bool v = m && static_cast<uint32_t>(__popc(sa)) == n_alpha;
      uint32_t pos, total;
      block_compact(v, s_cnt, pos, total);
      if (pass && v) {
        double f = 0.0;
        for (uint32_t t = u_t0[m->ua]; t < u_t0[m->u_end]; ++t)
          f += (__popc(pt_za[t] & ta) & 1u) ? -pt_c[2 * t] : pt_c[2 * t];
        src[n + pos] = colex_rank(sa);
        coef[n + pos] = f;
      }
      n += total;
    }
    if (!pass && threadIdx.x == 0) count[i] = n;
  }
}

// Image-class lists: one workgroup per alpha row; pass 0 counts the image
// classes whose source row lies in the sector, pass 1 writes (source rank,
// class, row) in class order.
__global__ __launch_bounds__(256) void k_pair_list(uint32_t pass, uint64_t da, uint32_t n_alpha,
                                                   const uint32_t* str_a, const uint32_t* cls, uint32_t n_cls,
                                                   const ClassMeta* meta, const uint32_t* off, uint32_t* count,
                                                   uint32_t* src, uint32_t* ent_cls, uint32_t* ent_row) {
  __shared__ uint32_t s_cnt[4];
  for (uint64_t i = blockIdx.x; i < da; i += gridDim.x) {
    const uint32_t ta = str_a[i];
    uint32_t n = pass ? off[i] : 0u;
    for (uint32_t k0 = 0; k0 < n_cls; k0 += 256) {
      const uint32_t k = k0 + threadIdx.x;
      const uint32_t sa = k < n_cls ? ta ^ meta[cls[k]].xa : 0u;
      const bool v = k < n_cls && static_cast<uint32_t>(__popc(sa)) == n_alpha;
      uint32_t pos, total;
      block_compact(v, s_cnt, pos, total);
      if (pass && v) {
        src[n + pos] = colex_rank(sa);
        ent_cls[n + pos] = cls[k];
        ent_row[n + pos] = static_cast<uint32_t>(i);
      }
      n += total;
    }
    if (!pass && threadIdx.x == 0) count[i] = n;
  }
}

// Images: one workgroup per entry (an alpha row and one of its image
// classes), one thread per slot j < n_img: the folded coefficient of the
// class's pair group on orbital pair j, 0 for slot n_pairs, then the
// X_beta = 0 group's folded factors.  The entry's class, row and class
// record are uniform across the workgroup; the pair-map row is read
// coalesced.
constexpr uint32_t kImgBlock = 128;
__global__ __launch_bounds__(kImgBlock) void k_pair_images(uint32_t n_img, uint32_t n_pairs, const uint32_t* str_a,
                                                           const uint32_t* ent_cls, const uint32_t* ent_row,
                                                           const ClassMeta* meta, const int32_t* pmap,
                                                           const uint32_t* pg_u0, const uint32_t* u_t0,
                                                           const uint32_t* pt_za, const double* pt_c,
                                                           const uint4* cls_f, const uint32_t* fu_t0,
                                                           const uint32_t* ft_za, const double* ft_c, double* img) {
  const uint64_t e = blockIdx.x;
  const uint32_t c = ent_cls[e], ta = str_a[ent_row[e]];
  const int32_t* prow = pmap + static_cast<uint64_t>(meta[c].pm) * n_pairs;
  const uint4 cf = cls_f[c];
  for (uint32_t j = threadIdx.x; j < n_img; j += kImgBlock) {
    double f = 0.0;
    if (j < n_pairs) {
      const int32_t g = prow[j];
      if (g >= 0) {
        const uint32_t u = pg_u0[g];
        for (uint32_t t = u_t0[u]; t < u_t0[u + 1]; ++t) f += (__popc(pt_za[t] & ta) & 1u) ? -pt_c[2 * t] : pt_c[2 * t];
      }
    } else if (j > n_pairs) {
      const uint32_t r = j - n_pairs - 1;
      if (r < cf.y) {
        const uint32_t u = cf.x + r;
        for (uint32_t t = fu_t0[u]; t < fu_t0[u + 1]; ++t) f += (__popc(ft_za[t] & ta) & 1u) ? -ft_c[t] : ft_c[t];
      }
    }
    img[e * n_img + j] = f;
  }
}

// ---- tables of the panel kernel (panel.h)

// Beta-only part of the X_alpha = 0 class per move and column: source column
// (two moves share a word) and coefficient; moves in the order of
// k_fact_moves, then of k_fact_quads.
__global__ void k_panel_moves(uint64_t db, uint32_t n_orb, uint32_t n_beta, uint32_t n_moves, uint32_t n_bb,
                              const uint32_t* str_b, const int32_t* pk, const int32_t* qk, const uint32_t* p_lo,
                              const uint32_t* q_lo, const uint32_t* zb, const double* c, uint16_t* src, double* coef) {
  const uint32_t ne = n_orb - n_beta, n_ep = ne * (ne - 1) / 2;
  const uint32_t full = (n_orb == 32) ? 0xffffffffu : ((1u << n_orb) - 1u);
  const uint64_t n = static_cast<uint64_t>(n_bb) * db;
  for (uint64_t i = blockIdx.x * static_cast<uint64_t>(blockDim.x) + threadIdx.x; i < n;
       i += static_cast<uint64_t>(gridDim.x) * blockDim.x) {
    const uint32_t m = static_cast<uint32_t>(i / db);
    const uint64_t j = i % db;
    const uint32_t tb = str_b[j], emp = ~tb & full;
    uint32_t X;
    int32_t k;
    const uint32_t* lo;
    if (m < n_moves) {
      const uint32_t p = kth_bit(tb, m / ne), q = kth_bit(emp, m % ne);
      const uint32_t a = p < q ? p : q, b = p < q ? q : p;
      X = (1u << p) | (1u << q);
      k = pk[b * (b - 1) / 2 + a];
      lo = p_lo;
    } else {
      uint32_t a, b, d, e;
      pair_at((m - n_moves) / n_ep, n_beta, a, b);
      pair_at((m - n_moves) % n_ep, ne, d, e);
      X = (1u << kth_bit(tb, a)) | (1u << kth_bit(tb, b)) | (1u << kth_bit(emp, d)) | (1u << kth_bit(emp, e));
      k = qk[colex_rank(X)];
      lo = q_lo;
    }
    src[((m / 2) * db + j) * 2 + (m & 1u)] = static_cast<uint16_t>(colex_rank(tb ^ X));
    coef[m * db + j] = k >= 0 ? eval_rows(zb, c, lo[k], lo[k + 1], tb) : 0.0;
  }
}

// Per alpha row: the alpha-dependent part of the X_alpha = 0 pair groups
// (one value per orbital pair), then the diagonal group's folded factors.
__global__ __launch_bounds__(128) void k_panel_rows(uint64_t da, uint32_t n_pairs, uint32_t rank, uint32_t fu0,
                                                    const uint32_t* str_a, const uint32_t* al_lo,
                                                    const uint32_t* al_za, const double* al_c, const uint32_t* fu_t0,
                                                    const uint32_t* ft_za, const double* ft_c, double* img,
                                                    double* diag) {
  for (uint64_t i = blockIdx.x; i < da; i += gridDim.x) {
    const uint32_t ta = str_a[i];
    for (uint32_t j = threadIdx.x; j < n_pairs + rank; j += blockDim.x) {
      if (j < n_pairs)
        img[i * n_pairs + j] = eval_rows(al_za, al_c, al_lo[j], al_lo[j + 1], ta);
      else
        diag[i * rank + (j - n_pairs)] =
            eval_rows(ft_za, ft_c, fu_t0[fu0 + j - n_pairs], fu_t0[fu0 + j - n_pairs + 1], ta);
    }
  }
}

// The V entries that each target reads.  Targets are taken in groups of 64
// (group 8 j + w belongs to wave w of the panel workgroup); one wave per
// group.  Pass 0 writes, per tile of source columns, the most entries any
// lane of the group has; pass 1 places the entries of lane l at
// pull[(off + i) * 64 + l], i in the order of the lane's moves.
constexpr uint32_t kPullWaves = kPanelLanes / 64;
__global__ __launch_bounds__(64) void k_pull(uint32_t pass, uint32_t db, uint32_t n_orb, uint32_t n_beta,
                                             uint32_t n_tiles, const uint32_t* str_b, const uint32_t* zpair,
                                             uint8_t* cnt, const uint32_t* off, uint16_t* pull) {
  __shared__ uint8_t s_n[kPanelCols / kPanelTile][64];
  const uint32_t g = blockIdx.x, w = g % kPullWaves, jg = g / kPullWaves, lane = threadIdx.x;
  const uint32_t t = g * 64u + lane;
  for (uint32_t k = 0; k < n_tiles; ++k) s_n[k][lane] = 0;
  if (t < db) {
    const uint32_t full = (n_orb == 32) ? 0xffffffffu : ((1u << n_orb) - 1u);
    const uint32_t tb = str_b[t];
    for (uint32_t occ = tb; occ; occ &= occ - 1) {
      const uint32_t p = __ffs(occ) - 1;
      for (uint32_t emp = ~tb & full; emp; emp &= emp - 1) {
        const uint32_t q = __ffs(emp) - 1;
        const uint32_t a = p < q ? p : q, b = p < q ? q : p, pair = b * (b - 1) / 2 + a;
        const uint32_t src = colex_rank(tb ^ (1u << p) ^ (1u << q)), tile = src / kPanelTile;
        const uint32_t i = s_n[tile][lane]++;
        if (pass)
          pull[(static_cast<uint64_t>(off[(tile * kPullWaves + w) * 8u + jg]) + i) * 64u + lane] =
              static_cast<uint16_t>(pair * kPanelTile + src % kPanelTile + ((__popc(zpair[pair] & tb) & 1u) << 15));
      }
    }
  }
  if (pass) return;
  for (uint32_t k = 0; k < n_tiles; ++k) {
    uint32_t m = s_n[k][lane];
    for (int d = 32; d > 0; d >>= 1) m = max(m, static_cast<uint32_t>(__shfl_xor(m, d, 64)));
    if (lane == 0) cnt[(k * kPullWaves + w) * 8u + jg] = static_cast<uint8_t>(m);
  }
}

// First slot of every (tile, wave, group), in that order, and the records of
// FactorPlan::pull_cnt; total[0] = all slots, total[1] = the most of one tile.
// One workgroup of one wave (at most 64 tiles).
static_assert(kPanelCols / kPanelTile <= 64, "one lane per tile");
__global__ __launch_bounds__(64) void k_pull_offsets(uint32_t n_tiles, const uint8_t* cnt, uint32_t* off, uint4* rec,
                                                     uint32_t* total) {
  const uint32_t tile = threadIdx.x;
  const uint8_t* c = cnt + tile * kPullWaves * 8u;
  uint32_t sum = 0;
  if (tile < n_tiles)
    for (uint32_t i = 0; i < kPullWaves * 8u; ++i) sum += c[i];
  uint32_t incl = sum, most = sum;
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t v = __shfl_up(incl, d, 64);
    if (tile >= static_cast<uint32_t>(d)) incl += v;
    most = max(most, static_cast<uint32_t>(__shfl_xor(most, d, 64)));
  }
  if (tile == 63) {
    total[0] = incl;
    total[1] = most;
  }
  if (tile >= n_tiles) return;
  uint32_t at = 0;
  for (uint32_t w = 0; w < kPullWaves; ++w) {
    uint32_t lo = 0, hi = 0;
    const uint32_t first = at;
    for (uint32_t j = 0; j < 8; ++j) {
      const uint32_t n = c[w * 8u + j];
      off[(tile * kPullWaves + w) * 8u + j] = incl - sum + at;
      if (j < 4)
        lo |= n << (8 * j);
      else
        hi |= n << (8 * (j - 4));
      at += n;
    }
    rec[tile * kPullWaves + w] = make_uint4(lo, hi, first, incl - sum);
  }
}

// Column lists of the pair groups (xb, zb, code = magnitude index | sign << 15
// of their single coefficient): one wave per 64 columns.  Pass 0 writes the
// slots of four entries that the longest list needs; pass 1 writes the
// entries in group order and fills up with entries that read a zero.
__global__ __launch_bounds__(64) void k_column_lists(uint32_t pass, uint32_t db, const uint32_t* str_b,
                                                     const uint32_t* xb, const uint32_t* zb, const uint32_t* code,
                                                     uint32_t n_grp, bool narrow, uint32_t* slots,
                                                     const uint32_t* off, void* ent) {
  const uint32_t grp = blockIdx.x, lane = threadIdx.x, col = grp * 64u + lane;
  const uint32_t tb = col < db ? str_b[col] : 0u;
  const uint64_t base = pass ? off[grp] : 0u;
  uint32_t n = 0;
  auto put = [&](uint32_t w) {
    const uint64_t at = ((base + n / 4u) * 64u + lane) * 4u + n % 4u;
    if (pass && narrow) static_cast<uint16_t*>(ent)[at] = static_cast<uint16_t>((w & 0x7fffu) | (w >> 16));
    if (pass && !narrow) static_cast<uint32_t*>(ent)[at] = w;
    ++n;
  };
  if (col < db)
    for (uint32_t g = 0; g < n_grp; ++g) {
      if (__popc(tb & xb[g]) != 1) continue;
      put(colex_rank(tb ^ xb[g]) | ((code[g] ^ ((__popc(zb[g] & tb) & 1u) << 15)) << 16));
    }
  if (pass) {
    const uint32_t all = 4u * (off[grp + 1] - off[grp]);
    while (n < all) put(db);
    return;
  }
  for (int d = 32; d > 0; d >>= 1) n = max(n, static_cast<uint32_t>(__shfl_xor(n, d, 64)));
  if (lane == 0) slots[grp] = (n + 3u) / 4u;
}

__global__ void k_fill_u32(uint32_t* p, uint64_t n, uint32_t v) {
  for (uint64_t i = blockIdx.x * static_cast<uint64_t>(blockDim.x) + threadIdx.x; i < n;
       i += static_cast<uint64_t>(gridDim.x) * blockDim.x)
    p[i] = v;
}

// ---------------------------------------------------------------- host side

// The beta-only lists of the X_alpha = 0 class (one per pair group, then one
// per quad group) and, per orbital pair, the alpha list of what is left of
// its pair groups; false when the operator or the sector is not one that the
// panel kernel evaluates (see FactorPlan::panel).
struct PanelLists {
  std::vector<uint32_t> p_lo{0}, q_lo{0}, zb, al_lo{0}, al_za;
  std::vector<double> c, al_c;
};
bool panel_lists(const FactorPlan& F, const pbs_grouped& h, const pbs_space& sp, const HostTables& T,
                 const std::vector<ClassMeta>& meta, const std::vector<uint4>& cls_f,
                 const std::vector<uint32_t>& zpair, const std::vector<uint32_t>& icls, PanelLists* L) {
  if (F.c0 == 0xffffffffu || F.ns_sizes[2] != 0 || !h.pair_sign) return false;
  for (uint32_t c : icls)
    if (__builtin_popcount(meta[c].xa) != 2) return false;  // then a row has N_alpha (n_orb - N_alpha) at most
  const ClassMeta& m = meta[F.c0];
  if (m.q1 != m.g1 || (m.zg >= 0 && cls_f[F.c0].y == 0)) return false;
  const uint32_t gz_end = m.zg >= 0 ? m.g0 + 1 : m.g0;
  std::vector<std::vector<std::pair<uint32_t, double>>> al(h.n_pairs);
  for (uint32_t g = gz_end; g < m.q1; ++g) {
    const bool quad = g >= m.p1;
    uint32_t pair = 0;
    if (!quad) {
      const uint32_t x = T.pg_xb[g];
      const uint32_t lo = static_cast<uint32_t>(__builtin_ctz(x)), hi = 31u - static_cast<uint32_t>(__builtin_clz(x));
      pair = hi * (hi - 1) / 2 + lo;
    }
    if (g == m.p1) L->q_lo[0] = static_cast<uint32_t>(L->zb.size());
    for (uint32_t u = T.pg_u0[g]; u < T.pg_u0[g + 1]; ++u) {
      double b = 0.0;
      bool any = false;
      for (uint32_t t = T.u_t0[u]; t < T.u_t0[u + 1]; ++t) {
        if (T.pt_za[t] == 0u) {
          b += T.pt_c[t];
          any = true;
        } else if (quad || T.u_zb[u] != zpair[pair]) {
          return false;  // an alpha-dependent term without the pair's beta parity
        } else {
          al[pair].emplace_back(T.pt_za[t], T.pt_c[t]);
        }
      }
      if (any) {
        L->zb.push_back(T.u_zb[u]);
        L->c.push_back(b);
      }
    }
    (quad ? L->q_lo : L->p_lo).push_back(static_cast<uint32_t>(L->zb.size()));
  }
  for (const auto& l : al) {
    for (const auto& t : l) {
      L->al_za.push_back(t.first);
      L->al_c.push_back(t.second);
    }
    L->al_lo.push_back(static_cast<uint32_t>(L->al_za.size()));
  }
  return true;
}

// Pair groups of the lists kernel; false when the operator is not one that it
// evaluates (see lists.h).
struct ColumnGroups {
  std::vector<uint32_t> xb, zb, code;
  std::vector<double> mag;
};
constexpr size_t kMaxMagnitudes = 256;
bool column_groups(const HostTables& T, const ClassMeta& m, ColumnGroups* C) {
  if (m.xa != 0 || m.p1 != m.g1) return false;
  std::map<double, uint32_t> index;
  for (uint32_t g = m.zg >= 0 ? m.g0 + 1 : m.g0; g < m.g1; ++g) {
    const uint32_t u = T.pg_u0[g];
    if (T.pg_u0[g + 1] != u + 1) return false;
    double c = 0.0;
    for (uint32_t t = T.u_t0[u]; t < T.u_t0[u + 1]; ++t) {
      if (T.pt_za[t] != 0u) return false;
      c += T.pt_c[t];
    }
    if (!std::isfinite(c)) return false;
    const auto at = index.emplace(std::fabs(c), static_cast<uint32_t>(index.size())).first;
    if (at->second == C->mag.size()) C->mag.push_back(std::fabs(c));
    if (C->mag.size() > kMaxMagnitudes) return false;
    C->xb.push_back(T.pg_xb[g]);
    C->zb.push_back(T.u_zb[u]);
    C->code.push_back(at->second | (std::signbit(c) ? 0x8000u : 0u));
  }
  return !C->xb.empty();
}

}  // namespace

std::unique_ptr<FactorPlan> make_factor_plan(const pbs_grouped& h, const pbs_space& sp, bool move_tables,
                                             hipStream_t s) {
  auto plan = std::make_unique<FactorPlan>();
  FactorPlan& F = *plan;
  F.n_orb = sp.n_orb;
  F.n_beta = sp.n_beta;
  F.dim_beta = sp.dim_beta;
  const uint64_t db = sp.dim_beta;
  Staging st(s);
  HostTables T;
  std::vector<double> pt_c2;
  std::vector<ClassMeta> meta;
  std::vector<uint32_t> ns, zpair;
  st.fetch(zpair, h.zpair, h.n_pairs + 1);
  st.fetch(T.pg_u0, h.pg_u0, h.n_pgroup + 1);
  st.fetch(T.u_zb, h.u_zb, h.n_unique);
  st.fetch(T.u_t0, h.u_t0, h.n_unique + 1);
  st.fetch(T.pt_za, h.pt_za, h.n_pterm);
  st.fetch(T.pg_xb, h.pg_xb, h.n_pgroup);
  st.fetch(pt_c2, h.pt_c, 2ull * h.n_pterm);
  st.fetch(meta, h.cls_meta, h.n_class);
  st.fetch(ns, h.ns_list, h.n_ns);
  st.wait();
  T.pt_c.resize(h.n_pterm);
  for (uint32_t t = 0; t < h.n_pterm; ++t) T.pt_c[t] = pt_c2[2ull * t];

  // factor uniques (alpha side) and the beta lists of the table rows
  std::vector<uint32_t> fu_t0{0}, ft_za;
  std::vector<double> ft_c;
  std::vector<uint32_t> q_lo{0}, q_zb;
  std::vector<double> q_c;
  auto add_factor = [&](const std::vector<std::pair<uint32_t, double>>* a) {
    if (a)
      for (auto& t : *a) {
        ft_za.push_back(t.first);
        ft_c.push_back(t.second);
      }
    fu_t0.push_back(static_cast<uint32_t>(ft_za.size()));
  };
  auto add_row = [&](const std::vector<std::pair<uint32_t, double>>* b) {
    if (b)
      for (auto& t : *b) {
        q_zb.push_back(t.first);
        q_c.push_back(t.second);
      }
    q_lo.push_back(static_cast<uint32_t>(q_zb.size()));
  };

  // the class with X_alpha = 0: its pair groups (single moves) and quad groups
  // (double moves), when the sector kernel enumerates both
  const uint32_t ne = sp.n_orb - sp.n_beta;
  const uint32_t n_moves = sp.n_beta * ne;
  const uint64_t n_qmoves = host_binom(sp.n_beta, 2) * host_binom(ne, 2);
  uint32_t c0 = 0xffffffffu;
  for (uint32_t c : ns)
    if (meta[c].xa == 0) c0 = c;
  std::vector<GroupFactors> pf, qf;
  if (c0 != 0xffffffffu && sp.n_orb <= 16 && n_moves > 0 && n_qmoves > 0 && db < 65536) {
    const ClassMeta& m = meta[c0];
    const uint32_t gz_end = m.zg >= 0 ? m.g0 + 1 : m.g0;
    uint32_t r2 = 0, r3 = 0;
    for (uint32_t g = gz_end; g < m.p1; ++g) {
      pf.push_back(factor_group(T, g));
      r2 = std::max(r2, pf.back().rank);
    }
    for (uint32_t g = m.p1; g < m.q1; ++g) {
      qf.push_back(factor_group(T, g));
      r3 = std::max(r3, qf.back().rank);
    }
    const uint64_t n_fold = static_cast<uint64_t>(pf.size()) * r2 + static_cast<uint64_t>(qf.size()) * r3;
    // the tables hold every move of a target, present group or not: used
    // only when most orbital pairs / quadruples have a group (two-body
    // operators with dense integrals), where they replace long phase sums
    const bool dense = 2 * pf.size() >= h.n_pairs && 2 * qf.size() >= h.n_quads;
    if (dense && r2 >= 1 && r2 <= 2 && r3 >= 1 && r3 <= 2 && kFactZeroSlots + n_fold <= 4096) {
      F.c0 = c0;
      F.r2 = r2;
      F.r3 = r3;
    } else {
      pf.clear();
      qf.clear();
    }
  }
  std::vector<int32_t> pk(h.n_pairs + 1, -1), qk(h.n_quads ? h.n_quads : 1, -1);
  if (F.c0 != 0xffffffffu) {
    const ClassMeta& m = meta[c0];
    const uint32_t gz_end = m.zg >= 0 ? m.g0 + 1 : m.g0;
    F.c0_fu0 = 0;
    for (uint32_t k = 0; k < pf.size(); ++k) {
      const uint32_t x = T.pg_xb[gz_end + k];
      const uint32_t lo = static_cast<uint32_t>(__builtin_ctz(x)), hi = 31u - static_cast<uint32_t>(__builtin_clz(x));
      pk[hi * (hi - 1) / 2 + lo] = static_cast<int32_t>(k);
      for (uint32_t r = 0; r < F.r2; ++r) add_factor(r < pf[k].rank ? &pf[k].a[r] : nullptr);
    }
    F.c0_fq = static_cast<uint32_t>(fu_t0.size() - 1);
    for (uint32_t k = 0; k < qf.size(); ++k) {
      uint32_t x = T.pg_xb[m.p1 + k], id = 0;
      for (uint32_t j = 1; j <= 4; ++j) {
        const uint32_t b = static_cast<uint32_t>(__builtin_ctz(x));
        x &= x - 1;
        id += static_cast<uint32_t>(host_binom(b, j));
      }
      qk[id] = static_cast<int32_t>(k);
      for (uint32_t r = 0; r < F.r3; ++r) add_factor(r < qf[k].rank ? &qf[k].a[r] : nullptr);
    }
    F.c0_fu1 = static_cast<uint32_t>(fu_t0.size() - 1);
    F.n_f2 = static_cast<uint32_t>(pf.size());
    F.n_f3 = static_cast<uint32_t>(qf.size());
    F.n_moves = n_moves;
    F.n_qmoves = static_cast<uint32_t>(n_qmoves);
  }
  const uint32_t rows_p = static_cast<uint32_t>(q_lo.size() - 1);
  for (uint32_t k = 0; k < pf.size(); ++k)
    for (uint32_t r = 0; r < F.r2; ++r) add_row(r < pf[k].rank ? &pf[k].b[r] : nullptr);
  const uint32_t rows_q = static_cast<uint32_t>(q_lo.size() - 1);
  for (uint32_t k = 0; k < qf.size(); ++k)
    for (uint32_t r = 0; r < F.r3; ++r) add_row(r < qf[k].rank ? &qf[k].b[r] : nullptr);
  const uint32_t rows_z = static_cast<uint32_t>(q_lo.size() - 1);

  // X_beta = 0 groups of the non-simple classes, factored when that lowers
  // the number of beta terms a target evaluates
  std::vector<uint4> cls_f(h.n_class, make_uint4(0u, 0u, 0u, 0u));
  uint32_t n_zrows = 0;
  for (uint32_t c : ns) {
    const ClassMeta& m = meta[c];
    if (m.zg < 0) continue;
    GroupFactors G = factor_group(T, static_cast<uint32_t>(m.zg));
    if (G.rank == 0 || G.rank > kMaxR1 || G.rank >= G.n_uniques) continue;
    const uint32_t fu0 = static_cast<uint32_t>(fu_t0.size() - 1);
    for (uint32_t r = 0; r < G.rank; ++r) {
      add_factor(&G.a[r]);
      add_row(&G.b[r]);
    }
    cls_f[c] = make_uint4(fu0, G.rank, 0u, 0u);
    *reinterpret_cast<uint64_t*>(&cls_f[c].z) = static_cast<uint64_t>(n_zrows) * db;
    n_zrows += G.rank;
    F.max_r1 = std::max(F.max_r1, G.rank);
    ++F.n_f1;
  }
  F.n_fu = static_cast<uint32_t>(fu_t0.size() - 1);
  auto most_terms = [&](uint32_t a, uint32_t b) {
    uint32_t t = 0;
    for (uint32_t u = a; u < b; ++u) t = std::max(t, fu_t0[u + 1] - fu_t0[u]);
    return t;
  };
  F.t_pair = most_terms(F.c0_fu0, F.c0_fq);
  F.t_quad = most_terms(F.c0_fq, F.c0_fu1);
  F.t_zero = most_terms(F.c0_fu1, F.n_fu);
  F.n_ft = static_cast<uint32_t>(ft_za.size());

  // the class lists: simple classes (when every unique of every one of them
  // has beta Z-mask 0), image classes, and what is left without them
  const uint64_t da = sp.dim_alpha;
  std::vector<uint32_t> simple, icls, flag(h.n_class, 0u);
  bool plain = true;
  for (uint32_t c = 0; c < h.n_class && plain; ++c) {
    if (!(meta[c].flags & kClassSimple)) continue;
    simple.push_back(c);
    for (uint32_t u = meta[c].ua; u < meta[c].u_end; ++u) plain = plain && T.u_zb[u] == 0u;
  }
  F.alist = plain && !simple.empty();
  if (F.alist) F.n_alpha = sp.n_alpha;
  if (F.alist && h.pair_sign) {
    for (uint32_t c : ns) {
      const ClassMeta& m = meta[c];
      if (c == F.c0 || m.pm < 0 || !(m.flags & kClassPairsSingle) || m.p1 != m.g1) continue;
      if (m.zg >= 0 && (cls_f[c].y == 0 || cls_f[c].y > 2)) continue;
      icls.push_back(c);
      flag[c] = 1u;
    }
  }
  F.plist = !icls.empty();
  std::vector<uint32_t> rest[3];
  F.ns_sizes.assign(3, 0u);
  for (uint32_t c : ns) {
    F.ns_uniques += meta[c].u_end - meta[c].ua;
    F.ns_groups += meta[c].g1 - meta[c].g0;
    for (int k = 0; k < 3; ++k)
      if (!((k != 1 && c == F.c0) || (k != 0 && flag[c]))) rest[k].push_back(c);
  }
  for (int k = 0; k < 3; ++k) F.ns_sizes[k] = static_cast<uint32_t>(rest[k].size());
  PanelLists L;
  const int variant =
      panel_variant_for(sp.dim_alpha, sp.dim_beta, h.n_pairs, sp.n_alpha * (sp.n_orb - sp.n_alpha) + 1u);
  bool panel = F.plist && variant >= 0 && panel_lists(F, h, sp, T, meta, cls_f, zpair, icls, &L);

  ColumnGroups cols;
  const bool blist = F.alist && F.c0 == 0xffffffffu && ns.size() == 1 && sp.n_orb <= 16 && db < 65536 &&
                     column_groups(T, meta[ns[0]], &cols);
  const uint32_t col_groups = static_cast<uint32_t>((db + 63) / 64);

  // tables whose sizes are known, and the temporaries of this call
  // (a plan built for the panel kernel alone leaves the sector kernel's move tables out)
  const bool moves = F.c0 != 0xffffffffu;
  const bool tables = moves && move_tables;
  Slab own, tmp;
  own.upload(F.fu_t0, fu_t0);
  own.upload(F.ft_za, ft_za);
  own.upload(F.ft_c, ft_c);
  own.upload(F.cls_f, cls_f);
  for (int k = 0; k < 3; ++k) own.upload(F.ns_rest[k], rest[k]);
  if (F.plist) own.upload(F.pimg_flag, flag);
  // (the panel kernel loads a first F row for every image class, also where
  // no class has one: then a row of zeros, which its evaluation leaves out)
  own.add(F.fz, static_cast<uint64_t>(panel ? std::max(n_zrows, 1u) : n_zrows) * db);
  DevBuf<uint32_t> d_qlo, d_qzb, d_simple, d_icls, cnt_a, cnt_p, ent_row;
  DevBuf<double> d_qc;
  DevBuf<int32_t> d_pk, d_qk;
  tmp.upload(d_qlo, q_lo);
  tmp.upload(d_qzb, q_zb);
  tmp.upload(d_qc, q_c);
  if (moves) {
    tmp.upload(d_pk, pk);
    tmp.upload(d_qk, qk);
  }
  if (tables) {
    own.add(F.em, static_cast<uint64_t>(n_moves) * db);
    own.add(F.fp, static_cast<uint64_t>(n_moves) * F.r2 * db);
    own.add(F.eq, n_qmoves * db);
    own.add(F.fq, n_qmoves * F.r3 * db);
  }
  if (F.alist) {
    tmp.upload(d_simple, simple);
    tmp.add(cnt_a, da);
    own.add(F.alist_off, da + 1);
  }
  if (F.plist) {
    tmp.upload(d_icls, icls);
    tmp.add(cnt_p, da);
    own.add(F.plist_off, da + 1);
    F.n_img = h.n_pairs + 3;
  }
  DevBuf<uint32_t> d_plo, d_ql2, d_zb, d_allo, d_alza, pull_off, pull_total;
  DevBuf<double> d_c, d_alc;
  DevBuf<uint8_t> pull_n;
  uint32_t n_rec = 0;
  const uint32_t pull_groups = static_cast<uint32_t>((db + 63) / 64);
  if (panel) {
    F.n_bb = F.n_moves + F.n_qmoves;
    F.n_tiles = static_cast<uint32_t>((db + kPanelTile - 1) / kPanelTile);
    const ClassMeta& m = meta[F.c0];
    F.diag_rank = m.zg >= 0 ? cls_f[F.c0].y : 0u;
    F.diag_off = cls_f[F.c0].z | (static_cast<uint64_t>(cls_f[F.c0].w) << 32);
    n_rec = F.n_tiles * kPullWaves;
    tmp.upload(d_plo, L.p_lo);
    tmp.upload(d_ql2, L.q_lo);
    tmp.upload(d_zb, L.zb);
    tmp.upload(d_c, L.c);
    tmp.upload(d_allo, L.al_lo);
    tmp.upload(d_alza, L.al_za);
    tmp.upload(d_alc, L.al_c);
    tmp.add(pull_n, 8ull * n_rec);
    tmp.add(pull_off, 8ull * n_rec);
    tmp.add(pull_total, 2);
    own.add(F.bb_src, (F.n_bb + 1ull) / 2ull * db);
    own.add(F.bb_c, F.n_bb * db);
    own.add(F.c0img, da * h.n_pairs);
    own.add(F.diag_a, da * F.diag_rank);
    own.add(F.pull_cnt, n_rec);
  }
  DevBuf<uint32_t> d_bx, d_bz, d_bcode, bl_slots;
  if (blist) {
    const ClassMeta& m = meta[ns[0]];
    F.bl_ua = m.ua;
    F.bl_ub = m.zg >= 0 ? m.u_z : m.ua;
    F.n_mag = static_cast<uint32_t>(cols.mag.size());
    F.bl_narrow = F.n_mag == 1 && db < 32768;
    tmp.upload(d_bx, cols.xb);
    tmp.upload(d_bz, cols.zb);
    tmp.upload(d_bcode, cols.code);
    tmp.add(bl_slots, col_groups);
    own.add(F.bl_off, col_groups + 1);
    own.upload(F.bl_mag, cols.mag);
  }
  DevBuf<char> tmp_mem;
  st.commit(own, F.mem[0], false);
  st.commit(tmp, tmp_mem, true);

  // counts first: they come back while the other tables are built
  const unsigned row_grid = static_cast<unsigned>(std::min<uint64_t>(da, 65536));
  std::vector<uint32_t> ca, cp, slots, col_slots;
  if (blist) {
    hipLaunchKernelGGL(k_column_lists, dim3(col_groups), dim3(64), 0, s, 0u, static_cast<uint32_t>(db),
                       sp.str_beta.get(), d_bx.get(), d_bz.get(), d_bcode.get(),
                       static_cast<uint32_t>(cols.xb.size()), F.bl_narrow, bl_slots.get(), nullptr, nullptr);
    st.fetch(col_slots, bl_slots, col_groups);
    exclusive_scan_u32(bl_slots.get(), F.bl_off.get(), col_groups, F.bl_off.get() + col_groups, s);
  }
  if (F.alist) {
    hipLaunchKernelGGL(k_alpha_list, dim3(row_grid), dim3(256), 0, s, 0u, da, sp.n_alpha, sp.str_alpha.get(),
                       d_simple.get(), static_cast<uint32_t>(simple.size()), h.cls_meta.get(), h.u_t0.get(),
                       h.pt_za.get(), h.pt_c.get(), nullptr, cnt_a.get(), nullptr, nullptr);
    st.fetch(ca, cnt_a, da);
    exclusive_scan_u32(cnt_a.get(), F.alist_off.get(), da, F.alist_off.get() + da, s);
  }
  if (F.plist) {
    hipLaunchKernelGGL(k_pair_list, dim3(row_grid), dim3(256), 0, s, 0u, da, sp.n_alpha, sp.str_alpha.get(),
                       d_icls.get(), static_cast<uint32_t>(icls.size()), h.cls_meta.get(), nullptr, cnt_p.get(),
                       nullptr, nullptr, nullptr);
    st.fetch(cp, cnt_p, da);
    exclusive_scan_u32(cnt_p.get(), F.plist_off.get(), da, F.plist_off.get() + da, s);
  }
  if (panel) {
    // (every slot count is below 256, so a fill of 32-bit zeros clears four)
    hipLaunchKernelGGL(k_fill_u32, dim3(grid_for(2ull * n_rec, 256, 4096)), dim3(256), 0, s,
                       reinterpret_cast<uint32_t*>(pull_n.get()), 2ull * n_rec, 0u);
    hipLaunchKernelGGL(k_pull, dim3(pull_groups), dim3(64), 0, s, 0u, static_cast<uint32_t>(db), sp.n_orb, sp.n_beta,
                       F.n_tiles, sp.str_beta.get(), h.zpair.get(), pull_n.get(), nullptr, nullptr);
    hipLaunchKernelGGL(k_pull_offsets, dim3(1), dim3(64), 0, s, F.n_tiles, pull_n.get(), pull_off.get(),
                       F.pull_cnt.get(), pull_total.get());
    st.fetch(slots, pull_total, 2);
  }
  PBS_HIP(hipGetLastError());
  if (panel && n_zrows == 0)
    hipLaunchKernelGGL(k_fill_u32, dim3(grid_for(2 * db, 256, 4096)), dim3(256), 0, s,
                       reinterpret_cast<uint32_t*>(F.fz.get()), 2 * db, 0u);
  if (n_zrows) {
    const uint64_t n = static_cast<uint64_t>(n_zrows) * db;
    hipLaunchKernelGGL(k_fact_rows, dim3(grid_for(n, 256, 65536)), dim3(256), 0, s, n_zrows, db, sp.str_beta.get(),
                       d_qlo.get() + rows_z, d_qzb.get(), d_qc.get(), F.fz.get());
  }
  if (tables) {
    const uint64_t nm = static_cast<uint64_t>(n_moves) * db, nq = n_qmoves * db;
    hipLaunchKernelGGL(k_fact_moves, dim3(grid_for(nm, 256, 65536)), dim3(256), 0, s, db, sp.n_orb, sp.n_beta, F.r2,
                       sp.str_beta.get(), d_pk.get(), d_qlo.get() + rows_p, d_qzb.get(), d_qc.get(), F.em.get(),
                       F.fp.get());
    const uint32_t slot0 = kFactZeroSlots + F.n_f2 * F.r2;
    hipLaunchKernelGGL(k_fact_quads, dim3(grid_for(nq, 256, 65536)), dim3(256), 0, s, db, sp.n_orb, sp.n_beta,
                       F.r3, slot0, sp.str_beta.get(), d_qk.get(), d_qlo.get() + rows_q, d_qzb.get(), d_qc.get(),
                       F.eq.get(), F.fq.get());
  }
  if (panel) {
    hipLaunchKernelGGL(k_panel_moves, dim3(grid_for(F.n_bb * db, 256, 65536)), dim3(256), 0, s, db, sp.n_orb,
                       sp.n_beta, F.n_moves, F.n_bb, sp.str_beta.get(), d_pk.get(), d_qk.get(), d_plo.get(),
                       d_ql2.get(), d_zb.get(), d_c.get(), reinterpret_cast<uint16_t*>(F.bb_src.get()), F.bb_c.get());
    hipLaunchKernelGGL(k_panel_rows, dim3(row_grid), dim3(128), 0, s, da, h.n_pairs, F.diag_rank, cls_f[F.c0].x,
                       sp.str_alpha.get(), d_allo.get(), d_alza.get(), d_alc.get(), F.fu_t0.get(), F.ft_za.get(),
                       F.ft_c.get(), F.c0img.get(), F.diag_a.get());
  }
  PBS_HIP(hipGetLastError());
  st.wait();

  // the lists and images, whose sizes the counts give
  uint64_t n_list = 0, n_ent = 0;
  for (uint32_t v : ca) {
    n_list += v;
    F.alist_max = std::max(F.alist_max, v);
  }
  for (uint32_t v : cp) n_ent += v;
  PBS_REQUIRE(n_ent < (1ull << 31), PBS_ERR_RANGE, "more than 2^31 alpha-image entries");
  panel = panel && slots[1] <= kPanelPullSlots;
  // absent entries read V's zero; a tile's copy may run past the last slot
  const uint64_t pull_words = panel ? 32ull * (slots[0] + kPanelPullSlots) : 0u;
  Slab lists;
  // (the lists kernel reads a fixed number of entries, past the last list too)
  lists.add(F.alist_src, n_list + (blist ? kListRowsAhead : 0u));
  lists.add(F.alist_c, n_list + (blist ? kListRowsAhead : 0u));
  lists.add(F.plist_src, n_ent);
  lists.add(F.plist_cls, n_ent);
  lists.add(F.pimg, n_ent * F.n_img);
  lists.add(F.pull, pull_words / 4);
  uint64_t n_slots = 0;
  for (uint32_t v : col_slots) n_slots += v;
  // a wave loads a fixed number of slots, past the last list too
  if (blist) lists.add(F.bl_ent, 64ull * (n_slots + kListSlotsAhead) * (F.bl_narrow ? 1u : 2u));
  st.commit(lists, F.mem[1], false);
  if (n_list)
    hipLaunchKernelGGL(k_alpha_list, dim3(row_grid), dim3(256), 0, s, 1u, da, sp.n_alpha, sp.str_alpha.get(),
                       d_simple.get(), static_cast<uint32_t>(simple.size()), h.cls_meta.get(), h.u_t0.get(),
                       h.pt_za.get(), h.pt_c.get(), F.alist_off.get(), nullptr, F.alist_src.get(), F.alist_c.get());
  if (blist) {
    hipLaunchKernelGGL(k_column_lists, dim3(col_groups), dim3(64), 0, s, 1u, static_cast<uint32_t>(db),
                       sp.str_beta.get(), d_bx.get(), d_bz.get(), d_bcode.get(),
                       static_cast<uint32_t>(cols.xb.size()), F.bl_narrow, nullptr, F.bl_off.get(), F.bl_ent.get());
    F.blist = true;
  }
  if (n_ent) {
    ent_row = DevBuf<uint32_t>(n_ent, s);
    hipLaunchKernelGGL(k_pair_list, dim3(row_grid), dim3(256), 0, s, 1u, da, sp.n_alpha, sp.str_alpha.get(),
                       d_icls.get(), static_cast<uint32_t>(icls.size()), h.cls_meta.get(), F.plist_off.get(), nullptr,
                       F.plist_src.get(), F.plist_cls.get(), ent_row.get());
    hipLaunchKernelGGL(k_pair_images, dim3(static_cast<unsigned>(n_ent)), dim3(kImgBlock), 0, s, F.n_img, h.n_pairs,
                       sp.str_alpha.get(), F.plist_cls.get(), ent_row.get(), h.cls_meta.get(), h.pmap.get(),
                       h.pg_u0.get(), h.u_t0.get(), h.pt_za.get(), h.pt_c.get(), F.cls_f.get(), F.fu_t0.get(),
                       F.ft_za.get(), F.ft_c.get(), F.pimg.get());
  }
  if (panel) {
    hipLaunchKernelGGL(k_fill_u32, dim3(grid_for(pull_words, 256, 4096)), dim3(256), 0, s,
                       reinterpret_cast<uint32_t*>(F.pull.get()), pull_words, kPanelZero | (kPanelZero << 16));
    hipLaunchKernelGGL(k_pull, dim3(pull_groups), dim3(64), 0, s, 1u, static_cast<uint32_t>(db), sp.n_orb, sp.n_beta,
                       F.n_tiles, sp.str_beta.get(), h.zpair.get(), pull_n.get(), pull_off.get(),
                       reinterpret_cast<uint16_t*>(F.pull.get()));
    F.panel = true;
  }
  PBS_HIP(hipGetLastError());
  PBS_HIP(hipStreamSynchronize(s));
  return plan;
}

}  // namespace pbs

using namespace pbs;

extern "C" {

pbs_status pbs_grouped_factor(pbs_grouped* h, const pbs_space* sp, void* stream) {
  return guarded([&] {
    PBS_REQUIRE(h != nullptr && sp != nullptr, PBS_ERR_ARG, "null handle");
    PBS_REQUIRE(sp->sector, PBS_ERR_ARG, "factored evaluation needs a spin-sector space");
    PBS_REQUIRE(h->has_sector && h->half == sp->n_orb, PBS_ERR_ARG, "operator lacks sector tables for this split");
    PBS_REQUIRE(h->real_coef, PBS_ERR_UNSUPPORTED, "factored evaluation needs real sector-form coefficients");
    h->fplan.reset();
    Scratch scratch(as_stream(stream));  // temporaries of this call
    h->fplan = make_factor_plan(*h, *sp, true, as_stream(stream));
  });
}

pbs_status pbs_grouped_set_factored(pbs_grouped* h, int32_t mode) {
  return guarded([&] {
    PBS_REQUIRE(h != nullptr, PBS_ERR_ARG, "null handle");
    PBS_REQUIRE(mode >= 0 && mode <= 7, PBS_ERR_ARG, "factored-evaluation mode must be 0..7");
    h->fact_on = static_cast<uint32_t>(mode);
  });
}

pbs_status pbs_grouped_factor_info(const pbs_grouped* h, uint32_t* info) {
  return guarded([&] {
    PBS_REQUIRE(h != nullptr && info != nullptr, PBS_ERR_ARG, "null argument");
    const FactorPlan* F = h->fplan.get();
    info[0] = F ? 1u : 0u;
    info[1] = F ? F->n_f1 : 0u;
    info[2] = F ? F->max_r1 : 0u;
    info[3] = F ? F->n_f2 : 0u;
    info[4] = F ? F->r2 : 0u;
    info[5] = F ? F->n_f3 : 0u;
    info[6] = F ? F->r3 : 0u;
    info[7] = F ? F->n_beta : 0u;
    info[8] = F && F->alist ? 1u : 0u;
    info[9] = F ? F->n_alpha : 0u;
    info[10] = F && F->plist ? 1u : 0u;
  });
}

}  // extern "C"
