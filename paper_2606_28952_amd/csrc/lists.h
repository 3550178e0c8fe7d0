// Lists kernel: sectors whose rows are too long for the sector kernel's staging,
// with few hops per spin (the 32-qubit Hubbard sector).
//
// Applies when every class is a simple class (alpha lists) or the X_alpha = 0
// class, whose groups other than the diagonal one are single-unique pair groups
// without alpha parities: then the pair groups' coefficients depend on the
// target column alone, and each column's valid ones are listed once per
// operator (FactorPlan::bl_*).
//
// A workgroup owns one target row.  The row itself is staged in LDS (103 KB for
// 12,870 single-precision columns), where the column lists gather from it; the
// alpha lists gather the same columns of other rows, coalesced; the diagonal
// group's folded coefficients become two 256-entry tables over the bytes of the
// target string.  Bound by the alpha gathers' way through the caches (17 rows
// read per row written): the 4 x 4 Hubbard sector in complex64 takes 3.74 ms, in
// which 25.5 GB come from behind L2 (6.9 TB/s); without the alpha gathers it
// takes 2.06 ms, without the column lists 3.63.  Evaluating
// every pair group per target with its rank lookup and phase sum, and gathering
// the row through L2 (the rows kernel), took 7.45 ms.  Loads issued where they
// are used, not ahead of the column's evaluation: 5.09 ms.
#pragma once

#include <type_traits>

#include "panel.h"
#include "sector.h"

namespace pbs {
namespace {

constexpr int kLB = 1024;
constexpr uint32_t kSlotsAhead = kListSlotsAhead;

struct ListsArgs {
  const uint32_t* bl_off;  // per 64 columns: first slot of four entries per column
  const void* bl_ent;      // [slot][64] of uint4, or of uint2 when narrow
  const double* bl_mag;    // distinct magnitudes
  uint32_t n_mag;
  uint32_t ua, ub;  // uniques of the diagonal group
  uint32_t off_tab, off_f, off_z, off_mag;  // LDS byte offsets; the row is at 0
};

// Workgroup w runs on XCD w mod 8.  Rows go out in windows of consecutive ones,
// kListsRun to an XCD: its L2 then sees source rows that neighbours share, and
// the memory-side cache one window's sources.  One contiguous range of rows per
// XCD keeps eight windows alive: 5.09 ms where plain order took 4.77 (both before
// loads were issued ahead); runs of 1 to 128 rows are within 1%.
constexpr uint32_t kListsRun = 32;
__device__ inline uint32_t lists_row_of(uint32_t w, uint32_t n) {
  constexpr uint32_t kWindow = kXcds * kListsRun;
  const uint32_t base = w / kWindow * kWindow, i = w % kWindow;
  return base + kWindow <= n ? base + i % kXcds * kListsRun + i / kXcds : w;
}

__device__ inline double with_sign(double v, uint32_t bit31) {
  return __longlong_as_double(__double_as_longlong(v) ^ (static_cast<long long>(static_cast<uint64_t>(bit31) << 32)));
}

// Four entries of a column: source columns, signs in bit 31, magnitude indexes.
// ONE: all magnitudes are equal, so an entry needs no lookup and 16 bits hold it.
template <bool ONE>
struct ColumnEntries;
template <>
struct ColumnEntries<true> {
  uint2 w;
  __device__ uint32_t source(int i) const { return ((i & 2 ? w.y : w.x) >> (i & 1 ? 16 : 0)) & 0x7fffu; }
  __device__ uint32_t sign(int i) const { return ((i & 2 ? w.y : w.x) << (i & 1 ? 0 : 16)) & 0x80000000u; }
  __device__ uint32_t mag(int) const { return 0; }
};
template <>
struct ColumnEntries<false> {
  uint4 w;
  __device__ uint32_t word(int i) const { return i == 0 ? w.x : i == 1 ? w.y : i == 2 ? w.z : w.w; }
  __device__ uint32_t source(int i) const { return word(i) & 0xffffu; }
  __device__ uint32_t sign(int i) const { return word(i) & 0x80000000u; }
  __device__ uint32_t mag(int i) const { return (word(i) >> 16) & 0x7fffu; }
};

template <class T, bool EXPVAL, bool ONE, bool QUEUED>
__global__ __launch_bounds__(kLB) void k_apply_lists(SectorArgs P, ListsArgs L, const T* __restrict__ psi,
                                                     T* __restrict__ out, double* __restrict__ partial,
                                                     const uint32_t* skip) {
  extern __shared__ __align__(16) unsigned char smem[];
  using Entries = ColumnEntries<ONE>;
  if (QUEUED && *skip) return;  // see Form
  const uint32_t row = lists_row_of(blockIdx.x, gridDim.x);
  const uint32_t ia = row + P.row_begin, db = P.dim_beta;
  T* s_row = reinterpret_cast<T*>(smem);  // [db + 1]: an absent entry reads the zero behind the row
  double* s_tab = reinterpret_cast<double*>(smem + L.off_tab);  // [2][256]
  double* s_F = reinterpret_cast<double*>(smem + L.off_f);
  uint32_t* s_Fz = reinterpret_cast<uint32_t*>(smem + L.off_z);
  double* s_mag = reinterpret_cast<double*>(smem + L.off_mag);
  const T* own = psi + static_cast<uint64_t>(ia) * db;
  const uint32_t ta = P.str_a[ia], nu = L.ub - L.ua;
  // the last wave folds first (a chain of dependent loads), the others start
  // with the row, all of it in flight at once
  if (threadIdx.x >= kLB - 64) fold_uniques<true>(P, L.ua, L.ub, ta, s_F, s_Fz, threadIdx.x - (kLB - 64), 64);
  constexpr uint32_t kStage = sizeof(T) > 8 ? 8 : 16;
  for (uint32_t i0 = threadIdx.x; i0 < db; i0 += kStage * kLB) {
    typedef uint32_t Raw __attribute__((ext_vector_type(sizeof(T) / 4), aligned(8)));
    Raw v[kStage];
#pragma unroll
    for (uint32_t k = 0; k < kStage; ++k) v[k] = reinterpret_cast<const Raw*>(own)[min(i0 + k * kLB, db - 1u)];
#pragma unroll
    for (uint32_t k = 0; k < kStage; ++k)
      if (i0 + k * kLB < db) reinterpret_cast<Raw*>(s_row)[i0 + k * kLB] = v[k];
  }
  if (threadIdx.x == 0) s_row[db] = T{};
  if (!ONE)
    for (uint32_t i = threadIdx.x; i < L.n_mag; i += kLB) s_mag[i] = L.bl_mag[i];
  __syncthreads();
  bool mixed = false;  // some diagonal mask has bits in both bytes
  if (threadIdx.x < 512) {
    const uint32_t byte = threadIdx.x & 255u, high = threadIdx.x >> 8;
    double f = 0.0;
    for (uint32_t u = 0; u < nu; ++u) {
      const uint32_t z = s_Fz[u], lo = z & 255u, hi = z >> 8;
      if (high ? (lo == 0u && hi != 0u) : hi == 0u) f += signed_by(s_F[u], __popc((high ? hi : lo) & byte));
    }
    s_tab[threadIdx.x] = f;
  }
  for (uint32_t u = 0; u < nu; ++u) mixed = mixed || ((s_Fz[u] & 255u) != 0u && (s_Fz[u] >> 8) != 0u);
  __syncthreads();

  const uint32_t a0 = ldc(P.alist_off + ia), a1 = ldc(P.alist_off + ia + 1);
  const double one = ONE ? ldc(L.bl_mag) : 0.0;
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t n_list = a1 - a0;
  double e_re = 0.0, e_im = 0.0, nrm = 0.0;
  // The row's columns with N gathers of the simple classes in flight, N even and
  // the list no shorter than N - 1: where it has N - 1 entries the first is loaded
  // again and left out of the sums, a longer list ends in a loop.
  // A column's entries are loaded first, then the gathers, which arrive while
  // the entries are evaluated: loads return in order.
  auto sweep = [&](auto ahead) {
    constexpr uint32_t N = decltype(ahead)::value;
    for (uint32_t c0 = __builtin_amdgcn_readfirstlane(threadIdx.x & ~63u); c0 < db; c0 += kLB) {
      const uint32_t col = c0 + lane;
      const bool live = col < db;
      const uint32_t colc = live ? col : db - 1u;
      const uint32_t tb = P.str_b[colc];
      const T* psi_col = psi + colc;
      double ar[4] = {0.0, 0.0, 0.0, 0.0}, ai[4] = {0.0, 0.0, 0.0, 0.0};
      const uint32_t q0 = ldc(L.bl_off + c0 / 64u), q1 = ldc(L.bl_off + c0 / 64u + 1u);
      const Entries* ent = static_cast<const Entries*>(L.bl_ent) + lane;
      Entries w[kSlotsAhead];
      T a[N > 0 ? N : 1];
#pragma unroll
      for (uint32_t i = 0; i < kSlotsAhead; ++i) w[i] = ent[static_cast<uint64_t>(q0 + i) * 64u];
      // (the list is read again for each column group: held in scalar registers
      // across the sweep, it spills, at a vector instruction per word)
      const uint32_t* src = P.alist_src + a0;
      const double* coef = P.alist_c + a0;
      asm volatile("" : "+s"(src), "+s"(coef));
#pragma unroll
      for (uint32_t i = 0; i < N; ++i)
        a[i] = psi_col[static_cast<uint64_t>(i + 1 < N || i < n_list ? ldc(src + i) : ldc(src)) * db];
      __builtin_amdgcn_sched_barrier(0);
      auto column = [&](const Entries& e) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const T v = s_row[e.source(i)];
          const double c = with_sign(ONE ? one : s_mag[e.mag(i)], e.sign(i));
          Coef<true>::mac(c, static_cast<double>(v.x), static_cast<double>(v.y), ar[i], ai[i]);
        }
      };
#pragma unroll
      for (uint32_t i = 0; i < kSlotsAhead; ++i)
        if (q0 + i < q1) column(w[i]);
      for (uint32_t q = q0 + kSlotsAhead; q < q1; ++q) column(ent[static_cast<uint64_t>(q) * 64u]);
      double f = s_tab[tb & 255u] + s_tab[256u + (tb >> 8)];
      if (mixed)
        for (uint32_t u = 0; u < nu; ++u) {
          const uint32_t z = s_Fz[u];
          if ((z & 255u) != 0u && (z >> 8) != 0u) f += signed_by(s_F[u], __popc(z & tb));
        }
      const T self = s_row[colc];
      const double pr = static_cast<double>(self.x), pi = static_cast<double>(self.y);
      Coef<true>::mac(f, pr, pi, ar[0], ai[0]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (uint32_t i = 0; i < N; ++i) {
        if (i + 1 == N && i >= n_list) break;
        Coef<true>::mac(ldc(coef + i), widen(a[i].x), widen(a[i].y), ar[i & 3], ai[i & 3]);
      }
      for (uint32_t e = a0 + N; e < a1; ++e) {
        const T v = psi_col[static_cast<uint64_t>(ldc(P.alist_src + e)) * db];
        Coef<true>::mac(ldc(P.alist_c + e), static_cast<double>(v.x), static_cast<double>(v.y), ar[1], ai[1]);
      }
      const double acc_r = (ar[0] + ar[1]) + (ar[2] + ar[3]);
      const double acc_i = (ai[0] + ai[1]) + (ai[2] + ai[3]);
      if (live) {
        if (EXPVAL) {
          e_re = fma(pr, acc_r, fma(pi, acc_i, e_re));
          e_im = fma(pr, acc_i, fma(-pi, acc_r, e_im));
          nrm = fma(pr, pr, fma(pi, pi, nrm));
        }
        if (!EXPVAL || out) Amp<T>::store(out, static_cast<uint64_t>(ia) * db + col, acc_r, acc_i);
      }
    }
  };
  constexpr uint32_t kAhead = sizeof(T) > 8 ? 12 : kListRowsAhead;  // (registers: 20 gathers of 16 bytes spill)
  switch ((min(n_list, kAhead) + 1u) / 2u) {
    case 0: sweep(std::integral_constant<uint32_t, 0>{}); break;
    case 1: sweep(std::integral_constant<uint32_t, 2>{}); break;
    case 2: sweep(std::integral_constant<uint32_t, 4>{}); break;
    case 3: sweep(std::integral_constant<uint32_t, 6>{}); break;
    case 4: sweep(std::integral_constant<uint32_t, 8>{}); break;
    case 5: sweep(std::integral_constant<uint32_t, 10>{}); break;
    case 6: sweep(std::integral_constant<uint32_t, 12>{}); break;
    case 7: sweep(std::integral_constant<uint32_t, kAhead < 14 ? 0 : 14>{}); break;
    case 8: sweep(std::integral_constant<uint32_t, kAhead < 16 ? 0 : 16>{}); break;
    case 9: sweep(std::integral_constant<uint32_t, kAhead < 18 ? 0 : 18>{}); break;
    default: sweep(std::integral_constant<uint32_t, kAhead < 20 ? 0 : 20>{}); break;
  }
  if (EXPVAL) block_reduce3_store<kLB>(e_re, e_im, nrm, partial + 3ull * row);
}

}  // namespace
}  // namespace pbs
