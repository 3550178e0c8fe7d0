// Panel kernel: the operator-state product of a factored two-body operator
// on the matrix cores (Section 2.4, Eqs. precomp_alpha, sreverse_sum).
//
// The mixed part of H (an alpha class X_alpha != 0 flipping two orbitals
// times a beta pair flip) is, for one target alpha row t_a,
//   out[t_a][j] += sum over moves m of j  s(m, j) V[pair(m)][j ^ X(m)],
//   V[pair][c]   = sum over classes e     img[e][pair] psi[t_a ^ X_e][c],
// where img holds the row's alpha images (every phase and coefficient folded
// per alpha string) and s the move's beta parity.  V is a dense product of a
// (pairs x classes) matrix with (classes x columns) source rows read
// straight from memory, so it runs on v_mfma_f64_16x16x4_f64 with float64
// operands and accumulation; only the second step gathers, and it gathers
// each move once per target instead of once per target and class.
//
// One workgroup of eight waves owns up to four alpha rows (two with 2,048 and
// more columns) and all their beta columns (a part of them in a launch of few
// rows, k_apply_panel_part), one workgroup per compute unit:
//  * X_alpha = 0 class: its beta-only part (pair and quad groups without
//    alpha Z-masks, a float64 coefficient per move and column) gathers from
//    the staged target rows, one table read for all of them; its diagonal
//    group through the F rows; what is left of its pair groups depends on t_a
//    and carries the parity of the orbital pair, so it joins V as one more
//    class whose source row is the target row;
//  * simple classes through the alpha lists (whole source rows, coalesced,
//    read once for all rows of the workgroup);
//  * then row by row the X_beta = 0 groups of the image classes through their
//    two F rows, and V in tiles of kPanelTile columns: wave w computes the 16
//    columns w & 3 of the 16-pair tiles 2t + (w >> 2), the row's image matrix
//    in LDS, the next tile's source columns loading behind the products.  The
//    tile goes to LDS, and while the next one is computed every lane adds the
//    entries that its targets read from it, listed per sector in a table
//    (k_pull in factor.hip) that all rows share.
// Each output is summed by one thread in an order that does not depend on
// the split into workgroups: no atomics, results are bitwise reproducible.
//
// What bounds it at 28 qubits (3,432 x 3,432, 50 classes, 91 pairs; complex64,
// 10.3 ms against 17.1 for the sector kernel; complex128 at 26 qubits 2.06
// against 3.39): V's 96 x 52 x D products are 235 GFLOP, 3.3 ms at the 73
// TFLOP/s that float64 matrix instructions reach here, and take 4.0 ms, the
// gathers 0.7 (the sparse form, 49 moves x 49 classes per target, is 113
// GFLOP but two 8-byte LDS reads for each: 10 ms in the sector kernel); the
// alpha lists 2.8 ms for 40 GB past L1 (of which 23 GB miss L2), the beta-only
// part 1.7 ms for 29 GB of table (3.2 ms with one row per workgroup), the
// X_beta = 0 groups 0.8.
#pragma once

#include "sector.h"

namespace pbs {
namespace {

constexpr int kPB = static_cast<int>(kPanelLanes);
constexpr int kPW = kPB / 64;                                    // waves

struct PanelArgs {
  uint32_t dim_alpha, dim_beta, n_tiles;
  uint32_t row_begin, rows;  // target rows of the launch
  uint32_t n_blk;            // blocks that split them evenly
  uint32_t n_img, n_pairs, n_bb, diag_rank;
  uint64_t diag_off;  // of the diagonal group's F rows in fz (doubles)
  const uint32_t* alist_off;
  const uint32_t* alist_src;
  const double* alist_c;
  const uint32_t* plist_off;
  const uint32_t* plist_src;
  const uint32_t* plist_cls;
  const double* pimg;
  const double* c0img;   // [dim_alpha][n_pairs]
  const double* diag_a;  // [dim_alpha][diag_rank]
  const uint4* cls_f;
  const double* fz;
  const uint32_t* bb_src;  // [ceil(n_bb / 2)][dim_beta]: source columns of moves 2i, 2i + 1
  const double* bb_c;      // [n_bb][dim_beta]
  const uint4* pull;         // per tile, wave and target group: slots of 64 two-byte entries
  const uint4* pull_cnt;     // [n_tiles][waves]: slots per target group (a byte each, x and y), first slot of the
                             // wave in its tile (z), first slot of the tile (w)
};

typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// An amplitude widened where it is used: left to itself the compiler widens
// each one as soon as it arrives, and waits for it there.
__device__ __forceinline__ double widen(float v) {
  double d;
  asm volatile("v_cvt_f64_f32 %0, %1" : "=v"(d) : "v"(v));
  return d;
}
__device__ __forceinline__ double widen(double v) {
  asm volatile("" : "+v"(v));
  return v;
}

// The same for operands of a matrix instruction, which must not read a register
// in the two wait states after a vector instruction wrote it: the compiler keeps
// that distance for instructions it knows, not for one inside an asm, so the asm
// waits itself.
__device__ __forceinline__ double widen_operand(float v) {
  double d;
  asm volatile("v_cvt_f64_f32 %0, %1\n\ts_nop 1" : "=v"(d) : "v"(v));
  return d;
}
__device__ __forceinline__ double widen_operand(double v) { return widen(v); }

// Software pipeline over entries 0 .. n - 1: the loads of D - 1 entries are in
// flight while one is evaluated (past the end the last entry is loaded again).
template <int D, class B, class L, class E>
__device__ __forceinline__ void pipelined(uint32_t n, B (&buf)[D], const L& load, const E& eval) {
  if (n == 0) return;
#pragma unroll
  for (int d = 0; d + 1 < D; ++d) load(min(static_cast<uint32_t>(d), n - 1u), buf[d]);
  for (uint32_t e = 0; e < n; e += D) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
      load(min(e + d + D - 1u, n - 1u), buf[(d + D - 1) % D]);
      __builtin_amdgcn_sched_barrier(0);  // the buffers' loads stay in order
      eval(e + d, buf[d]);
      if (e + d + 1 >= n) return;
    }
  }
}

// Target alpha rows ia .. ia + nr - 1 (nr <= R); the energy partials of row
// ia + r go to slot + 3 r.  NT: target columns per lane and row (dim_beta <=
// NT kPB); MT: 16-pair tiles per wave (n_pairs <= 32 MT); KS: K steps of four
// classes (at most 4 KS - 1 image classes per row).
// Args: PanelArgs, as kernel argument or in the constant address space.
// QUEUED: nothing is done when *stop is not zero.  PART: of the row's groups of
// kPB columns, those from j0 on (else all, j0 = 0).
template <class T, bool EXPVAL, int NT, int MT, int KS, int R, bool QUEUED, bool PART, class Args>
__device__ __forceinline__ void panel_body(const Args& P, const T* __restrict__ psi, T* __restrict__ out,
                                           double* __restrict__ slot, uint32_t ia, uint32_t nr,
                                           const uint32_t* stop, uint32_t j0) {
  extern __shared__ __align__(16) unsigned char smem[];
  const uint32_t tid = threadIdx.x, lane = tid & 63u;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t db = P.dim_beta;
  double ar[R][NT], ai[R][NT];
  uint32_t cb[NT];  // this lane's target columns (the last one repeated past the end)
#pragma unroll
  for (int j = 0; j < NT; ++j) {
#pragma unroll
    for (int r = 0; r < R; ++r) ar[r][j] = ai[r][j] = 0.0;
    cb[j] = min(tid + (j0 + j) * kPB, db - 1u);
  }

  // X_alpha = 0: kS rows staged side by side, so that one table entry and
  // one gather serve them all
  constexpr int kS = sizeof(T) == 8 || R == 1 ? R : 2;
  constexpr int kH = NT > 4 ? (NT + 1) / 2 : NT;  // the lane's columns in two parts: fewer registers in flight
  T* s_st = reinterpret_cast<T*>(smem);
#pragma unroll
  for (int g = 0; g < R; g += kS) {
    if (static_cast<uint32_t>(g) >= nr) break;
    if (g) __syncthreads();
#pragma unroll
    for (int r = 0; r < kS; ++r)
      if (static_cast<uint32_t>(g + r) < nr) {
        const T* rowg = psi + static_cast<uint64_t>(ia + g + r) * db;
        for (uint32_t c = tid; c < db; c += kPB) s_st[c * kS + r] = rowg[c];
      }
    const bool skip = QUEUED && g == 0 && *stop != 0;
    __syncthreads();
    if (skip) return;
    // beta-only part, two moves per step, the next two loading
    auto gather = [&](uint32_t col, double c, int j) {
#pragma unroll
      for (int r = 0; r < kS; r += 2)
        if (static_cast<uint32_t>(g + r) < nr) {
          constexpr int kPair = kS > 1 ? 1 : 0;
          double x0, y0, x1, y1;
          Amp<T>::load(s_st, col * kS + r, x0, y0);
          if (kPair) Amp<T>::load(s_st, col * kS + r + kPair, x1, y1);
          Coef<true>::mac(c, x0, y0, ar[g + r][j], ai[g + r][j]);
          if (kPair) Coef<true>::mac(c, x1, y1, ar[g + r + kPair][j], ai[g + r + kPair][j]);
        }
    };
    struct Moves {
      uint32_t s[kH];
      double c0[kH], c1[kH];
    } moves[2];
    const uint32_t n2 = P.n_bb / 2u;
#pragma unroll
    for (int h = 0; h < NT; h += kH) {
      auto load = [&](uint32_t i, Moves& b) {
        const uint32_t* sp = P.bb_src + static_cast<uint64_t>(i) * db;
        const double* cp = P.bb_c + static_cast<uint64_t>(2u * i) * db;
#pragma unroll
        for (int j = 0; j < kH; ++j)
          if (h + j < NT) {
            b.s[j] = sp[cb[h + j]];
            b.c0[j] = cp[cb[h + j]];
            b.c1[j] = (cp + db)[cb[h + j]];
          }
      };
      auto eval = [&](uint32_t, const Moves& b) {
#pragma unroll
        for (int j = 0; j < kH; ++j)
          if (h + j < NT) {
            gather(b.s[j] & 0xffffu, widen(b.c0[j]), h + j);
            gather(b.s[j] >> 16, widen(b.c1[j]), h + j);
          }
      };
      pipelined(n2, moves, load, eval);
    }
    if (P.n_bb & 1u) {
#pragma unroll
      for (int j = 0; j < NT; ++j)
          gather(P.bb_src[static_cast<uint64_t>(n2) * db + cb[j]] & 0xffffu,
                 P.bb_c[static_cast<uint64_t>(2u * n2) * db + cb[j]], j);
    }
    // diagonal group: sum_k A_k(t_a) F_k(column)
    if (P.diag_rank) {
#pragma unroll
      for (int r = 0; r < kS; ++r)
        if (static_cast<uint32_t>(g + r) < nr) {
          double f[NT];
#pragma unroll
          for (int j = 0; j < NT; ++j) f[j] = 0.0;
#pragma unroll 4
          for (uint32_t k = 0; k < P.diag_rank; ++k) {
            const double a = ldc(P.diag_a + static_cast<uint64_t>(ia + g + r) * P.diag_rank + k);
            const double* fr = P.fz + P.diag_off + static_cast<uint64_t>(k) * db;
#pragma unroll
            for (int j = 0; j < NT; ++j)
              f[j] = fma(a, fr[cb[j]], f[j]);
          }
#pragma unroll
          for (int j = 0; j < NT; ++j)
            {
              double x, y;
              Amp<T>::load(s_st, cb[j] * kS + r, x, y);
              Coef<true>::mac(f[j], x, y, ar[g + r][j], ai[g + r][j]);
            }
        }
    }
  }

  // simple classes: the rows' lists scattered over the source rows, then the
  // source rows that any list names in ascending order (the workgroups in
  // flight sweep them together, so they meet in L2)
  {
    const uint32_t da = P.dim_alpha;
    double* s_c = reinterpret_cast<double*>(smem);  // [R][da]
    uint32_t* s_src = reinterpret_cast<uint32_t*>(smem + 8ull * R * da);
    uint32_t* s_cnt = s_src + da;  // one count per wave
    __syncthreads();
    for (uint32_t i = tid; i < R * da; i += kPB) s_c[i] = 0.0;
    for (uint32_t i = tid; i < da; i += kPB) s_src[i] = 0u;
    __syncthreads();
    for (uint32_t r = 0; r < nr; ++r) {
      const uint32_t a0 = ldc(P.alist_off + ia + r), a1 = ldc(P.alist_off + ia + r + 1);
      for (uint32_t i = a0 + tid; i < a1; i += kPB) {
        const uint32_t src = P.alist_src[i];  // at most once per row
        s_c[r * da + src] = P.alist_c[i];
        s_src[src] |= 1u << r;  // rows are taken one after the other
      }
      __syncthreads();
    }
    uint32_t n = 0;
    for (uint32_t i0 = 0; i0 < da; i0 += kPB) {
      const uint32_t i = i0 + tid;
      const uint32_t m = i < da ? s_src[i] : 0u;
      const uint64_t bal = __ballot(m != 0u);
      if (lane == 0) s_cnt[wave] = static_cast<uint32_t>(__popcll(bal));
      __syncthreads();  // and every mask of this step is read
      uint32_t at = n, total = 0;
      for (uint32_t w = 0; w < kPW; ++w) {
        at += w < wave ? s_cnt[w] : 0u;
        total += s_cnt[w];
      }
      if (m) s_src[at + static_cast<uint32_t>(__popcll(bal & ((1ull << lane) - 1ull)))] = i | (m << 24);
      n += total;
      __syncthreads();
    }
    // the list is read 64 entries at a time, one per lane
    struct Rows {
      T a[kH];
      double c[R];
      uint32_t rows;
    } list[4];
#pragma unroll
    for (int h = 0; h < NT; h += kH) {
      uint32_t mine = 0;
      auto load = [&](uint32_t e, Rows& b) {  // entries in order, from 0
        if ((e & 63u) == 0u) mine = s_src[min(e + lane, n - 1u)];
        const uint32_t w = __builtin_amdgcn_readlane(mine, e & 63u), src = w & 0xffffffu;
        const T* p = psi + static_cast<uint64_t>(src) * db;
#pragma unroll
        for (int r = 0; r < R; ++r) b.c[r] = s_c[r * da + src];
#pragma unroll
        for (int j = 0; j < kH; ++j)
          if (h + j < NT) b.a[j] = p[cb[h + j]];
        b.rows = w >> 24;
      };
      auto eval = [&](uint32_t, const Rows& b) {
        double xr[kH], xi[kH];
#pragma unroll
        for (int j = 0; j < kH; ++j)
          if (h + j < NT) {
            xr[j] = widen(b.a[j].x);
            xi[j] = widen(b.a[j].y);
          }
#pragma unroll
        for (int r = 0; r < R; ++r)
          if ((b.rows >> r) & 1u) {
#pragma unroll
            for (int j = 0; j < kH; ++j)
              if (h + j < NT) Coef<true>::mac(b.c[r], xr[j], xi[j], ar[r][h + j], ai[r][h + j]);
          }
      };
      pipelined(n, list, load, eval);
    }
  }

  // mixed part, row by row
  double2* s_v = reinterpret_cast<double2*>(smem);
  double* s_a = reinterpret_cast<double*>(smem + kPanelVBytes);           // [2 MT][KS][64]
  uint32_t* s_so = reinterpret_cast<uint32_t*>(s_a + 2 * MT * KS * 64);  // source row offsets, [4 KS]
  uint32_t* s_rk = s_so + 4 * KS;                                          // X_beta = 0 rank
  uint64_t* s_fo = reinterpret_cast<uint64_t*>(s_rk + 4 * KS);             // its F rows
  double2* s_fa = reinterpret_cast<double2*>(s_fo + 4 * KS);               // its folded factors
  static_assert(kPanelPullSlots * 128u == 2u * 16u * kPB, "two steps of 16 bytes per lane");
  u32x4* s_pull = reinterpret_cast<u32x4*>(smem + kPanelMixBytes);           // the tile's entries
  const uint32_t quarter = wave & 3u, mh = wave >> 2, n16 = lane & 15u, k4 = lane >> 4;
  for (uint32_t r = 0; r < nr; ++r) {
    const uint32_t row = ia + r;
    const uint32_t i0 = ldc(P.plist_off + row), n_e = ldc(P.plist_off + row + 1) - i0;
    __syncthreads();
    for (uint32_t i = tid; i < 2u * MT * KS * 64u; i += kPB) {
      const uint32_t l = i & 63u, k = (i >> 6) % KS, t = (i >> 6) / KS;
      const uint32_t e = 4u * k + (l >> 4), pair = t * 16u + (l & 15u);
      double v = 0.0;
      if (pair < P.n_pairs) {
        if (e < n_e) v = P.pimg[static_cast<uint64_t>(i0 + e) * P.n_img + pair];
        if (e == n_e) v = P.c0img[static_cast<uint64_t>(row) * P.n_pairs + pair];
      }
      s_a[i] = v;
    }
    if (tid < 4 * KS) {
      s_so[tid] = (tid < n_e ? P.plist_src[i0 + tid] : row) * db;
      if (tid < n_e) {
        const uint4 cf = P.cls_f[P.plist_cls[i0 + tid]];
        const double* im = P.pimg + static_cast<uint64_t>(i0 + tid) * P.n_img + P.n_pairs + 1u;
        s_rk[tid] = cf.y;
        s_fo[tid] = cf.z | (static_cast<uint64_t>(cf.w) << 32);
        s_fa[tid] = make_double2(im[0], cf.y > 1 ? im[1] : 0.0);
      }
    }
    if (tid == 0) s_v[kPanelZero] = make_double2(0.0, 0.0);
    __syncthreads();
    // X_beta = 0 groups of the image classes
    {
      struct Zero {
        T x[kH];
        double f0[kH], f1[kH];
      } zero[2];
#pragma unroll
      for (int h = 0; h < NT; h += kH) {
        auto load = [&](uint32_t e, Zero& z) {
          const uint64_t fo = s_fo[e];
          const double* f0 =
              P.fz + ((static_cast<uint64_t>(__builtin_amdgcn_readfirstlane(static_cast<uint32_t>(fo >> 32))) << 32) |
                      static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<uint32_t>(fo))));
          // with one factor (or none) the second read repeats the first
          const double* f1 = f0 + (__builtin_amdgcn_readfirstlane(s_rk[e]) > 1u ? db : 0u);
          const T* p = psi + __builtin_amdgcn_readfirstlane(s_so[e]);
#pragma unroll
          for (int j = 0; j < kH; ++j)
            if (h + j < NT) {
              z.x[j] = p[cb[h + j]];
              z.f0[j] = f0[cb[h + j]];
              z.f1[j] = f1[cb[h + j]];
            }
        };
        auto eval = [&](uint32_t e, const Zero& z) {
          if (__builtin_amdgcn_readfirstlane(s_rk[e]) == 0u) return;
          const double2 a = s_fa[e];
#pragma unroll
          for (int j = 0; j < kH; ++j)
            if (h + j < NT)
              Coef<true>::mac(fma(a.x, widen(z.f0[j]), a.y * widen(z.f1[j])), widen(z.x[j].x), widen(z.x[j].y),
                              ar[0][h + j], ai[0][h + j]);
        };
        pipelined(n_e, zero, load, eval);
      }
    }

    // V tile by tile: the products of tile t + 1 run while tile t is gathered
    T b[KS];
    auto load = [&](uint32_t tile, int k) {
      b[k] = psi[s_so[4 * k + k4] + min(tile * kPanelTile + quarter * 16u + n16, db - 1u)];
    };
#pragma unroll
    for (int k = 0; k < KS; ++k) load(0, k);
    const double* my_a = s_a + mh * (KS * 64u) + lane;  // tile 2t + mh, step k: at (2t KS + k) 64
    // entries of the tile in LDS, read four slots at a time
    uint4 cw = make_uint4(0u, 0u, 0u, 0u);
    uint32_t at = 0;  // byte offset of this lane's next entry
    auto pull = [&](int j) {
      const uint32_t jg = PART ? j0 + j : static_cast<uint32_t>(j);
      const uint32_t n = ((jg < 4 ? cw.x : cw.y) >> (8 * (jg & 3))) & 255u;
      for (uint32_t i = 0; i < n; i += kPanelPullRead) {
        uint32_t e[kPanelPullRead];
        double2 v[kPanelPullRead];
#pragma unroll
        for (uint32_t q = 0; q < kPanelPullRead; ++q)
          e[q] = *reinterpret_cast<const uint16_t*>(smem + kPanelMixBytes + at + 128u * q);
#pragma unroll
        for (uint32_t q = 0; q < kPanelPullRead; ++q) v[q] = s_v[i + q < n ? e[q] & 0x1fffu : kPanelZero];
#pragma unroll
        for (uint32_t q = 0; q < kPanelPullRead; ++q) {
          ar[0][j] += signed_by_bit31(v[q].x, e[q] << 16);
          ai[0][j] += signed_by_bit31(v[q].y, e[q] << 16);
        }
        at += 128u * min(n - i, kPanelPullRead);
      }
    };
    // the slots of the groups before j0 in a wave's list of a tile
    auto before = [&](const uint4& c) {
      uint32_t n = 0;
      if (PART)
        for (uint32_t j = 0; j < j0; ++j) n += ((j < 4 ? c.x : c.y) >> (8 * (j & 3))) & 255u;
      return n;
    };
    auto counts = [&](uint32_t tile) {
      const uint32_t* c = reinterpret_cast<const uint32_t*>(P.pull_cnt + tile * kPW + wave);
      return make_uint4(ldc(c), ldc(c + 1), ldc(c + 2), ldc(c + 3));
    };
    uint4 next = counts(0);
    for (uint32_t tile = 0; tile < P.n_tiles; ++tile) {
      const uint4 cn = next;
      // this tile's entries, 16 bytes per lane and step, stored with the tile
      const u32x4* ps = reinterpret_cast<const u32x4*>(P.pull) + static_cast<uint64_t>(cn.w) * 8u + tid;
      const u32x4 pe0 = ps[0], pe1 = ps[kPB];
      next = counts(min(tile + 1, P.n_tiles - 1u));
      f64x4 vr[MT], vi[MT];
      double av[MT];
#pragma unroll
      for (int t = 0; t < MT; ++t) {
        vr[t] = vi[t] = f64x4{0.0, 0.0, 0.0, 0.0};
        av[t] = my_a[2 * t * KS * 64];
      }
#pragma unroll
      for (int k = 0; k < KS; ++k) {
        // classes past the end hold the target row, which the X_alpha = 0
        // class reads too, against zeros
        const double xr = widen_operand(b[k].x), xi = widen_operand(b[k].y);
        load(tile + 1, k);
        double cur[MT];
#pragma unroll
        for (int t = 0; t < MT; ++t) {
          cur[t] = av[t];
          if (k + 1 < KS) av[t] = my_a[(2 * t * KS + k + 1) * 64];
        }
#pragma unroll
        for (int t = 0; t < MT; ++t) {
          vr[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(cur[t], xr, vr[t], 0, 0, 0);
          vi[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(cur[t], xi, vi[t], 0, 0, 0);
        }
        if (k < NT) pull(k);
      }
      __syncthreads();  // the previous tile is gathered
      cw = cn;
      at = (cn.z + before(cn)) * 128u + lane * 2u;
      s_pull[tid] = pe0;
      s_pull[kPB + tid] = pe1;
#pragma unroll
      for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          s_v[((2u * t + mh) * 16u + 4u * i + k4) * kPanelTile + quarter * 16u + n16] =
              make_double2(vr[t][i], vi[t][i]);
      __syncthreads();
    }
#pragma unroll
    for (int j = 0; j < NT; ++j) pull(j);

    // the row is complete: store it, move the next row's sums down
    double e_re = 0.0, e_im = 0.0, nrm = 0.0;
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      const uint32_t col = tid + (j0 + j) * kPB;
      if (col < db) {
        const uint64_t t = static_cast<uint64_t>(row) * db + col;
        if (EXPVAL) {
          double pr, pi;
          Amp<T>::load(psi, t, pr, pi);
          e_re = fma(pr, ar[0][j], fma(pi, ai[0][j], e_re));
          e_im = fma(pr, ai[0][j], fma(-pi, ar[0][j], e_im));
          nrm = fma(pr, pr, fma(pi, pi, nrm));
        }
        if (!EXPVAL || out) Amp<T>::store(out, t, ar[0][j], ai[0][j]);
      }
#pragma unroll
      for (int q = 0; q + 1 < R; ++q) {
        ar[q][j] = ar[q + 1][j];
        ai[q][j] = ai[q + 1][j];
      }
    }
    if (EXPVAL) {
      __syncthreads();
      block_reduce3_store<kPB>(e_re, e_im, nrm, slot + 3ull * r, reinterpret_cast<double(*)[kPW]>(smem));
    }
  }
}

// Row block of workgroup w of n: workgroup w runs on XCD w mod 8, and an XCD
// takes consecutive blocks, whose rows name similar source rows.
__device__ inline uint32_t panel_block_of(uint32_t w, uint32_t n) {
  const uint32_t per = n / kXcds;
  return w < per * kXcds ? w % kXcds * per + w / kXcds : w;
}

// Workgroup w: one of the n_blk row blocks that split the launch's rows evenly.
template <class T, bool EXPVAL, int NT, int MT, int KS, int R, bool QUEUED>
__global__ __launch_bounds__(kPB) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_apply_panel(
    PanelArgs P, const T* __restrict__ psi, T* __restrict__ out, double* __restrict__ partial, const uint32_t* skip) {
  const uint64_t b = panel_block_of(blockIdx.x, gridDim.x);
  const uint32_t r0 = static_cast<uint32_t>(b * P.rows / P.n_blk);
  const uint32_t r1 = static_cast<uint32_t>((b + 1) * P.rows / P.n_blk);
  // (no block is empty, but without the test the compiler places 30 more register
  // moves in the body: 28 qubits, complex64, 10.31 ms without, 10.29 with it)
  if (r1 > r0)
    panel_body<T, EXPVAL, NT, MT, KS, R, QUEUED, false>(P, psi, out, partial + 3ull * r0, P.row_begin + r0, r1 - r0,
                                                        skip, 0);
}

// Launches of few rows (a share of a sector): `parts` workgroups per row, NT
// groups of kPB columns each, so that a short launch fills more of the device.
// Every part computes the row's V for itself; the rest of its work is its own
// columns'.  Outputs have the same bits (nothing is summed across columns).  16 of
// the 3,432 rows of 28 qubits, complex64: 1.35 ms with two rows per workgroup,
// 0.82 with one, 0.45 in seven parts; 128 of the 924 rows of (12; 6, 6): 0.63 with
// four, 0.23 with one, 0.15 in two parts (the sector kernel: 0.29 and 0.15).
template <class T, bool EXPVAL, int NT, int MT, int KS>
__global__ __launch_bounds__(kPB) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_apply_panel_part(
    PanelArgs P, const T* __restrict__ psi, T* __restrict__ out, double* __restrict__ partial, uint32_t parts) {
  const uint32_t b = panel_block_of(blockIdx.x, gridDim.x), row = b / parts;
  panel_body<T, EXPVAL, NT, MT, KS, 1, false, true>(P, psi, out, partial + 3ull * b, P.row_begin + row, 1, nullptr,
                                                    (b - row * parts) * NT);
}

// A job of a batched launch of one panel variant.
struct PanelJob {
  PanelArgs args;  // every row
  const void* psi;
  void* out;
  uint32_t block_base;  // first work item of the job
  uint32_t first;       // its first energy partial (one per row)
};

// Work item w (one row block of one job) belongs to the job with the largest
// block_base <= w; a persistent launch walks the items with the grid's stride.
template <class T, bool EXPVAL, int NT, int MT, int KS, int R>
__global__ __launch_bounds__(kPB) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_apply_panel_batch(
    const PanelJob* __restrict__ jobs, uint32_t n_jobs, uint32_t n_items, double* __restrict__ partial) {
  typedef const __attribute__((address_space(4))) PanelJob ConstJob;
  for (uint32_t w = blockIdx.x; w < n_items; w += gridDim.x) {
    if (w != blockIdx.x) __syncthreads();  // the previous item is done with LDS
    uint32_t lo = 0, hi = n_jobs;
    while (hi - lo > 1) {
      const uint32_t mid = (lo + hi) / 2;
      if (ldc(&jobs[mid].block_base) <= w)
        lo = mid;
      else
        hi = mid;
    }
    ConstJob& J = *(ConstJob*)(jobs + lo);
    const uint64_t b = panel_block_of(w - J.block_base, J.args.n_blk);
    const uint32_t r0 = static_cast<uint32_t>(b * J.args.rows / J.args.n_blk);
    const uint32_t r1 = static_cast<uint32_t>((b + 1) * J.args.rows / J.args.n_blk);
    panel_body<T, EXPVAL, NT, MT, KS, R, false, false>(J.args, static_cast<const T*>(J.psi), static_cast<T*>(J.out),
                                                       partial + 3ull * (J.first + r0), r0, r1 - r0, nullptr, 0);
  }
}

template <class T, int NT, int MT, int KS, int R>
void* panel_variant(bool expval, Form form) {
  if (form == Form::kBatch)
    return expval ? reinterpret_cast<void*>(k_apply_panel_batch<T, true, NT, MT, KS, R>)
                  : reinterpret_cast<void*>(k_apply_panel_batch<T, false, NT, MT, KS, R>);
  if (form == Form::kQueued) return reinterpret_cast<void*>(k_apply_panel<T, false, NT, MT, KS, R, true>);
  return expval ? reinterpret_cast<void*>(k_apply_panel<T, true, NT, MT, KS, R, false>)
                : reinterpret_cast<void*>(k_apply_panel<T, false, NT, MT, KS, R, false>);
}

// NT of a part: one group of columns, or two.
template <class T, int MT, int KS>
void* panel_part_variant(bool expval, bool two) {
  if (two)
    return expval ? reinterpret_cast<void*>(k_apply_panel_part<T, true, 2, MT, KS>)
                  : reinterpret_cast<void*>(k_apply_panel_part<T, false, 2, MT, KS>);
  return expval ? reinterpret_cast<void*>(k_apply_panel_part<T, true, 1, MT, KS>)
                : reinterpret_cast<void*>(k_apply_panel_part<T, false, 1, MT, KS>);
}

}  // namespace

// Kernel of a shape (PanelShape::variant); each storage type and half of the
// variants is defined in its own translation unit (panel_<storage>_<width>.hip).
void* panel_kernel_c64_narrow(bool expval, Form form, int variant);
void* panel_kernel_c64_wide(bool expval, Form form, int variant);
void* panel_kernel_c128_narrow(bool expval, Form form, int variant);
void* panel_kernel_c128_wide(bool expval, Form form, int variant);

// Kernel of a part of a row, for the variants of several groups of columns
// (panel_<storage>_part.hip).
void* panel_part_c64(bool expval, bool two, int variant);
void* panel_part_c128(bool expval, bool two, int variant);

inline void* panel_part(pbs_dtype dt, bool expval, bool two, int variant) {
  return dt == PBS_C128 ? panel_part_c128(expval, two, variant) : panel_part_c64(expval, two, variant);
}

inline void* panel_kernel(pbs_dtype dt, bool expval, Form form, int variant) {
  if (variant >= kPanelWide)
    return dt == PBS_C128 ? panel_kernel_c128_wide(expval, form, variant)
                          : panel_kernel_c64_wide(expval, form, variant);
  return dt == PBS_C128 ? panel_kernel_c128_narrow(expval, form, variant)
                        : panel_kernel_c64_narrow(expval, form, variant);
}

}  // namespace pbs
