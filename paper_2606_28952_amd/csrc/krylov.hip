// Real-time propagation psi <- exp(-i H dt) psi by short-iterative Lanczos
// (Section 2.1, Eq. real_time_evolution; the paper lists Krylov propagation
// among the consumers of the operator engine without fixing an algorithm, so
// this is the textbook method of Park and Light, 1986).
//
// Device work per Lanczos vector: one operator-state product (the sector or
// full-space apply), the three-term recurrence (alpha_j from one dot with the
// newest vector) followed by one full pass of classical Gram-Schmidt against
// all basis vectors (two multi-axpy sweeps: the first subtracts the
// recurrence terms and returns the projections, the second subtracts those
// and returns the norm), and a scale.  Inner products accumulate in float64 with a fixed-order two-stage
// reduction (deterministic).  Norms, alpha, beta and the coefficients of the
// sweeps stay on the device (LanczosState), so all m vectors are queued
// without a wait: at 24 qubits in double precision (0.85 M amplitudes, m = 12)
// the 37 round trips to the host took 1.1 ms of a 3.06 ms step.  A run that
// ends early (zero norm, breakdown) sets a flag that turns the queued kernels
// into empty ones.  The k x k tridiagonal matrix (k <= 16) is
// diagonalised on the host by cyclic Jacobi rotations and exp(-i T dt) e_1
// combines the basis vectors on the device.
#include <cmath>

#include "handles.h"

namespace pbs {
// the apply launcher lives in apply.hip; nothing is done when *skip is not zero
void apply_launch(const pbs_grouped& h, const pbs_space& sp, pbs_dtype dt, const void* psi, void* out, hipStream_t s,
                  const uint32_t* skip);

namespace {

constexpr int kKB = 256;
constexpr int kMaxK = 16;
constexpr unsigned kKGrid = 4096;  // up to 16 waves per SIMD for the streaming kernels

template <class T>
struct KAmp;
template <>
struct KAmp<double2> {
  __device__ static inline double2 ld(const double2* p, uint64_t i) { return p[i]; }
  __device__ static inline void st(double2* p, uint64_t i, double r, double m) { p[i] = make_double2(r, m); }
  // the value st() stores, read back as float64
  __device__ static inline double2 stored(double r, double m) { return make_double2(r, m); }
};
template <>
struct KAmp<float2> {
  __device__ static inline double2 ld(const float2* p, uint64_t i) {
    const float2 v = p[i];
    return make_double2(v.x, v.y);
  }
  __device__ static inline void st(float2* p, uint64_t i, double r, double m) {
    p[i] = make_float2(static_cast<float>(r), static_cast<float>(m));
  }
  __device__ static inline double2 stored(double r, double m) {
    return make_double2(static_cast<float>(r), static_cast<float>(m));
  }
};

struct Coeffs {
  double re[kMaxK];
  double im[kMaxK];
};

// What a step keeps on the device between its kernels.
struct LanczosState {
  Coeffs c;                           // coefficients of the next sweep
  double alpha[kMaxK], beta[kMaxK];
  double nrm, scale, last_b, inv;     // |psi|; largest |alpha|, b so far; last b; 1 / (norm to divide by)
  uint32_t k, done;                   // vectors so far; the run has ended
};

// Blocks of the kernels that end in a reduction.  Each thread sums several
// elements before its block reduces (24 sums by shuffles at 12 vectors).  A
// step of 12 vectors of 0.85 M double-precision amplitudes takes 2520 us with an
// element per thread (3336 blocks), 2166 with 2048 blocks, 1984 with 1024, 1881
// with 512 and 1829 with 256.  Large states do not miss the blocks: a step of
// 165.6 M amplitudes takes 264.8 ms in complex128 with 512, 267.9 with 1024, 269.3
// with 2048, and 117.9, 115.7, 120.1 in complex64; of 35 M in complex128 42.9, 44.0,
// 44.8; of 4.1 M in complex64 5.98, 5.95, 6.15.
constexpr unsigned kDotGrid = 512;

// Block partials of ND complex sums held by every thread (ar, ai):
// partial[(2i + {0,1}) * blocks + b], wave shuffles then a fixed-order sum over
// the block's waves.
template <int ND>
__device__ inline void block_partials(const double (&ar)[ND], const double (&ai)[ND], double* __restrict__ partial) {
  __shared__ double red[2 * ND][kKB / 64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int i = 0; i < ND; ++i) {
    double a = ar[i], b = ai[i];
    for (int d = 32; d > 0; d >>= 1) {
      a += __shfl_xor(a, d, 64);
      b += __shfl_xor(b, d, 64);
    }
    if (lane == 0) {
      red[2 * i][wave] = a;
      red[2 * i + 1][wave] = b;
    }
  }
  __syncthreads();
  if (threadIdx.x < 2 * ND) {
    double s = 0.0;
    for (int w = 0; w < kKB / 64; ++w) s += red[threadIdx.x][w];
    partial[static_cast<uint64_t>(threadIdx.x) * gridDim.x + blockIdx.x] = s;
  }
}

// Block partials (2i, 2i + 1) of conj(x_i) * y.
// The vector count is a template argument so that the kernel holds exactly
// NV accumulator pairs (registers, hence resident waves, follow NV).
template <class T, int NV>
__global__ __launch_bounds__(kKB) void k_multidot(uint64_t n, const T* __restrict__ xbase, uint64_t stride,
                                                  const T* __restrict__ y, double* __restrict__ partial,
                                                  const uint32_t* done) {
  if (done && *done) return;
  double ar[NV], ai[NV];
#pragma unroll
  for (int i = 0; i < NV; ++i) ar[i] = ai[i] = 0.0;
  for (uint64_t t = blockIdx.x * static_cast<uint64_t>(kKB) + threadIdx.x; t < n;
       t += static_cast<uint64_t>(gridDim.x) * kKB) {
    const double2 w = KAmp<T>::ld(y, t);
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const double2 v = KAmp<T>::ld(xbase + i * stride, t);
      ar[i] = fma(v.x, w.x, fma(v.y, w.y, ar[i]));
      ai[i] = fma(v.x, w.y, fma(-v.y, w.x, ai[i]));
    }
  }
  block_partials<NV>(ar, ai, partial);
}

// What the sums of block partials update in the state.
enum : int { kSumNorm = 0, kSumAlpha = 1, kSumProject = 2, kSumBeta = 3 };

// Value v = sum over blocks of partial[v * nblocks + b] in a fixed order (a
// wave per value), then thread 0 turns the values into the state's next
// entries.  One wave per value, where one block that took the values in turn
// needed 66 us for 24 values of 3336 blocks; this takes 5 (of 512 blocks).
constexpr int kSumBlock = 1024;
template <int MODE>
__global__ __launch_bounds__(kSumBlock) void k_sum_partials(const double* partial, int nblocks, int nvals, uint32_t j,
                                                            LanczosState* st) {
  if (MODE != kSumNorm && st->done) return;
  __shared__ double val[2 * kMaxK];
  const int lane = threadIdx.x & 63;
  for (int v = threadIdx.x >> 6; v < nvals; v += kSumBlock / 64) {
    double s = 0.0;
    for (int b = lane; b < nblocks; b += 64) s += partial[static_cast<uint64_t>(v) * nblocks + b];
    for (int d = 32; d > 0; d >>= 1) s += __shfl_xor(s, d, 64);
    if (lane == 0) val[v] = s;
  }
  __syncthreads();
  if (MODE == kSumAlpha || MODE == kSumProject) {
    // sweep coefficients: the recurrence terms, or minus the projections
    const uint32_t i = threadIdx.x;
    if (i <= j) {
      double re = 0.0, im = 0.0;
      if (MODE == kSumProject || i == j) {
        const uint32_t at = MODE == kSumProject ? i : 0u;
        re = -val[2 * at];
        im = -val[2 * at + 1];
      } else if (i + 1 == j) {
        re = -st->beta[i];
      }
      st->c.re[i] = re;
      st->c.im[i] = im;
    }
    if (MODE == kSumAlpha && i == 0) st->alpha[j] = val[0];
    return;
  }
  if (threadIdx.x != 0) return;
  if (MODE == kSumNorm) {
    const double nrm = sqrt(val[0]);
    st->nrm = nrm;
    st->inv = 1.0 / nrm;
    st->scale = 0.0;
    st->last_b = 0.0;
    st->k = 0;
    st->done = nrm > 0.0 ? 0u : 1u;
    return;
  }
  const double b = sqrt(val[0] < 0.0 ? 0.0 : val[0]);
  const double a = fabs(st->alpha[j]);
  const double big = a < b ? b : a;  // a where b is NaN
  const double scale = st->scale < big ? big : st->scale;
  st->scale = scale;
  st->last_b = b;
  st->k = j + 1;
  if (b <= 1e-14 * scale) {
    st->done = 1u;
  } else {
    st->beta[j] = b;
    st->inv = 1.0 / b;
  }
}

// y <- beta_scale * y + sum_i c_i x_i   (float64 arithmetic, one rounding to T)
template <class T>
__global__ __launch_bounds__(kKB) void k_multiaxpy(uint64_t n, int nv, const T* __restrict__ xbase, uint64_t stride,
                                                   Coeffs c, double y_scale, T* __restrict__ y) {
  for (uint64_t t = blockIdx.x * static_cast<uint64_t>(kKB) + threadIdx.x; t < n;
       t += static_cast<uint64_t>(gridDim.x) * kKB) {
    double r = 0.0, m = 0.0;
    if (y_scale != 0.0) {
      const double2 w = KAmp<T>::ld(y, t);
      r = y_scale * w.x;
      m = y_scale * w.y;
    }
#pragma unroll
    for (int i = 0; i < kMaxK; ++i) {
      if (i < nv) {
        const double2 v = KAmp<T>::ld(xbase + i * stride, t);
        r = fma(c.re[i], v.x, fma(-c.im[i], v.y, r));
        m = fma(c.re[i], v.y, fma(c.im[i], v.x, m));
      }
    }
    KAmp<T>::st(y, t, r, m);
  }
}

// Fused Gram-Schmidt pass: y <- y + sum_i c_i x_i, and from the same sweep
// over the elements the block partials that k_multidot would write for the
// updated y as stored: with NORM = false the inner products conj(x_i) y of
// the same x_i (the next pass's projections), with NORM = true |y|^2 (as
// k_multidot(y, y)).  Each thread visits the same elements in the same order
// as in k_multidot, so the reduced values are those of the unfused sequence
// bit for bit; y is read and written once instead of read three times and
// written once.
template <class T, bool NORM, int NV>
__global__ __launch_bounds__(kKB) void k_multiaxpy_dot(uint64_t n, const T* __restrict__ xbase, uint64_t stride,
                                                       const LanczosState* __restrict__ st, T* __restrict__ y,
                                                       double* __restrict__ partial) {
  if (st->done) return;
  const Coeffs& c = st->c;
  constexpr int kD = NORM ? 1 : NV;
  double ar[kD], ai[kD];
#pragma unroll
  for (int i = 0; i < kD; ++i) ar[i] = ai[i] = 0.0;
  for (uint64_t t = blockIdx.x * static_cast<uint64_t>(kKB) + threadIdx.x; t < n;
       t += static_cast<uint64_t>(gridDim.x) * kKB) {
    const double2 w0 = KAmp<T>::ld(y, t);
    double r = w0.x, m = w0.y;
    double2 v[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      v[i] = KAmp<T>::ld(xbase + i * stride, t);
      r = fma(c.re[i], v[i].x, fma(-c.im[i], v[i].y, r));
      m = fma(c.re[i], v[i].y, fma(c.im[i], v[i].x, m));
    }
    KAmp<T>::st(y, t, r, m);
    const double2 w = KAmp<T>::stored(r, m);
    if (NORM) {
      ar[0] = fma(w.x, w.x, fma(w.y, w.y, ar[0]));
      ai[0] = fma(w.x, w.y, fma(-w.y, w.x, ai[0]));
    } else {
#pragma unroll
      for (int i = 0; i < kD; ++i) {
        ar[i] = fma(v[i].x, w.x, fma(v[i].y, w.y, ar[i]));
        ai[i] = fma(v[i].x, w.y, fma(-v[i].y, w.x, ai[i]));
      }
    }
  }
  block_partials<kD>(ar, ai, partial);
}

// Launches K<NV> for the runtime count nv in 1..kMaxK.
template <template <int> class K, int NV = 1, class... A>
void launch_nv(int nv, dim3 grid, hipStream_t s, A... args) {
  if constexpr (NV <= kMaxK) {
    if (nv == NV) {
      hipLaunchKernelGGL(K<NV>::fn(), grid, dim3(kKB), 0, s, args...);
      return;
    }
    launch_nv<K, NV + 1>(nv, grid, s, args...);
  } else {
    PBS_REQUIRE(false, PBS_ERR_RANGE, "vector count outside 1..16");
  }
}
template <class T>
struct DotK {
  template <int NV>
  struct K {
    static auto fn() { return k_multidot<T, NV>; }
  };
};
template <class T, bool NORM>
struct AxpyDotK {
  template <int NV>
  struct K {
    static auto fn() { return k_multiaxpy_dot<T, NORM, NV>; }
  };
};

// y <- x / (norm in the state)
template <class T>
__global__ __launch_bounds__(kKB) void k_scale_copy(uint64_t n, const T* __restrict__ x,
                                                    const LanczosState* __restrict__ st, T* __restrict__ y) {
  if (st->done) return;
  const double s = st->inv;
  for (uint64_t t = blockIdx.x * static_cast<uint64_t>(kKB) + threadIdx.x; t < n;
       t += static_cast<uint64_t>(gridDim.x) * kKB) {
    const double2 v = KAmp<T>::ld(x, t);
    KAmp<T>::st(y, t, s * v.x, s * v.y);
  }
}

// Cyclic Jacobi eigen-decomposition of a symmetric k x k matrix (row-major);
// on return a holds the eigenvalues on its diagonal and u the eigenvectors
// (columns).
void jacobi_eigen(int k, std::vector<double>& a, std::vector<double>& u) {
  u.assign(static_cast<size_t>(k) * k, 0.0);
  for (int i = 0; i < k; ++i) u[i * k + i] = 1.0;
  for (int sweep = 0; sweep < 100; ++sweep) {
    double off = 0.0, diag = 0.0;
    for (int i = 0; i < k; ++i) {
      diag += a[i * k + i] * a[i * k + i];
      for (int j = i + 1; j < k; ++j) off += a[i * k + j] * a[i * k + j];
    }
    if (off <= 1e-34 * (diag + 1e-300)) break;
    for (int p = 0; p < k; ++p) {
      for (int q = p + 1; q < k; ++q) {
        const double apq = a[p * k + q];
        if (apq == 0.0) continue;
        const double theta = (a[q * k + q] - a[p * k + p]) / (2.0 * apq);
        const double t = (theta >= 0 ? 1.0 : -1.0) / (std::fabs(theta) + std::sqrt(theta * theta + 1.0));
        const double c = 1.0 / std::sqrt(t * t + 1.0), s = t * c;
        for (int r = 0; r < k; ++r) {  // A <- A J (columns p, q)
          const double arp = a[r * k + p], arq = a[r * k + q];
          a[r * k + p] = c * arp - s * arq;
          a[r * k + q] = s * arp + c * arq;
        }
        for (int r = 0; r < k; ++r) {  // A <- J^T A (rows p, q)
          const double apr = a[p * k + r], aqr = a[q * k + r];
          a[p * k + r] = c * apr - s * aqr;
          a[q * k + r] = s * apr + c * aqr;
        }
        for (int r = 0; r < k; ++r) {  // U <- U J
          const double urp = u[r * k + p], urq = u[r * k + q];
          u[r * k + p] = c * urp - s * urq;
          u[r * k + q] = s * urp + c * urq;
        }
      }
    }
  }
}

size_t elem_size(pbs_dtype dt) { return dt == PBS_C128 ? 16 : 8; }

// block partials (kDotGrid of them are used), then the state
size_t partial_doubles() { return static_cast<size_t>(kKGrid) * 2 * kMaxK; }
static_assert((kKGrid - kDotGrid) * 2 * kMaxK * sizeof(double) >= sizeof(LanczosState), "the state follows the partials");

uint64_t workspace_bytes(const pbs_space& sp, pbs_dtype dt, uint32_t m) {
  const uint64_t vec = sp.dim * elem_size(dt);
  return (m + 1) * ((vec + 255) & ~255ull) + (partial_doubles() + 2 * kMaxK) * sizeof(double);
}

template <class T>
class Lanczos {
 public:
  Lanczos(const pbs_grouped& h, const pbs_space& sp, pbs_dtype dt, uint32_t m, unsigned char* work, hipStream_t s)
      : h_(h), sp_(sp), dt_(dt), m_(m), s_(s), n_(sp.dim) {
    stride_ = (n_ * sizeof(T) + 255) & ~255ull;
    V_ = reinterpret_cast<T*>(work);
    W_ = reinterpret_cast<T*>(work + m * stride_);
    partial_ = reinterpret_cast<double*>(work + (m + 1) * stride_);
    st_ = reinterpret_cast<LanczosState*>(partial_ + static_cast<size_t>(kDotGrid) * 2 * kMaxK);
    grid_ = grid_for(n_, kKB, kKGrid);
    dot_grid_ = grid_for(n_, kKB, kDotGrid);
  }
  T* vec(uint32_t i) const { return reinterpret_cast<T*>(reinterpret_cast<unsigned char*>(V_) + i * stride_); }
  uint64_t stride_elems() const { return stride_ / sizeof(T); }

  // sums the partials of the last kernel into the state
  template <int MODE>
  void sum(int nvals, uint32_t j) {
    hipLaunchKernelGGL(k_sum_partials<MODE>, dim3(1), dim3(kSumBlock), 0, s_, partial_, static_cast<int>(dot_grid_),
                       nvals, j, st_);
    PBS_HIP(hipGetLastError());
  }
  // y <- y + sum_i c_i x_i with the state's coefficients, then the partials of
  // sum_i conj(x_i) y, or of |y|^2
  template <bool NORM>
  void sweep(int nv, T* y) {
    launch_nv<AxpyDotK<T, NORM>::template K>(nv, dim3(dot_grid_), s_, n_, vec(0), stride_elems(), st_, y, partial_);
  }
  void axpy(const T* xbase, int nv, const double* cre, const double* cim, double y_scale, T* y) {
    Coeffs c{};
    for (int i = 0; i < nv; ++i) {
      c.re[i] = cre[i];
      c.im[i] = cim[i];
    }
    hipLaunchKernelGGL((k_multiaxpy<T>), dim3(grid_), dim3(kKB), 0, s_, n_, nv, xbase, stride_elems(), c, y_scale, y);
    PBS_HIP(hipGetLastError());
  }

  void step(T* psi, double dt, double* info) {
    launch_nv<DotK<T>::template K>(1, dim3(dot_grid_), s_, n_, psi, stride_elems(), psi, partial_,
                                   static_cast<const uint32_t*>(nullptr));
    sum<kSumNorm>(2, 0);
    hipLaunchKernelGGL((k_scale_copy<T>), dim3(grid_), dim3(kKB), 0, s_, n_, psi, st_, vec(0));
    PBS_HIP(hipGetLastError());
    for (uint32_t j = 0; j < m_; ++j) {
      apply_launch(h_, sp_, dt_, vec(j), W_, s_, &st_->done);
      // the three-term recurrence: alpha_j = <v_j, w> on the fresh product
      // (H is Hermitian, so w has no other component in exact arithmetic)
      launch_nv<DotK<T>::template K>(1, dim3(dot_grid_), s_, n_, vec(j), stride_elems(), W_, partial_, &st_->done);
      sum<kSumAlpha>(2, j);
      // subtract alpha_j v_j + beta_{j-1} v_{j-1}, and in the same sweep the
      // projections on every basis vector (full re-orthogonalisation)
      sweep<false>(static_cast<int>(j + 1), W_);
      sum<kSumProject>(2 * static_cast<int>(j + 1), j);
      // subtract those, and in the same sweep |w|^2
      sweep<true>(static_cast<int>(j + 1), W_);
      sum<kSumBeta>(2, j);
      if (j + 1 == m_) break;
      hipLaunchKernelGGL((k_scale_copy<T>), dim3(grid_), dim3(kKB), 0, s_, n_, W_, st_, vec(j + 1));
      PBS_HIP(hipGetLastError());
    }
    const LanczosState st = read_scalar(st_, s_);
    const double nrm = st.nrm;
    info[0] = nrm;
    if (!(nrm > 0.0)) {
      info[1] = 0.0;
      info[2] = 0.0;
      info[3] = 0.0;
      return;
    }
    const uint32_t k = st.k;
    const double *alpha = st.alpha, *beta = st.beta;
    // exp(-i T dt) e_1 from the eigen-decomposition of the tridiagonal T
    std::vector<double> a(static_cast<size_t>(k) * k, 0.0), u;
    for (uint32_t i = 0; i < k; ++i) a[i * k + i] = alpha[i];
    for (uint32_t i = 0; i + 1 < k; ++i) a[i * k + i + 1] = a[(i + 1) * k + i] = beta[i];
    jacobi_eigen(static_cast<int>(k), a, u);
    double cre[kMaxK], cim[kMaxK];
    for (uint32_t r = 0; r < k; ++r) {
      double sr = 0.0, si = 0.0;
      for (uint32_t q = 0; q < k; ++q) {
        const double lam = a[q * k + q];
        const double w = u[r * k + q] * u[0 * k + q];
        sr += w * std::cos(lam * dt);
        si -= w * std::sin(lam * dt);
      }
      cre[r] = nrm * sr;
      cim[r] = nrm * si;
    }
    axpy(vec(0), static_cast<int>(k), cre, cim, 0.0, psi);
    PBS_HIP(hipStreamSynchronize(s_));
    info[1] = alpha[0];
    info[2] = static_cast<double>(k);
    info[3] = st.last_b;
  }

 private:
  const pbs_grouped& h_;
  const pbs_space& sp_;
  pbs_dtype dt_;
  uint32_t m_;
  hipStream_t s_;
  uint64_t n_;
  uint64_t stride_ = 0;
  T* V_ = nullptr;
  T* W_ = nullptr;
  double* partial_ = nullptr;
  LanczosState* st_ = nullptr;
  unsigned grid_ = 1, dot_grid_ = 1;
};

}  // namespace
}  // namespace pbs

using namespace pbs;

extern "C" {

pbs_status pbs_krylov_workspace_bytes(const pbs_space* sp, pbs_dtype dt, uint32_t m, uint64_t* bytes) {
  return guarded([&] {
    PBS_REQUIRE(sp != nullptr && bytes != nullptr, PBS_ERR_ARG, "null argument");
    PBS_REQUIRE(dt == PBS_C128 || dt == PBS_C64, PBS_ERR_ARG, "unknown dtype");
    PBS_REQUIRE(m >= 1 && m <= static_cast<uint32_t>(kMaxK), PBS_ERR_RANGE, "m must be 1..16");
    *bytes = workspace_bytes(*sp, dt, m);
  });
}

pbs_status pbs_krylov_step(const pbs_grouped* h, const pbs_space* sp, pbs_dtype dt, void* psi, double dt_step,
                           uint32_t m, void* work, uint64_t work_bytes, double* info, void* stream) {
  return guarded([&] {
    PBS_REQUIRE(h != nullptr && sp != nullptr && psi != nullptr && work != nullptr && info != nullptr,
                PBS_ERR_ARG, "null argument");
    PBS_REQUIRE(dt == PBS_C128 || dt == PBS_C64, PBS_ERR_ARG, "unknown dtype");
    PBS_REQUIRE(m >= 1 && m <= static_cast<uint32_t>(kMaxK), PBS_ERR_RANGE, "m must be 1..16");
    PBS_REQUIRE(std::isfinite(dt_step), PBS_ERR_ARG, "dt is not finite");
    PBS_REQUIRE(work_bytes >= workspace_bytes(*sp, dt, m), PBS_ERR_ARG, "workspace too small");
    const auto a = reinterpret_cast<uintptr_t>(psi), w = reinterpret_cast<uintptr_t>(work);
    const uint64_t pb = sp->dim * elem_size(dt);
    PBS_REQUIRE(a + pb <= w || w + work_bytes <= a, PBS_ERR_ARG, "psi overlaps the workspace");
    hipStream_t s = as_stream(stream);
    unsigned char* wk = static_cast<unsigned char*>(work);
    if (dt == PBS_C128) {
      Lanczos<double2> L(*h, *sp, dt, m, wk, s);
      L.step(static_cast<double2*>(psi), dt_step, info);
    } else {
      Lanczos<float2> L(*h, *sp, dt, m, wk, s);
      L.step(static_cast<float2*>(psi), dt_step, info);
    }
  });
}

}  // extern "C"
