// Device primitives: exclusive scan, stable LSD radix sort on multiword keys,
// starts of runs of equal keys.  They carry the canonical reduction of Section 2.3
// (radix sort of the binary symplectic keys, then a linear merge) and the
// grouping of Eq. topological_group.
#include "pbs_internal.h"

namespace pbs {

namespace {

constexpr int kScanBlock = 256;
constexpr int kScanItems = 8;
constexpr uint64_t kScanTile = kScanBlock * kScanItems;

// Exclusive scan of one value per thread across a 256-thread block (4 wave64s).
__device__ inline uint32_t block_exclusive_scan(uint32_t v, uint32_t* lds_wave, uint32_t& block_total) {
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  uint32_t incl = v;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    uint32_t t = __shfl_up(incl, d, 64);
    if (lane >= d) incl += t;
  }
  if (lane == 63) lds_wave[wave] = incl;
  __syncthreads();
  uint32_t wave_off = 0;
  uint32_t total = 0;
  for (int w = 0; w < kScanBlock / 64; ++w) {
    uint32_t t = lds_wave[w];
    if (w < wave) wave_off += t;
    total += t;
  }
  __syncthreads();
  block_total = total;
  return wave_off + incl - v;
}

__global__ __launch_bounds__(kScanBlock) void k_scan_partials(const uint32_t* in, uint64_t n, uint32_t* partial) {
  __shared__ uint32_t lds[kScanBlock / 64];
  const uint64_t base = blockIdx.x * kScanTile + threadIdx.x * kScanItems;
  uint32_t s = 0;
#pragma unroll
  for (int j = 0; j < kScanItems; ++j) {
    uint64_t i = base + j;
    if (i < n) s += in[i];
  }
  uint32_t total;
  (void)block_exclusive_scan(s, lds, total);
  if (threadIdx.x == 0) partial[blockIdx.x] = total;
}

// Single block: exclusive scan of the per-tile partial sums.
__global__ __launch_bounds__(kScanBlock) void k_scan_partials_scan(uint32_t* partial, uint64_t nb, uint32_t* total_out) {
  __shared__ uint32_t lds[kScanBlock / 64];
  uint32_t carry = 0;
  for (uint64_t c = 0; c < nb; c += kScanBlock) {
    uint64_t i = c + threadIdx.x;
    uint32_t v = i < nb ? partial[i] : 0u;
    uint32_t tot;
    uint32_t ex = block_exclusive_scan(v, lds, tot);
    if (i < nb) partial[i] = carry + ex;
    carry += tot;
  }
  if (threadIdx.x == 0 && total_out) *total_out = carry;
}

// Sum of the partials before this block's tile, for launches without
// k_scan_partials_scan: every block adds them up itself (nb <= kScanMidTiles
// values from cache), which is cheaper than one more launch between the two
// passes.
__device__ inline uint32_t partials_before(const uint32_t* partial, uint32_t* lds) {
  uint32_t v = 0;
  for (uint32_t i = threadIdx.x; i < blockIdx.x; i += kScanBlock) v += partial[i];
  uint32_t tot;
  (void)block_exclusive_scan(v, lds, tot);
  return tot;
}

// scanned: partial holds prefix sums already; otherwise raw tile sums, and the
// last block writes the total.
__global__ __launch_bounds__(kScanBlock) void k_scan_apply(const uint32_t* in, uint32_t* out, uint64_t n,
                                                           const uint32_t* partial, bool scanned,
                                                           uint32_t* total_out) {
  __shared__ uint32_t lds[kScanBlock / 64];
  const uint64_t base = blockIdx.x * kScanTile + threadIdx.x * kScanItems;
  uint32_t v[kScanItems];
  uint32_t s = 0;
#pragma unroll
  for (int j = 0; j < kScanItems; ++j) {
    uint64_t i = base + j;
    v[j] = i < n ? in[i] : 0u;
    s += v[j];
  }
  const uint32_t before = scanned ? partial[blockIdx.x] : partials_before(partial, lds);
  uint32_t tot;
  uint32_t run = before + block_exclusive_scan(s, lds, tot);
#pragma unroll
  for (int j = 0; j < kScanItems; ++j) {
    uint64_t i = base + j;
    if (i < n) out[i] = run;
    run += v[j];
  }
  if (!scanned && total_out && blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) *total_out = before + tot;
}

// Single block: the whole scan for short inputs, tile after tile with a running
// carry; in == out is allowed (each thread reads its items before the block
// scan and writes them after it).  A tile takes 2.5 us of latency, the two
// launches of the next form 9 us together, so the line lies at four tiles.
constexpr uint64_t kScanSingleTiles = 4;
constexpr uint64_t kScanMidTiles = 1024;
__global__ __launch_bounds__(kScanBlock) void k_scan_single(const uint32_t* in, uint32_t* out, uint64_t n,
                                                            uint32_t* total_out) {
  __shared__ uint32_t lds[kScanBlock / 64];
  uint32_t carry = 0;
  for (uint64_t c = 0; c < n; c += kScanTile) {
    const uint64_t base = c + threadIdx.x * kScanItems;
    uint32_t v[kScanItems];
    uint32_t s = 0;
#pragma unroll
    for (int j = 0; j < kScanItems; ++j) {
      const uint64_t i = base + j;
      v[j] = i < n ? in[i] : 0u;
      s += v[j];
    }
    uint32_t tot;
    uint32_t run = carry + block_exclusive_scan(s, lds, tot);
#pragma unroll
    for (int j = 0; j < kScanItems; ++j) {
      const uint64_t i = base + j;
      if (i < n) out[i] = run;
      run += v[j];
    }
    carry += tot;
  }
  if (threadIdx.x == 0 && total_out) *total_out = carry;
}

// ---------------------------------------------------------------- radix sort
// Only bits that differ between items take part: the varying bits of word 0,
// then of word 1, and so on, form one long key that is cut into 8-bit digits,
// so masks over n qubits take ceil(2 n / 8) passes.  A digit is a few runs of
// adjacent bits, each from one word.
struct Digit {
  uint32_t n, bits;
  uint8_t word[8], shift[8], len[8];
};

__host__ __device__ inline uint32_t trailing_zeros(uint64_t v) { return static_cast<uint32_t>(__builtin_ctzll(v)); }

// Takes the next digit (up to 8 of the lowest bits left) out of the masks.
template <class Mask>
__host__ __device__ inline bool next_digit(Mask* left, int nw, Digit& d) {
  d.n = d.bits = 0;
  for (int w = 0; w < nw; ++w) {
    uint64_t v = left[w];
    while (v != 0 && d.bits < 8) {
      const uint32_t shift = trailing_zeros(v);
      const uint64_t up = ~(v >> shift);
      uint32_t len = up == 0 ? 64u : trailing_zeros(up);
      len = len < 8 - d.bits ? len : 8 - d.bits;
      d.word[d.n] = static_cast<uint8_t>(w);
      d.shift[d.n] = static_cast<uint8_t>(shift);
      d.len[d.n] = static_cast<uint8_t>(len);
      ++d.n;
      d.bits += len;
      v &= ~(((1ull << len) - 1ull) << shift);
    }
    left[w] = v;
    if (d.bits == 8) break;
  }
  return d.bits != 0;
}

__device__ inline uint32_t digit_of(const uint64_t* keys, uint64_t m, uint64_t i, const Digit& d) {
  uint32_t v = 0, at = 0;
  for (uint32_t j = 0; j < d.n; ++j) {
    v |= static_cast<uint32_t>((keys[d.word[j] * m + i] >> d.shift[j]) & ((1u << d.len[j]) - 1u)) << at;
    at += d.len[j];
  }
  return v;
}

constexpr int kSortBlock = 1024;
constexpr int kSortWaves = kSortBlock / 64;
constexpr int kSortChunks = 4;  // per wave: 4 x 64 adjacent items
constexpr uint32_t kSortTile = kSortBlock * kSortChunks;
// Up to this many tiles a scatter block adds up the digit counts of the tiles
// before it by itself; above, a scan of all counts runs in between.  At 17
// tiles (66,000 items) the scan's launch took 20 us of a pass.  Every block
// reads the counts of all tiles, 128 KB at 128 tiles (2 us from cache), and that
// grows with the square of the size, so the two launches of the scan (9 us) win
// somewhat above.
constexpr uint32_t kSortSumTiles = 128;

// OR over all items of (key ^ key[0]) per word: the bits that vary.  Few
// blocks with one atomic per word each: with 1024 blocks and an atomic per
// wave the kernel took 96 us for 65,000 items, all of it atomics on the same words.
constexpr uint32_t kVaryBlocks = 512;
__global__ __launch_bounds__(256) void k_varying_bits(const uint64_t* keys, uint64_t m, int nw, unsigned long long* out) {
  __shared__ uint64_t part[4];
  for (int w = 0; w < nw; ++w) {
    const uint64_t* k = keys + static_cast<uint64_t>(w) * m;
    const uint64_t ref = k[0];
    uint64_t acc = 0;
    const uint64_t step = gridDim.x * 256ull;
    uint64_t i = blockIdx.x * 256ull + threadIdx.x;
    for (; i + 3 * step < m; i += 4 * step)
      acc |= (k[i] ^ ref) | (k[i + step] ^ ref) | (k[i + 2 * step] ^ ref) | (k[i + 3 * step] ^ ref);
    for (; i < m; i += step) acc |= (k[i] ^ ref);
    for (int d = 32; d > 0; d >>= 1) acc |= __shfl_xor(acc, d, 64);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
      acc = part[0] | part[1] | part[2] | part[3];
      if (acc) atomicOr(out + w, static_cast<unsigned long long>(acc));
    }
    __syncthreads();
  }
}

// Digit counts per tile: at [tile][digit], or [digit][tile] when they are
// scanned in a pass of their own.
__global__ __launch_bounds__(kSortBlock) void k_radix_hist(const uint64_t* keys, uint64_t m, Digit d, bool scanned,
                                                           uint32_t* counts, uint32_t nblk) {
  __shared__ uint32_t h[256];
  if (threadIdx.x < 256) h[threadIdx.x] = 0;
  __syncthreads();
  const uint64_t start = static_cast<uint64_t>(blockIdx.x) * kSortTile;
  const uint64_t end = start + kSortTile < m ? start + kSortTile : m;
  for (uint64_t i = start + threadIdx.x; i < end; i += kSortBlock) atomicAdd(&h[digit_of(keys, m, i, d)], 1u);
  __syncthreads();
  if (threadIdx.x < 256)
    counts[scanned ? static_cast<uint64_t>(threadIdx.x) * nblk + blockIdx.x
                   : static_cast<uint64_t>(blockIdx.x) * 256 + threadIdx.x] = h[threadIdx.x];
}

// Stable ranks of a wave's chunks of 64 items: items with equal digits are
// matched by eight ballots, and the wave's running digit counts (its own row
// of cnt, so that no barrier is needed between chunks) order the chunks.
template <int CHUNKS>
__device__ inline void wave_ranks(const uint32_t (&dg)[CHUNKS], const bool (&valid)[CHUNKS], volatile uint32_t* cnt,
                                  uint32_t (&rank)[CHUNKS]) {
  const int lane = threadIdx.x & 63;
  const unsigned long long below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
#pragma unroll
  for (int c = 0; c < CHUNKS; ++c) {
    unsigned long long peers = __ballot(valid[c]);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const bool bit = (dg[c] >> b) & 1u;
      const unsigned long long mb = __ballot(bit);
      peers &= bit ? mb : ~mb;
    }
    const uint32_t in_chunk = static_cast<uint32_t>(__popcll(peers & below));
    const uint32_t before = cnt[dg[c]];
    rank[c] = before + in_chunk;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    if (valid[c] && in_chunk == 0) cnt[dg[c]] = before + static_cast<uint32_t>(__popcll(peers));
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  }
}

// Exclusive scan over the 256 digits of one value per thread of the first four
// waves (every thread of the block calls it).
__device__ inline uint32_t digit_scan(uint32_t v, uint32_t* lds_wave) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t incl = v;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t t = __shfl_up(incl, d, 64);
    if (lane >= d) incl += t;
  }
  if (lane == 63 && wave < 4) lds_wave[wave] = incl;
  __syncthreads();
  uint32_t off = 0;
  for (int w = 0; w < 4; ++w)
    if (w < wave) off += lds_wave[w];
  return off + incl - v;
}

// Stable scatter of one tile of 4096 items: 16 waves rank 256 adjacent items
// each on their own, then the tile is put in order in LDS, one array after the
// other, and written as runs of adjacent items.  Bound by latency for small
// inputs and by the writes for large ones: 3.3 M items of two words take 38 us
// (3.5 TB/s), 58 when every item was written from where it stood; 66,000 items
// went from 26 us to 18 against a 256-thread block that ranked a tile 256 items
// at a time.
__global__ __launch_bounds__(kSortBlock) void k_radix_scatter(const uint64_t* kin, uint64_t* kout, int nw, const uint32_t* vin,
                                                              uint32_t* vout, uint64_t m, Digit d, bool scanned,
                                                              const uint32_t* counts, uint32_t nblk) {
  __shared__ uint32_t cnt[kSortWaves][256];
  __shared__ uint64_t stage[kSortTile];
  __shared__ uint8_t digit_at[kSortTile];
  __shared__ uint32_t shift_of[256];  // global minus local position of a digit's items
  __shared__ uint32_t lds_wave[8];
  uint32_t* part = reinterpret_cast<uint32_t*>(stage);  // [2][4][256], until the tile is staged
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  for (int j = tid; j < kSortWaves * 256; j += kSortBlock) (&cnt[0][0])[j] = 0;
  const uint32_t q = tid >> 8, digit = tid & 255;
  if (!scanned) {
    uint32_t before = 0, total = 0;
    for (uint32_t b = q; b < nblk; b += 4) {
      const uint32_t v = counts[static_cast<uint64_t>(b) * 256 + digit];
      total += v;
      if (b < blockIdx.x) before += v;
    }
    part[q * 256 + digit] = before;
    part[1024 + q * 256 + digit] = total;
  }
  const uint64_t tile = static_cast<uint64_t>(blockIdx.x) * kSortTile;
  const uint32_t here = static_cast<uint32_t>(m - tile < kSortTile ? m - tile : kSortTile);
  const uint32_t first = wave * (64 * kSortChunks) + lane;
  uint32_t dg[kSortChunks], rank[kSortChunks];
  bool valid[kSortChunks];
#pragma unroll
  for (int c = 0; c < kSortChunks; ++c) {
    valid[c] = first + 64 * c < here;
    dg[c] = valid[c] ? digit_of(kin, m, tile + first + 64 * c, d) : 0u;
  }
  __syncthreads();
  wave_ranks(dg, valid, cnt[wave], rank);
  uint32_t before = 0, total = 0;
  if (scanned) {
    if (tid < 256) before = counts[static_cast<uint64_t>(tid) * nblk + blockIdx.x];
  } else if (tid < 256) {
    for (int j = 0; j < 4; ++j) {
      before += part[j * 256 + tid];
      total += part[1024 + j * 256 + tid];
    }
  }
  const uint32_t smaller = digit_scan(total, lds_wave);  // its barrier also ends the ranking
  uint32_t mine = 0;
  if (tid < 256)
    for (int w = 0; w < kSortWaves; ++w) mine += cnt[w][tid];
  const uint32_t local = digit_scan(mine, lds_wave + 4);
  if (tid < 256) {
    shift_of[tid] = before + smaller - local;
    uint32_t run = local;
    for (int w = 0; w < kSortWaves; ++w) {
      const uint32_t v = cnt[w][tid];
      cnt[w][tid] = run;
      run += v;
    }
  }
  __syncthreads();
#pragma unroll
  for (int c = 0; c < kSortChunks; ++c) {
    if (!valid[c]) continue;
    rank[c] += cnt[wave][dg[c]];  // now the local position, below `here`
    digit_at[rank[c]] = static_cast<uint8_t>(dg[c]);
  }
  uint32_t pos[kSortChunks];
  for (int w = 0; w <= nw; ++w) {
    const uint64_t* kw = kin + static_cast<uint64_t>(w) * m + tile;
    uint64_t v[kSortChunks];
#pragma unroll
    for (int c = 0; c < kSortChunks; ++c)
      if (valid[c]) v[c] = w < nw ? kw[first + 64 * c] : vin[tile + first + 64 * c];
    if (w > 0) __syncthreads();
#pragma unroll
    for (int c = 0; c < kSortChunks; ++c)
      if (valid[c]) stage[rank[c]] = v[c];
    __syncthreads();
    if (w == 0) {
#pragma unroll
      for (int c = 0; c < kSortChunks; ++c) {
        const uint32_t j = tid + kSortBlock * c;
        pos[c] = j < here ? j + shift_of[digit_at[j]] : 0u;
        if (pos[c] >= m) pos[c] = 0;  // unreachable with consistent counts; keeps writes in bounds
      }
    }
#pragma unroll
    for (int c = 0; c < kSortChunks; ++c) {
      const uint32_t j = tid + kSortBlock * c;
      if (j >= here) continue;
      if (w < nw)
        kout[static_cast<uint64_t>(w) * m + pos[c]] = stage[j];
      else
        vout[pos[c]] = static_cast<uint32_t>(stage[j]);
    }
  }
}

// Whole sort of at most 8192 items by one block: varying bits, every pass (on
// 16-bit positions in LDS; the keys stay where they are and come from cache)
// and the final gather.  One launch and no read-back, where the passes above
// take two launches each: 5,800 items of three words (five passes) take 59 us
// where the passes, their launches and the read-back took about 180.
constexpr int kOneChunks = 8;
constexpr uint32_t kOneBlockItems = kSortBlock * kOneChunks;
__global__ __launch_bounds__(kSortBlock) void k_sort_one_block(uint64_t* keys, uint32_t* vals, uint32_t m, int nw) {
  __shared__ uint16_t ord[kOneBlockItems];
  __shared__ uint32_t cnt[kSortWaves][256];
  __shared__ uint32_t lds_wave[4];
  __shared__ unsigned long long vary[2 * kMaxWords];  // bits left to sort by (thread 0's after the first pass)
  __shared__ Digit digit;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  if (tid < 2 * kMaxWords) vary[tid] = 0ull;
  for (uint32_t i = tid; i < m; i += kSortBlock) ord[i] = static_cast<uint16_t>(i);
  __syncthreads();
  for (int w = 0; w < nw; ++w) {
    const uint64_t ref = keys[static_cast<uint64_t>(w) * m];
    uint64_t acc = 0;
    for (uint32_t i = tid; i < m; i += kSortBlock) acc |= keys[static_cast<uint64_t>(w) * m + i] ^ ref;
    for (int d = 32; d > 0; d >>= 1) acc |= __shfl_xor(acc, d, 64);
    if (lane == 0 && acc) atomicOr(&vary[w], static_cast<unsigned long long>(acc));
  }
  __syncthreads();
  const uint32_t first = wave * (64 * kOneChunks) + lane;
  for (;;) {  // at most one pass per 8 varying bits
    if (tid == 0) (void)next_digit(vary, nw, digit);
    __syncthreads();
    if (digit.bits == 0) break;
    const Digit& d = digit;
    for (int j = tid; j < kSortWaves * 256; j += kSortBlock) (&cnt[0][0])[j] = 0;
    uint32_t dg[kOneChunks], rank[kOneChunks], at[kOneChunks];
    bool valid[kOneChunks];
#pragma unroll
    for (int c = 0; c < kOneChunks; ++c) {
      valid[c] = first + 64 * c < m;
      at[c] = valid[c] ? ord[first + 64 * c] : 0u;
      dg[c] = valid[c] ? digit_of(keys, m, at[c], d) : 0u;
    }
    __syncthreads();
    wave_ranks(dg, valid, cnt[wave], rank);
    __syncthreads();
    uint32_t total = 0;
    if (tid < 256)
      for (int w = 0; w < kSortWaves; ++w) total += cnt[w][tid];
    const uint32_t smaller = digit_scan(total, lds_wave);
    if (tid < 256) {
      uint32_t run = smaller;
      for (int w = 0; w < kSortWaves; ++w) {
        const uint32_t v = cnt[w][tid];
        cnt[w][tid] = run;
        run += v;
      }
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < kOneChunks; ++c)
      if (valid[c]) ord[(cnt[wave][dg[c]] + rank[c]) & (kOneBlockItems - 1)] = static_cast<uint16_t>(at[c]);
    __syncthreads();
  }
  // gather in place, one array after the other (loads end before stores begin)
  for (int w = 0; w <= nw; ++w) {
    uint64_t v[kOneChunks];
#pragma unroll
    for (int c = 0; c < kOneChunks; ++c) {
      const uint32_t i = first + 64 * c;
      if (i < m) v[c] = w < nw ? keys[static_cast<uint64_t>(w) * m + ord[i]] : vals[ord[i]];
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < kOneChunks; ++c) {
      const uint32_t i = first + 64 * c;
      if (i >= m) continue;
      if (w < nw)
        keys[static_cast<uint64_t>(w) * m + i] = v[c];
      else
        vals[i] = static_cast<uint32_t>(v[c]);
    }
  }
}

// ---------------------------------------------------------------- runs of equal keys
// Tile of 2048 items, 256 at a time: head flags as wave ballots.  The two
// passes (counts, then positions of the heads) compare the keys twice instead
// of writing and scanning a flag per item.
constexpr int kRunChunks = 8;
__device__ inline bool run_head(const uint64_t* keys, uint64_t m, int nw, uint64_t i) {
  if (i == 0) return true;
  for (int w = 0; w < nw; ++w)
    if (keys[static_cast<uint64_t>(w) * m + i] != keys[static_cast<uint64_t>(w) * m + i - 1]) return true;
  return false;
}

__global__ __launch_bounds__(kScanBlock) void k_run_counts(const uint64_t* keys, uint64_t m, int nw, uint32_t* partial) {
  __shared__ uint32_t lds[kScanBlock / 64];
  const uint64_t base = blockIdx.x * kScanTile + threadIdx.x;
  uint32_t n = 0;
#pragma unroll
  for (int j = 0; j < kRunChunks; ++j) {
    const uint64_t i = base + j * kScanBlock;
    n += i < m && run_head(keys, m, nw, i) ? 1u : 0u;
  }
  uint32_t total;
  (void)block_exclusive_scan(n, lds, total);
  if (threadIdx.x == 0) partial[blockIdx.x] = total;
}

__global__ __launch_bounds__(kScanBlock) void k_run_starts(const uint64_t* keys, uint64_t m, int nw,
                                                           const uint32_t* partial, bool scanned, uint32_t* start,
                                                           uint32_t* total_out) {
  constexpr int kWaves = kScanBlock / 64;
  __shared__ uint32_t lds[kWaves];
  __shared__ uint32_t cnt[kRunChunks * kWaves];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint64_t base = blockIdx.x * kScanTile + threadIdx.x;
  unsigned long long heads[kRunChunks];
#pragma unroll
  for (int j = 0; j < kRunChunks; ++j) {
    const uint64_t i = base + j * kScanBlock;
    heads[j] = __ballot(i < m && run_head(keys, m, nw, i));
    if (lane == 0) cnt[j * kWaves + wave] = static_cast<uint32_t>(__popcll(heads[j]));
  }
  uint32_t run = scanned ? partial[blockIdx.x] : partials_before(partial, lds);
  __syncthreads();
  const unsigned long long below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
#pragma unroll
  for (int j = 0; j < kRunChunks; ++j)
    for (int w = 0; w < kWaves; ++w) {
      if (w == wave && (heads[j] >> lane & 1ull))
        start[run + static_cast<uint32_t>(__popcll(heads[j] & below))] = static_cast<uint32_t>(base + j * kScanBlock);
      run += cnt[j * kWaves + w];
    }
  if (!scanned && blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) *total_out = run;
}

__global__ void k_iota(uint32_t* v, uint64_t m) {
  for (uint64_t i = blockIdx.x * static_cast<uint64_t>(blockDim.x) + threadIdx.x; i < m;
       i += static_cast<uint64_t>(gridDim.x) * blockDim.x)
    v[i] = static_cast<uint32_t>(i);
}

}  // namespace

void iota_u32(uint32_t* v, uint64_t m, hipStream_t s) {
  if (m == 0) return;
  hipLaunchKernelGGL(k_iota, dim3(grid_for(m, 256, 65536)), dim3(256), 0, s, v, m);
  PBS_HIP(hipGetLastError());
}

size_t scan_scratch_bytes(uint64_t n) { return ((n + kScanTile - 1) / kScanTile + 1) * sizeof(uint32_t); }

void exclusive_scan_u32(const uint32_t* in, uint32_t* out, uint64_t n, uint32_t* total, hipStream_t s) {
  PBS_REQUIRE(n < (1ull << 32), PBS_ERR_RANGE, "scan length exceeds 2^32");
  if (n == 0) {
    if (total) PBS_HIP(hipMemsetAsync(total, 0, sizeof(uint32_t), s));
    return;
  }
  const uint64_t nb = (n + kScanTile - 1) / kScanTile;
  if (nb <= kScanSingleTiles) {  // one launch, no temporary
    hipLaunchKernelGGL(k_scan_single, dim3(1), dim3(kScanBlock), 0, s, in, out, n, total);
    PBS_HIP(hipGetLastError());
    return;
  }
  const bool scanned = nb > kScanMidTiles;
  DevBuf<uint32_t> partial(nb, s);
  hipLaunchKernelGGL(k_scan_partials, dim3(static_cast<unsigned>(nb)), dim3(kScanBlock), 0, s, in, n, partial.get());
  if (scanned)
    hipLaunchKernelGGL(k_scan_partials_scan, dim3(1), dim3(kScanBlock), 0, s, partial.get(), nb, total);
  hipLaunchKernelGGL(k_scan_apply, dim3(static_cast<unsigned>(nb)), dim3(kScanBlock), 0, s, in, out, n, partial.get(),
                     scanned, total);
  PBS_HIP(hipGetLastError());
  // `partial` is released on return: a temporary of the call's scratch scope
  // stays reserved until the scope ends (which waits for the stream); one
  // from hipMalloc must not be freed under queued work
  if (!partial.borrowed) PBS_HIP(hipStreamSynchronize(s));
}

void run_starts(const uint64_t* keys, uint64_t m, int nw, uint32_t* start, uint32_t* total, hipStream_t s) {
  if (m == 0) return;
  const uint64_t nb = (m + kScanTile - 1) / kScanTile;
  const bool scanned = nb > kScanMidTiles;
  DevBuf<uint32_t> partial(nb, s);
  hipLaunchKernelGGL(k_run_counts, dim3(static_cast<unsigned>(nb)), dim3(kScanBlock), 0, s, keys, m, nw,
                     partial.get());
  if (scanned)
    hipLaunchKernelGGL(k_scan_partials_scan, dim3(1), dim3(kScanBlock), 0, s, partial.get(), nb, total);
  hipLaunchKernelGGL(k_run_starts, dim3(static_cast<unsigned>(nb)), dim3(kScanBlock), 0, s, keys, m, nw,
                     partial.get(), scanned, start, total);
  PBS_HIP(hipGetLastError());
  if (!partial.borrowed) PBS_HIP(hipStreamSynchronize(s));  // as above
}

void radix_sort_keys(uint64_t* keys, uint32_t* vals, uint64_t m, int nw, hipStream_t s) {
  PBS_REQUIRE(m < (1ull << 32), PBS_ERR_RANGE, "sort length exceeds 2^32");
  PBS_REQUIRE(nw >= 1 && nw <= 2 * kMaxWords, PBS_ERR_RANGE, "too many key words");
  if (m <= 1) return;
  if (m <= kOneBlockItems) {
    hipLaunchKernelGGL(k_sort_one_block, dim3(1), dim3(kSortBlock), 0, s, keys, vals, static_cast<uint32_t>(m), nw);
    PBS_HIP(hipGetLastError());
    return;
  }
  DevBuf<unsigned long long> vary(nw, s);
  PBS_HIP(hipMemsetAsync(vary.get(), 0, nw * sizeof(unsigned long long), s));
  hipLaunchKernelGGL(k_varying_bits, dim3(grid_for(m, 256, kVaryBlocks)), dim3(256), 0, s, keys, m, nw, vary.get());
  PBS_HIP(hipGetLastError());
  std::vector<unsigned long long> left(nw);
  PBS_HIP(hipMemcpyAsync(left.data(), vary.get(), nw * sizeof(unsigned long long), hipMemcpyDeviceToHost, s));
  PBS_HIP(hipStreamSynchronize(s));

  const uint32_t nblk = static_cast<uint32_t>((m + kSortTile - 1) / kSortTile);
  const bool scanned = nblk > kSortSumTiles;
  DevBuf<uint64_t> ktmp(m * nw, s);
  DevBuf<uint32_t> vtmp(m, s);
  DevBuf<uint32_t> counts(static_cast<uint64_t>(nblk) * 256, s);
  uint64_t* kcur = keys;
  uint32_t* vcur = vals;
  uint64_t* kalt = ktmp.get();
  uint32_t* valt = vtmp.get();
  Digit d;
  while (next_digit(left.data(), nw, d)) {
    hipLaunchKernelGGL(k_radix_hist, dim3(nblk), dim3(kSortBlock), 0, s, kcur, m, d, scanned, counts.get(), nblk);
    if (scanned) exclusive_scan_u32(counts.get(), counts.get(), static_cast<uint64_t>(nblk) * 256, nullptr, s);
    hipLaunchKernelGGL(k_radix_scatter, dim3(nblk), dim3(kSortBlock), 0, s, kcur, kalt, nw, vcur, valt, m, d, scanned,
                       counts.get(), nblk);
    PBS_HIP(hipGetLastError());
    std::swap(kcur, kalt);
    std::swap(vcur, valt);
  }
  if (kcur != keys) {
    PBS_HIP(hipMemcpyAsync(keys, kcur, m * nw * sizeof(uint64_t), hipMemcpyDeviceToDevice, s));
    PBS_HIP(hipMemcpyAsync(vals, vcur, m * sizeof(uint32_t), hipMemcpyDeviceToDevice, s));
  }
  // temporaries of the call's scratch scope stay reserved until it ends;
  // hipMalloc'd ones are freed on return, after the queued work
  if (!(vary.borrowed && ktmp.borrowed && vtmp.borrowed && counts.borrowed)) PBS_HIP(hipStreamSynchronize(s));
}

}  // namespace pbs
