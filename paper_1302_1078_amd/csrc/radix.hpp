// radix.hpp -- stable LSD radix sort of (key, payload) pairs on the device.
//
// Used once per sparsity pattern (assembly, the CSC index, orderings).  A
// pass over a digit is three launches: per-tile digit counts, a scan of each
// digit's counts over the tiles, and the scatter.  What bounds a pass is the
// memory it moves (keys twice, payloads once, both written once); the rest of
// the design keeps it near that:
//   - digits of up to 10 bits: 38 key bits (2^19 rows and columns) take four
//     passes instead of the five of 8-bit digits.  Wider digits would leave
//     fewer than four elements of a tile per digit and write runs below the
//     32-byte sector.
//   - each wavefront ranks a contiguous part of its tile against counters of
//     its own, so the ranking loop has no workgroup barrier;
//   - the tile is put into digit order in LDS and leaves as runs, which the
//     next tile (same XCD, same L2) continues;
//   - the first pass reads its keys through a source functor and the last one
//     writes through a sink functor, so callers neither materialise keys nor
//     re-read the sorted pairs to take them apart.
// Integer arithmetic only; the result is the stable order, so deterministic.
// Measured on 8.65 M pairs of a 64-bit key and a double: 105 us a pass
// (scatter 74, 3.7 TB/s; count 23; scan 7).  Assembly of those triplets
// (2^19 rows) takes 586 us, against 1,165 us with 8-bit digits, a barrier per
// 256 ranked elements and values fetched by position after the sort.
#pragma once

#include <type_traits>

#include "device.hpp"
#include "internal.hpp"

namespace spx {
namespace radix {

constexpr int kItems = 16;
constexpr int kTile = kWG * kItems;  // 4096 elements per workgroup
constexpr int kMaxDigit = 10;
constexpr int kMaxBins = 1 << kMaxDigit;
constexpr int kWaves = kWG / kWave;
constexpr int kTileSpan = 4 * kTile;  // rows of a tile that tile_rows walks

inline int64_t tiles_of(int64_t n) { return (n + kTile - 1) / kTile; }

// Passes over `bits` key bits (never 0: with no bits one pass still moves the
// source to the sink).
inline int passes_for(int bits) { return bits <= kMaxDigit ? 1 : (bits + kMaxDigit - 1) / kMaxDigit; }

inline size_t count_bytes(int64_t n) {
  return align_up(sizeof(int32_t) * kMaxBins * static_cast<size_t>(tiles_of(n > 0 ? n : 1))) +
         align_up(sizeof(int32_t) * kMaxBins);
}

// Payload of a sort or partition of keys alone.
struct NoVal {
  __device__ __forceinline__ explicit NoVal(int = 0) {}
};

// A source gives raw(i), what is loaded for element i's key, and key(raw);
// they are apart so that a tile's loads are all issued before any use.
// check(raw) is called once per element, in the first pass's count.

// Pairs in two arrays: a source, and a sink for any pass.
template <typename K, typename V>
struct Pairs {
  K* k;
  V* v;
  __device__ __forceinline__ K raw(int64_t i) const { return k[i]; }
  __device__ __forceinline__ K key(K x) const { return x; }
  __device__ __forceinline__ void check(K) const {}
  __device__ __forceinline__ V val(int64_t i) const { return v[i]; }
  __device__ __forceinline__ void put_key(int64_t i, K x) const { k[i] = x; }
  __device__ __forceinline__ void put_val(int64_t i, V x) const { v[i] = x; }
};

__device__ __forceinline__ int32_t wave_incl_scan(int32_t v, int lane) {
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    const int32_t u = __shfl_up(v, off, kWave);
    if (lane >= off) v += u;
  }
  return v;
}

// Exclusive scan of one value per thread over the 256-thread workgroup;
// wsum: kWaves ints of LDS, free again after the call.
__device__ __forceinline__ int32_t block_excl_scan(int32_t v, int32_t* wsum, int32_t* total) {
  const int t = threadIdx.x, lane = t % kWave, w = t / kWave;
  const int32_t inc = wave_incl_scan(v, lane);
  if (lane == kWave - 1) wsum[w] = inc;
  __syncthreads();
  int32_t before = 0, all = 0;
#pragma unroll
  for (int i = 0; i < kWaves; ++i) {
    if (i < w) before += wsum[i];
    all += wsum[i];
  }
  __syncthreads();
  *total = all;
  return before + inc - v;
}

// Digit counts of each tile, digit-major: hist[d * ntiles + tile].
template <int DB, class Src>
__global__ __launch_bounds__(kWG) void k_count(const Src src, int64_t n, int shift, uint32_t mask,
                                               int32_t* __restrict__ hist, int32_t ntiles) {
  constexpr int NB = 1 << DB;
  __shared__ int32_t cnt[NB];
  const int t = threadIdx.x;
  const int tile = xcd_tile(blockIdx.x, gridDim.x);
  if (tile >= ntiles) return;
  for (int d = t; d < NB; d += kWG) cnt[d] = 0;
  const int64_t base = static_cast<int64_t>(tile) * kTile;
  decltype(src.raw(0)) raw[kItems];
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    const int64_t i = base + j * kWG + t;
    if (i < n) raw[j] = src.raw(i);
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kItems; ++j)
    if (base + j * kWG + t < n) {
      src.check(raw[j]);
      atomicAdd(&cnt[static_cast<uint32_t>(src.key(raw[j]) >> shift) & mask], 1);
    }
  __syncthreads();
  for (int d = t; d < NB; d += kWG) hist[static_cast<int64_t>(d) * ntiles + tile] = cnt[d];
}

// Exclusive scan over the tiles of each digit (one workgroup per digit, in
// place) and the digit's total.
static __global__ __launch_bounds__(kWG) void k_scan_digits(int32_t* __restrict__ hist, int32_t ntiles,
                                                            int32_t* __restrict__ totals) {
  constexpr int kPer = 4;
  __shared__ int32_t wsum[kWaves];
  int32_t* h = hist + static_cast<int64_t>(blockIdx.x) * ntiles;
  int32_t carry = 0;
  for (int32_t base = 0; base < ntiles; base += kWG * kPer) {
    int32_t x[kPer], s = 0;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      const int32_t i = base + static_cast<int32_t>(threadIdx.x) * kPer + j;
      x[j] = i < ntiles ? h[i] : 0;
      s += x[j];
    }
    int32_t all;
    int32_t run = carry + block_excl_scan(s, wsum, &all);
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      const int32_t i = base + static_cast<int32_t>(threadIdx.x) * kPer + j;
      if (i < ntiles) h[i] = run;
      run += x[j];
    }
    carry += all;
  }
  if (threadIdx.x == 0) totals[blockIdx.x] = carry;
}

// Stable scatter of one tile.  Wavefront w holds the tile's elements
// [1024 w, 1024 (w + 1)), 64 at a time in input order; lanes with the same
// digit find each other by ballots over the digit's bits, and the first of
// them advances the wavefront's counter (one wavefront's LDS accesses are
// performed in order, so the next round reads the advanced value).
template <int DB, class Src, class Dst>
__global__ __launch_bounds__(kWG) void k_scatter(const Src src, const Dst dst, int64_t n, int shift, uint32_t mask,
                                                 const int32_t* __restrict__ hist,
                                                 const int32_t* __restrict__ totals, int32_t ntiles) {
  using K = decltype(src.key(src.raw(0)));
  using V = decltype(src.val(0));
  constexpr int NB = 1 << DB;
  constexpr int PERD = NB / kWG;  // digits per thread
  static_assert(NB >= kWG && kTile <= 65535, "digits per thread; 16-bit ranks");
  constexpr size_t kElem = sizeof(K) > sizeof(V) ? sizeof(K) : sizeof(V);
  constexpr bool kVal = !std::is_same<V, NoVal>::value;
  __shared__ __align__(16) char s_buf[kTile * kElem];
  __shared__ uint16_t s_cnt[kWaves][NB];
  __shared__ int32_t s_goff[NB];
  __shared__ int32_t s_wsum[kWaves];
  K* s_key = reinterpret_cast<K*>(s_buf);
  V* s_val = reinterpret_cast<V*>(s_buf);
  const int t = threadIdx.x, lane = t % kWave, w = t / kWave;
  const int tile = xcd_tile(blockIdx.x, gridDim.x);
  if (tile >= ntiles) return;
  const int64_t base = static_cast<int64_t>(tile) * kTile;
  const int32_t here = static_cast<int32_t>(n - base < kTile ? n - base : kTile);
  const uint64_t lt_mask = (lane == 0) ? 0ull : ((~0ull) >> (64 - lane));

  K key[kItems];
  V val[kVal ? kItems : 1];
  int32_t before[PERD], gtot[PERD];  // this tile's offset in each digit, and the digit's total
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    const int32_t i = w * (kTile / kWaves) + j * kWave + lane;
    key[j] = i < here ? src.key(src.raw(base + i)) : K(0);
    if constexpr (kVal) val[j] = i < here ? src.val(base + i) : V(0);
  }
#pragma unroll
  for (int j = 0; j < PERD; ++j) {
    const int d = t * PERD + j;
    before[j] = hist[static_cast<int64_t>(d) * ntiles + tile];
    gtot[j] = totals[d];
  }
  for (int i = t; i < kWaves * NB; i += kWG) (&s_cnt[0][0])[i] = 0;
  __syncthreads();
  uint16_t rank[kItems];
  volatile uint16_t* cnt = s_cnt[w];
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    const bool valid = w * (kTile / kWaves) + j * kWave + lane < here;
    const uint32_t d = static_cast<uint32_t>(key[j] >> shift) & mask;
    uint64_t peers = __ballot(valid);
#pragma unroll
    for (int b = 0; b < DB; ++b) {
      const bool bit = (d >> b) & 1u;
      const uint64_t bal = __ballot(bit);
      peers &= bit ? bal : ~bal;
    }
    const int r = __popcll(peers & lt_mask);
    const uint16_t old = cnt[d];
    rank[j] = static_cast<uint16_t>(old + r);
    if (valid && r == 0) cnt[d] = static_cast<uint16_t>(old + __popcll(peers));
  }
  __syncthreads();
  // counters become start positions: by digit, then by wavefront
  int32_t tot[PERD], mine = 0, gmine = 0, all;
#pragma unroll
  for (int j = 0; j < PERD; ++j) {
    int32_t run = 0;
#pragma unroll
    for (int v = 0; v < kWaves; ++v) {
      const int32_t c = s_cnt[v][t * PERD + j];
      s_cnt[v][t * PERD + j] = static_cast<uint16_t>(run);
      run += c;
    }
    tot[j] = run;
    mine += run;
    gmine += gtot[j];
  }
  int32_t start = block_excl_scan(mine, s_wsum, &all);
  int32_t gstart = block_excl_scan(gmine, s_wsum, &all);
#pragma unroll
  for (int j = 0; j < PERD; ++j) {
    const int d = t * PERD + j;
#pragma unroll
    for (int v = 0; v < kWaves; ++v) s_cnt[v][d] = static_cast<uint16_t>(s_cnt[v][d] + start);
    s_goff[d] = gstart + before[j] - start;
    start += tot[j];
    gstart += gtot[j];
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    const bool valid = w * (kTile / kWaves) + j * kWave + lane < here;
    rank[j] = static_cast<uint16_t>(rank[j] + s_cnt[w][static_cast<uint32_t>(key[j] >> shift) & mask]);
    if (valid) s_key[rank[j]] = key[j];
  }
  __syncthreads();
  int32_t to[kItems];
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    const int32_t i = j * kWG + t;
    if (i < here) {
      const K k = s_key[i];
      to[j] = s_goff[static_cast<uint32_t>(k >> shift) & mask] + i;
      dst.put_key(to[j], k);
    }
  }
  if constexpr (kVal) {
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kItems; ++j)
      if (w * (kTile / kWaves) + j * kWave + lane < here) s_val[rank[j]] = val[j];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kItems; ++j)
      if (j * kWG + t < here) dst.put_val(to[j], s_val[j * kWG + t]);
  }
}

// A round of a kWG-way search of rows lo < hi <= 2^31 - 1: thread t looks at
// row search_at, and `all` of them (a prefix) being at or before the sought
// row narrows the range.  No intermediate leaves int32 or is formed in it.
__host__ __device__ inline int32_t search_step(int32_t lo, int32_t hi) { return (hi - lo - 1) / kWG + 1; }
__host__ __device__ inline int64_t search_at(int32_t lo, int32_t step, int t) {
  return static_cast<int64_t>(lo) + static_cast<int64_t>(t + 1) * step;
}
__host__ __device__ inline void search_narrow(int32_t& lo, int32_t& hi, int32_t step, int32_t all) {
  lo += all * step;  // below hi: the rows counted are
  const int64_t end = static_cast<int64_t>(lo) + step;
  if (end < hi) hi = static_cast<int32_t>(end);
}

// Rows of the nonzeros [base, base + here) of a CSR pattern, here <= kTile:
// row[j] belongs to position base + 1024 w + 64 j + lane (w: wavefront).  The
// tile's first row is found by a 256-way search of rowptr, every later
// non-empty row marks its first nonzero in s_row (kTile ints of LDS), and a
// running maximum fills the gaps: a row is looked at by one thread, whatever
// its length.  A tile that spans more than kTileSpan rows (runs of empty rows;
// 64 rounds of the walk, 0.3 us each) searches rowptr for each nonzero
// instead: 5,000 nonzeros in 10 M rows took 12.1 ms for the CSC index when
// one workgroup walked them all.  Called by the whole workgroup.
__device__ __forceinline__ void tile_rows(const int32_t* __restrict__ rowptr, int32_t m, int32_t base, int32_t here,
                                          int32_t* s_row, int32_t* s_wsum, int32_t (&row)[kItems]) {
  const int t = threadIdx.x, lane = t % kWave, w = t / kWave;
  int32_t lo = 0, hi = m;  // rowptr[lo] <= base < rowptr[hi]
  while (hi - lo > 1) {
    const int32_t step = search_step(lo, hi);
    const int64_t at = search_at(lo, step, t);
    const bool below = at < hi && rowptr[at] <= base;
    const int c = __popcll(__ballot(below));
    if (lane == 0) s_wsum[w] = c;
    __syncthreads();
    int32_t all = 0;
#pragma unroll
    for (int i = 0; i < kWaves; ++i) all += s_wsum[i];
    __syncthreads();
    search_narrow(lo, hi, step, all);
  }
  const bool far = static_cast<int64_t>(lo) + kTileSpan < m && rowptr[lo + kTileSpan] < base + here;
  for (int i = t; i < kTile; i += kWG) s_row[i] = lo;
  if (far) {
    // the last row that starts at or before the nonzero, by halving steps
    int32_t step = 1;
    while (step <= (m - 1 - lo) / 2) step *= 2;
#pragma unroll
    for (int j = 0; j < kItems; ++j) row[j] = lo;
    for (; step > 0; step /= 2) {
      int32_t at[kItems];
#pragma unroll
      for (int j = 0; j < kItems; ++j) {
        const int64_t r = static_cast<int64_t>(row[j]) + step;
        at[j] = r < m ? rowptr[r] : 0x7fffffff;
      }
#pragma unroll
      for (int j = 0; j < kItems; ++j) {
        const int32_t i = w * (kTile / kWaves) + j * kWave + lane;
        if (at[j] <= base + min(i, here - 1)) row[j] += step;
      }
    }
    return;
  }
  __syncthreads();
  for (int64_t r = static_cast<int64_t>(lo) + 1 + t; r < m; r += kWG) {
    const int32_t q = rowptr[r];
    if (q >= base + here) break;
    if (q > base && rowptr[r + 1] > q) s_row[q - base] = static_cast<int32_t>(r);
  }
  __syncthreads();
  int32_t carry = lo;
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    int32_t v = max(carry, s_row[w * (kTile / kWaves) + j * kWave + lane]);
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
      const int32_t u = __shfl_up(v, off, kWave);
      if (lane >= off) v = max(v, u);
    }
    row[j] = v;
    carry = __shfl(v, kWave - 1, kWave);
  }
  if (lane == 0) s_wsum[w] = carry;
  __syncthreads();
  int32_t before = lo;
  for (int i = 0; i < w; ++i) before = max(before, s_wsum[i]);
#pragma unroll
  for (int j = 0; j < kItems; ++j) row[j] = max(row[j], before);
  __syncthreads();
}

template <class Src, class Dst>
spx_status pass(const Src& src, const Dst& dst, int64_t n, int shift, int width, void* counts, hipStream_t st) {
  const int32_t ntiles = static_cast<int32_t>(tiles_of(n));
  const unsigned grid = (static_cast<unsigned>(ntiles) + 7) / 8 * 8;
  const uint32_t mask = (1u << width) - 1u;
  int32_t* hist = static_cast<int32_t*>(counts);
  int32_t* totals = reinterpret_cast<int32_t*>(static_cast<char*>(counts) +
                                               align_up(sizeof(int32_t) * kMaxBins * static_cast<size_t>(ntiles)));
  if (width <= 8) {
    k_count<8><<<grid, kWG, 0, st>>>(src, n, shift, mask, hist, ntiles);
    SPX_LAUNCHED("radix::k_count");
    k_scan_digits<<<1 << 8, kWG, 0, st>>>(hist, ntiles, totals);
    SPX_LAUNCHED("radix::k_scan_digits");
    k_scatter<8><<<grid, kWG, 0, st>>>(src, dst, n, shift, mask, hist, totals, ntiles);
  } else {
    k_count<kMaxDigit><<<grid, kWG, 0, st>>>(src, n, shift, mask, hist, ntiles);
    SPX_LAUNCHED("radix::k_count");
    k_scan_digits<<<kMaxBins, kWG, 0, st>>>(hist, ntiles, totals);
    SPX_LAUNCHED("radix::k_scan_digits");
    k_scatter<kMaxDigit><<<grid, kWG, 0, st>>>(src, dst, n, shift, mask, hist, totals, ntiles);
  }
  SPX_LAUNCHED("radix::k_scatter");
  return SPX_OK;
}

// Sort n >= 1 pairs of `src` by the low `bits` key bits into `last`, in
// `passes` >= passes_for(bits) passes.  Passes before the last one write `a`,
// then `b`, then `a` again: `last` may be the pair of arrays that the final
// intermediate pass does not use (`a` for an odd number of passes, `b` for an
// even one).  The first pass alone reads `src`, all of it while it writes: `b`
// may be the arrays `src` reads; `a` may not, nor may `last` if there is one
// pass.
template <typename K, typename V, class Src, class Dst>
spx_status sort(const Src& src, const Pairs<K, V>& a, const Pairs<K, V>& b, const Dst& last, int64_t n, int bits,
                int passes, void* counts, hipStream_t st) {
  const int width = (bits + passes - 1) / passes;
  spx_status s = SPX_OK;
  for (int p = 0; p < passes && s == SPX_OK; ++p) {
    const int shift = p * width;
    const bool fin = p + 1 == passes;
    const Pairs<K, V>& from = (p & 1) ? a : b;
    const Pairs<K, V>& to = (p & 1) ? b : a;
    if (p == 0) s = fin ? pass(src, last, n, shift, width, counts, st) : pass(src, to, n, shift, width, counts, st);
    else s = fin ? pass(from, last, n, shift, width, counts, st) : pass(from, to, n, shift, width, counts, st);
  }
  return s;
}

}  // namespace radix
}  // namespace spx
