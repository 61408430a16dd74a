// assemble.hip -- CSR assembly from triplets, structural validation and the
// CSC index of the transpose, all on the device.
//
// CRS (paper Sec. 3): rowptr[0] = 0, rowptr[m] = tau, the column ids of row i
// in colind[rowptr[i] .. rowptr[i+1]-1].  Canonical form here: columns
// strictly ascending inside a row; duplicate (i, j) triplets summed in input
// order.  A stable radix sort on the key (row, column) keeps duplicates in
// input order, so each run is summed front to back with plain FP64 adds.  The values travel
// with the keys: fetching them by position after the sort costs a random
// 8-byte read per triplet, more than the 4 bytes per triplet and pass that an
// index would save.
#include "device.hpp"
#include "internal.hpp"
#include "radix.hpp"

namespace spx {

namespace {

// Triplets as the source of the first sort pass.  A triplet out of range sets
// *bad and sorts as (0, 0).
struct CooSrc {
  const int32_t* r;
  const int32_t* c;
  const double* v;
  int32_t m, n;
  int cbits;
  int32_t* bad;
  __device__ __forceinline__ int2 raw(int64_t i) const { return make_int2(r[i], c[i]); }
  __device__ __forceinline__ bool ok(int2 x) const {
    return static_cast<uint32_t>(x.x) < static_cast<uint32_t>(m) && static_cast<uint32_t>(x.y) < static_cast<uint32_t>(n);
  }
  __device__ __forceinline__ uint64_t key(int2 x) const {
    return ok(x) ? (static_cast<uint64_t>(x.x) << cbits) | static_cast<uint64_t>(x.y) : 0;
  }
  __device__ __forceinline__ void check(int2 x) const {
    if (!ok(x)) atomicOr(bad, 1);
  }
  __device__ __forceinline__ double val(int64_t i) const { return v[i]; }
};

// Heads of a tile: sorted positions whose key differs from the one before.
__device__ __forceinline__ bool is_head(const uint64_t* keys, int64_t i) { return i == 0 || keys[i] != keys[i - 1]; }

__global__ __launch_bounds__(kWG) void k_count_heads(const uint64_t* __restrict__ keys, int64_t nnz,
                                                     int32_t* __restrict__ counts) {
  __shared__ int32_t wsum[radix::kWaves];
  const int64_t base = static_cast<int64_t>(blockIdx.x) * radix::kTile;
  int32_t c = 0, all;
#pragma unroll
  for (int j = 0; j < radix::kItems; ++j) {
    const int64_t i = base + j * kWG + threadIdx.x;
    if (i < nnz) c += is_head(keys, i);
  }
  (void)radix::block_excl_scan(c, wsum, &all);
  if (threadIdx.x == 0) counts[blockIdx.x] = all;
}

// Each lane stores `value` at the `count` entries of p that begin with `from`.
// A lane's few entries it stores itself; longer runs the wavefront stores one
// after the other, 64 entries at a time (runs of empty rows: 5,000 triplets of
// 10 M rows leave 2,000 entries to each head).  Called by the whole wavefront.
__device__ __forceinline__ void wave_fill(int32_t* __restrict__ p, uint32_t from, uint32_t count, int32_t value) {
  constexpr uint32_t kOwn = 8;
  uint64_t runs = __ballot(count > kOwn);
  if (count <= kOwn)
    for (uint32_t i = 0; i < count; ++i) p[static_cast<size_t>(from) + i] = value;
  while (runs) {
    const int l = __ffsll(static_cast<unsigned long long>(runs)) - 1;
    runs &= runs - 1;
    int32_t* f = p + static_cast<uint32_t>(__shfl(static_cast<int>(from), l, kWave));
    const uint32_t n = static_cast<uint32_t>(__shfl(static_cast<int>(count), l, kWave));
    const int32_t v = __shfl(value, l, kWave);
    for (uint32_t i = threadIdx.x % kWave; i < n; i += kWave) f[i] = v;
  }
}

// Every head emits its run.  offs: the exclusive scan of the tiles' head
// counts; a head's place inside the tile comes from ballots, in sorted order.
// gridDim.y (a power of two) workgroups share a tile, each emitting every
// gridDim.y-th of its 64-position pieces (emit_share).
__global__ __launch_bounds__(kWG) void k_emit(const uint64_t* __restrict__ keys, const double* __restrict__ v,
                                              const int32_t* __restrict__ offs, const int32_t* __restrict__ bad,
                                              const int32_t* __restrict__ total, int64_t nnz, int32_t m, int cbits,
                                              int32_t* __restrict__ rowptr, int32_t* __restrict__ colind,
                                              double* __restrict__ values, int32_t* __restrict__ nnz_out) {
  __shared__ int32_t wcnt[radix::kWaves];
  const int t = threadIdx.x, lane = t % kWave, w = t / kWave;
  const uint64_t lt_mask = (lane == 0) ? 0ull : ((~0ull) >> (64 - lane));
  const int64_t base = static_cast<int64_t>(blockIdx.x) * radix::kTile + w * (radix::kTile / radix::kWaves);
  if (blockIdx.x == 0 && blockIdx.y == 0 && t == 0) *nnz_out = (*bad) ? -1 : *total;
  // the wavefront's keys and values, all loads issued at once; the key before
  // each comes from the lane before it
  uint64_t key[radix::kItems], heads[radix::kItems];
  double val[radix::kItems];
#pragma unroll
  for (int j = 0; j < radix::kItems; ++j) {
    const int64_t i = base + j * kWave + lane;
    key[j] = i < nnz ? keys[i] : ~0ull;
    val[j] = i < nnz ? v[i] : 0.0;
  }
  uint64_t carry = (base > 0 && base < nnz) ? keys[base - 1] : ~0ull;
  const uint64_t first = carry;
  int32_t mine = 0;
#pragma unroll
  for (int j = 0; j < radix::kItems; ++j) {
    const int64_t i = base + j * kWave + lane;
    const uint64_t up = __shfl_up(key[j], 1, kWave);
    const uint64_t prev = lane == 0 ? carry : up;
    heads[j] = __ballot(i < nnz && (i == 0 || key[j] != prev));
    carry = __shfl(key[j], kWave - 1, kWave);
    mine += __popcll(heads[j]);
  }
  if (lane == 0) wcnt[w] = mine;
  __syncthreads();
  int32_t run = offs[blockIdx.x];
  for (int i = 0; i < w; ++i) run += wcnt[i];
  const uint64_t cmask = (1ull << cbits) - 1ull;
  carry = first;
  uint32_t after = static_cast<uint32_t>(m) + 1u;  // the head of the last run: rows from here hold nothing
  int32_t total_out = 0;
#pragma unroll
  for (int j = 0; j < radix::kItems; ++j) {
    const int64_t i = base + j * kWave + lane;
    const uint64_t up = __shfl_up(key[j], 1, kWave);
    const uint64_t before = lane == 0 ? carry : up;
    carry = __shfl(key[j], kWave - 1, kWave);
    if ((j & (gridDim.y - 1)) != blockIdx.y) {
      run += __popcll(heads[j]);
      continue;
    }
    uint32_t from = 0, count = 0;  // rows whose offset this head sets
    int32_t out = 0;
    if ((heads[j] >> lane) & 1) {
      out = run + __popcll(heads[j] & lt_mask);
      double s = val[j];
      int64_t q = i + 1;
      // a run of one, unless the next position of this wavefront's 64 is no head
      const bool alone = lane + 1 < kWave && q < nnz && ((heads[j] >> (lane + 1)) & 1);
      if (!alone)
        while (q < nnz && keys[q] == key[j]) {
          s = s + v[q];
          ++q;
        }
      colind[out] = static_cast<int32_t>(key[j] & cmask);
      values[out] = s;
      const int32_t row = static_cast<int32_t>(key[j] >> cbits);
      from = (i == 0) ? 0u : static_cast<uint32_t>(before >> cbits) + 1u;
      count = static_cast<uint32_t>(row) + 1u - from;
      if (q == nnz) {
        after = static_cast<uint32_t>(row) + 1u;
        total_out = out + 1;
      }
    }
    wave_fill(rowptr, from, count, out);
    run += __popcll(heads[j]);
  }
  wave_fill(rowptr, after, static_cast<uint32_t>(m) + 1u - after, total_out);
}

__global__ void k_fill_i32(int32_t* __restrict__ p, int64_t n, int32_t value) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) p[i] = value;
}

__global__ void k_validate(int32_t m, int32_t n, int32_t nnz, const int32_t* __restrict__ rowptr,
                           const int32_t* __restrict__ colind, int32_t check_sorted,
                           int32_t* __restrict__ status) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i == 0 && (rowptr[0] != 0 || rowptr[m] != nnz)) atomicMax(status, 4);
  if (i >= m) return;
  const int32_t a = rowptr[i], b = rowptr[i + 1];
  if (a < 0 || b > nnz || a > b) {
    atomicMax(status, 3);
    return;
  }
  int32_t last = -1;
  for (int32_t p = a; p < b; ++p) {
    const int32_t c = colind[p];
    if (c < 0 || c >= n) {
      atomicMax(status, 2);
      return;
    }
    if (check_sorted && c <= last) {
      atomicMax(status, 1);
      return;
    }
    last = c;
  }
}

// Row of each nonzero.
__global__ __launch_bounds__(kWG) void k_expand_rows(const int32_t* __restrict__ rowptr, int32_t m, int32_t nnz,
                                                     int32_t* __restrict__ rowid) {
  __shared__ int32_t s_row[radix::kTile];
  __shared__ int32_t s_wsum[radix::kWaves];
  const int t = threadIdx.x, lane = t % kWave, w = t / kWave;
  const int32_t base = static_cast<int32_t>(blockIdx.x) * radix::kTile;
  const int32_t here = min(radix::kTile, nnz - base);
  int32_t row[radix::kItems];
  radix::tile_rows(rowptr, m, base, here, s_row, s_wsum, row);
#pragma unroll
  for (int j = 0; j < radix::kItems; ++j) {
    const int32_t i = w * (radix::kTile / radix::kWaves) + j * kWave + lane;
    if (i < here) rowid[base + i] = row[j];
  }
}

// CSR nonzeros as the source of a sort by column: the payload is the row and
// the CSR position, so neither is looked up after the sort.
struct ColSrc {
  const int32_t* colind;
  const int32_t* rowid;
  __device__ __forceinline__ uint32_t raw(int64_t i) const { return static_cast<uint32_t>(colind[i]); }
  __device__ __forceinline__ uint32_t key(uint32_t x) const { return x; }
  __device__ __forceinline__ void check(uint32_t) const {}
  __device__ __forceinline__ uint64_t val(int64_t i) const {
    return (static_cast<uint64_t>(static_cast<uint32_t>(rowid[i])) << 32) | static_cast<uint64_t>(i);
  }
};

struct CscSink {
  uint32_t* keys;
  int32_t* rowind;
  int32_t* perm;
  __device__ __forceinline__ void put_key(int64_t q, uint32_t k) const { keys[q] = k; }
  __device__ __forceinline__ void put_val(int64_t q, uint64_t v) const {
    rowind[q] = static_cast<int32_t>(v >> 32);
    perm[q] = static_cast<int32_t>(v & 0xffffffffu);
  }
};

// colptr from the column boundaries of the sorted columns.
__global__ void k_colptr(const uint32_t* __restrict__ keys, int32_t n, int64_t nnz, int32_t* __restrict__ colptr) {
  const int64_t q = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  const bool in = q < nnz;
  // column ids are assumed valid (0 <= col < n); a bad one counts as the last
  // column (none, -1, for n = 0), so it cannot write outside colptr[0 .. n]
  auto clamp = [n](uint32_t k) { return k < static_cast<uint32_t>(n) ? static_cast<int32_t>(k) : n - 1; };
  const int32_t prev = (in && q > 0) ? clamp(keys[q - 1]) : -1;
  const int32_t col = in ? clamp(keys[q]) : prev;
  wave_fill(colptr, static_cast<uint32_t>(prev + 1), col > prev ? static_cast<uint32_t>(col - prev) : 0u,
            static_cast<int32_t>(q));
  if (blockIdx.x + 1 == gridDim.x)
    wave_fill(colptr, static_cast<uint32_t>(col + 1), q == nnz - 1 ? static_cast<uint32_t>(n - col) : 0u,
              static_cast<int32_t>(nnz));
}

inline unsigned grid_for(int64_t n, int bs = 256) {
  return static_cast<unsigned>((n + bs - 1) / bs);
}

// Workgroups per tile of the emission: enough that few triplets (5,000 are two
// tiles) still spread over the device, which their runs of empty rows need.
unsigned emit_share(unsigned tiles) {
  unsigned share = 1;
  while (share < radix::kItems && tiles * share * 2 <= 512) share *= 2;
  return share;
}

struct CooWs {
  uint64_t* keys[2];
  double* vals;
  int32_t* counts;
  int32_t* bad;
  int32_t* total;
  void* radix;
  void* scan;
};

CooWs carve_coo(void* ws, int64_t nnz, size_t* bytes) {
  Carve cv(ws, ~size_t(0));
  const int64_t e = nnz > 0 ? nnz : 1;
  CooWs w;
  w.keys[0] = cv.take<uint64_t>(e);
  w.keys[1] = cv.take<uint64_t>(e);
  w.vals = cv.take<double>(e);
  w.counts = cv.take<int32_t>(radix::tiles_of(e));
  w.bad = cv.take<int32_t>(1);
  w.total = cv.take<int32_t>(1);
  w.radix = cv.take<char>(radix::count_bytes(e));
  w.scan = cv.take<char>(scan_workspace_bytes(radix::tiles_of(e)));
  *bytes = cv.used;
  return w;
}

struct CscWs {
  int32_t* rowid;
  uint32_t* keys[2];
  uint64_t* vals[2];
  void* radix;
};

// Passes before the last write keys[0] / vals[0] and, from three passes on,
// keys[1] / vals[1]; the last one leaves its keys in the pair it does not read.
CscWs carve_csc(void* ws, int32_t n, int64_t nnz, size_t* bytes) {
  Carve cv(ws, ~size_t(0));
  const int64_t e = nnz > 0 ? nnz : 1;
  CscWs w;
  w.rowid = cv.take<int32_t>(e);
  w.keys[0] = cv.take<uint32_t>(e);
  w.keys[1] = cv.take<uint32_t>(e);
  w.vals[0] = cv.take<uint64_t>(e);
  w.vals[1] = cv.take<uint64_t>(radix::passes_for(bits_for(n > 0 ? n - 1 : 0)) > 2 ? e : 1);
  w.radix = cv.take<char>(radix::count_bytes(e));
  *bytes = cv.used;
  return w;
}

}  // namespace
}  // namespace spx

using namespace spx;

extern "C" spx_status csr_from_coo_workspace_bytes(int32_t m, int32_t n, int64_t nnz_in,
                                                   size_t* bytes) {
  if (!bytes) return fail(SPX_ERR_INVALID, "csr_from_coo_workspace_bytes: bytes is null");
  if (m < 0 || n < 0 || nnz_in < 0)
    return fail(SPX_ERR_INVALID, "csr_from_coo_workspace_bytes: bad sizes m=%d n=%d nnz=%lld", m, n,
                (long long)nnz_in);
  {
    const spx_status s_nnz = check_nnz(nnz_in, "csr_from_coo_workspace_bytes");
    if (s_nnz != SPX_OK) return s_nnz;
  }
  carve_coo(nullptr, nnz_in, bytes);
  return SPX_OK;
}

extern "C" spx_status csr_from_coo(int32_t m, int32_t n, int64_t nnz_in, const int32_t* r,
                                   const int32_t* c, const double* v, int32_t* rowptr,
                                   int32_t* colind, double* values, int32_t* nnz_out,
                                   void* workspace, size_t ws_bytes, void* stream) {
  if (m < 0 || n < 0 || nnz_in < 0)
    return fail(SPX_ERR_INVALID, "csr_from_coo: bad sizes m=%d n=%d nnz=%lld", m, n, (long long)nnz_in);
  {
    const spx_status s_nnz = check_nnz(nnz_in, "csr_from_coo");
    if (s_nnz != SPX_OK) return s_nnz;
  }
  if (!rowptr || !nnz_out) return fail(SPX_ERR_INVALID, "csr_from_coo: null rowptr or nnz_out");
  if (nnz_in > 0 && (!r || !c || !v || !colind || !values))
    return fail(SPX_ERR_INVALID, "csr_from_coo: null triplet or output array");
  if (nnz_in > 0 && (m == 0 || n == 0))
    return fail(SPX_ERR_INVALID, "csr_from_coo: triplets given for an empty shape");
  size_t need;
  carve_coo(nullptr, nnz_in, &need);
  if (!workspace || ws_bytes < need)
    return fail(SPX_ERR_WORKSPACE, "csr_from_coo: workspace %zu < %zu bytes", ws_bytes, need);
  hipStream_t st = as_stream(stream);
  CooWs w = carve_coo(workspace, nnz_in, &need);
  const int cbits = bits_for(n > 0 ? n - 1 : 0);
  const int rbits = bits_for(m > 0 ? m - 1 : 0);
  k_fill_i32<<<1, 64, 0, st>>>(w.bad, 1, 0);
  SPX_LAUNCHED("k_fill_i32");
  if (nnz_in == 0) {
    k_fill_i32<<<grid_for(int64_t(m) + 1), 256, 0, st>>>(rowptr, int64_t(m) + 1, 0);
    SPX_LAUNCHED("k_fill_i32");
    k_fill_i32<<<1, 64, 0, st>>>(nnz_out, 1, 0);
    SPX_LAUNCHED("k_fill_i32");
    return SPX_OK;
  }
  // The last pass lands in the workspace, and the output `values` serves as
  // the other payload buffer (k_emit reads sorted pairs while it writes).  An
  // even number of passes writes `values` first in pass 0, beside other tiles'
  // reads of the triplets; where the two share memory (a permutation in place)
  // one more pass makes the number odd, and pass 0 then writes the workspace.
  const int bits = cbits + rbits;
  int passes = radix::passes_for(bits);
  const size_t vbytes = sizeof(double) * static_cast<size_t>(nnz_in), ibytes = vbytes / 2;
  if (overlap(values, vbytes, v, vbytes) || overlap(values, vbytes, r, ibytes) || overlap(values, vbytes, c, ibytes))
    passes |= 1;
  const int fin = (passes & 1) ? 0 : 1;
  radix::Pairs<uint64_t, double> buf[2];
  for (int i = 0; i < 2; ++i) buf[i] = {w.keys[i], i == fin ? w.vals : values};
  const CooSrc src{r, c, v, m, n, cbits, w.bad};
  spx_status s = radix::sort(src, buf[0], buf[1], buf[fin], nnz_in, bits, passes, w.radix, st);
  if (s != SPX_OK) return s;
  const unsigned tiles = static_cast<unsigned>(radix::tiles_of(nnz_in));
  k_count_heads<<<tiles, kWG, 0, st>>>(buf[fin].k, nnz_in, w.counts);
  SPX_LAUNCHED("k_count_heads");
  s = exclusive_scan_i32(w.counts, w.counts, tiles, w.total, w.scan, st);
  if (s != SPX_OK) return s;
  k_emit<<<dim3(tiles, emit_share(tiles)), kWG, 0, st>>>(buf[fin].k, buf[fin].v, w.counts, w.bad, w.total, nnz_in, m, cbits, rowptr, colind,
                                values, nnz_out);
  SPX_LAUNCHED("k_emit");
  return SPX_OK;
}

extern "C" spx_status csr_validate(int32_t m, int32_t n, int32_t nnz, const int32_t* rowptr,
                                   const int32_t* colind, int32_t check_sorted,
                                   int32_t* status_out, void* stream) {
  if (m < 0 || n < 0 || nnz < 0) return fail(SPX_ERR_INVALID, "csr_validate: negative size");
  {
    const spx_status s_nnz = check_nnz(nnz, "csr_validate");
    if (s_nnz != SPX_OK) return s_nnz;
  }
  if (!rowptr || !status_out || (nnz > 0 && !colind))
    return fail(SPX_ERR_INVALID, "csr_validate: null pointer");
  hipStream_t st = as_stream(stream);
  k_fill_i32<<<1, 64, 0, st>>>(status_out, 1, 0);
  SPX_LAUNCHED("k_fill_i32");
  k_validate<<<grid_for(int64_t(m) + 1), 256, 0, st>>>(m, n, nnz, rowptr, colind, check_sorted,
                                                       status_out);
  SPX_LAUNCHED("k_validate");
  return SPX_OK;
}

namespace {
size_t transpose_ws(int32_t n, int64_t nnz) {
  size_t bytes;
  carve_csc(nullptr, n, nnz, &bytes);
  return bytes;
}
}  // namespace

extern "C" spx_status csr_transpose_index_workspace_bytes(int32_t m, int32_t n, int32_t nnz,
                                                          size_t* bytes) {
  if (!bytes || m < 0 || n < 0 || nnz < 0)
    return fail(SPX_ERR_INVALID, "csr_transpose_index_workspace_bytes: bad arguments");
  *bytes = transpose_ws(n, nnz);
  return SPX_OK;
}

extern "C" spx_status csr_transpose_index(int32_t m, int32_t n, int32_t nnz, const int32_t* rowptr,
                                          const int32_t* colind, int32_t* colptr, int32_t* rowind,
                                          int32_t* perm, void* workspace, size_t ws_bytes,
                                          void* stream) {
  if (m < 0 || n < 0 || nnz < 0) return fail(SPX_ERR_INVALID, "csr_transpose_index: negative size");
  {
    const spx_status s_nnz = check_nnz(nnz, "csr_transpose_index");
    if (s_nnz != SPX_OK) return s_nnz;
  }
  if (!colptr || (nnz > 0 && (!rowptr || !colind || !rowind || !perm)))
    return fail(SPX_ERR_INVALID, "csr_transpose_index: null pointer");
  if (!workspace || ws_bytes < transpose_ws(n, nnz))
    return fail(SPX_ERR_WORKSPACE, "csr_transpose_index: workspace %zu < %zu bytes", ws_bytes,
                transpose_ws(n, nnz));
  hipStream_t st = as_stream(stream);
  if (nnz == 0) {
    k_fill_i32<<<grid_for(int64_t(n) + 1), 256, 0, st>>>(colptr, int64_t(n) + 1, 0);
    SPX_LAUNCHED("k_fill_i32");
    return SPX_OK;
  }
  size_t need;
  const CscWs w = carve_csc(workspace, n, nnz, &need);
  const unsigned tiles = static_cast<unsigned>(radix::tiles_of(nnz));
  k_expand_rows<<<tiles, kWG, 0, st>>>(rowptr, m, nnz, w.rowid);
  SPX_LAUNCHED("k_expand_rows");
  const int bits = bits_for(n > 0 ? n - 1 : 0);
  int passes = radix::passes_for(bits);
  // a single pass would write rowind and perm beside other tiles' reads of colind
  const size_t bytes = sizeof(int32_t) * static_cast<size_t>(nnz);
  if (passes == 1 && (overlap(rowind, bytes, colind, bytes) || overlap(perm, bytes, colind, bytes))) passes = 2;
  const int fin = (passes & 1) ? 0 : 1;
  const radix::Pairs<uint32_t, uint64_t> a{w.keys[0], w.vals[0]}, b{w.keys[1], w.vals[1]};
  spx_status s = radix::sort(ColSrc{colind, w.rowid}, a, b, CscSink{w.keys[fin], rowind, perm}, nnz, bits, passes,
                             w.radix, st);
  if (s != SPX_OK) return s;
  k_colptr<<<grid_for(nnz), 256, 0, st>>>(w.keys[fin], n, nnz, colptr);
  SPX_LAUNCHED("k_colptr");
  return SPX_OK;
}
