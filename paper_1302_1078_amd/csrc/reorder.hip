// reorder.hip -- matrix ordering (paper Sec. 4.4) and the structure metrics
// it is judged by (Sec. 4.1 UCLD, Sec. 4.2 vector access).
//
// csr_rcm is host code: reverse Cuthill-McKee is a breadth-first search, a
// one-time preprocessing step whose cost the paper leaves out of its timings
// (Sec. 4.5).  csr_permute applies an ordering on the device (relabel the
// triplets, then the regular COO -> CSR assembly).
//
// RCM reading (the paper used MATLAB's implementation and states no tie
// rules): graph = pattern of A + A^T without the diagonal; components are
// numbered in turn, each from the unnumbered vertex of least (degree,
// index) moved to a pseudo-peripheral vertex by George and Liu's rule (go to
// the least-(degree, index) vertex of the last BFS level while that makes
// the level structure deeper); each vertex's unnumbered neighbours are
// appended in ascending (degree, index); the numbering is reversed at the end.
#include <stdlib.h>

#include <algorithm>
#include <new>
#include <vector>

#include "device.hpp"
#include "internal.hpp"
#include "radix.hpp"

namespace spx {
namespace {

// Undirected graph of the pattern of A + A^T, self loops dropped, every
// neighbour list sorted and free of repeats.
struct SymGraph {
  std::vector<int64_t> start;  // n + 1
  std::vector<int32_t> nbr;
  int32_t degree(int32_t v) const { return static_cast<int32_t>(start[v + 1] - start[v]); }
};

void build_sym(int32_t n, const int32_t* rowptr, const int32_t* colind, SymGraph& g) {
  std::vector<int64_t> fill(static_cast<size_t>(n) + 1, 0);
  for (int32_t i = 0; i < n; ++i)
    for (int32_t p = rowptr[i]; p < rowptr[i + 1]; ++p) {
      const int32_t j = colind[p];
      if (j == i) continue;
      ++fill[i + 1];
      ++fill[j + 1];
    }
  for (int32_t i = 0; i < n; ++i) fill[i + 1] += fill[i];
  std::vector<int32_t> raw(static_cast<size_t>(fill[n]));
  std::vector<int64_t> cur(fill.begin(), fill.end() - 1);
  for (int32_t i = 0; i < n; ++i)
    for (int32_t p = rowptr[i]; p < rowptr[i + 1]; ++p) {
      const int32_t j = colind[p];
      if (j == i) continue;
      raw[cur[i]++] = j;
      raw[cur[j]++] = i;
    }
  g.start.assign(static_cast<size_t>(n) + 1, 0);
  g.nbr.clear();
  g.nbr.reserve(raw.size());
  for (int32_t v = 0; v < n; ++v) {
    auto b = raw.begin() + fill[v], e = raw.begin() + fill[v + 1];
    std::sort(b, e);
    e = std::unique(b, e);
    g.nbr.insert(g.nbr.end(), b, e);
    g.start[v + 1] = static_cast<int64_t>(g.nbr.size());
  }
}

// Breadth-first level structure from `root` over vertices not yet numbered;
// `depth` is filled for the vertices reached (and reset by the caller's
// `touched` list).  Returns the number of levels; `last` gets the deepest level.
int32_t level_structure(const SymGraph& g, int32_t root, const std::vector<char>& numbered,
                        std::vector<int32_t>& depth, std::vector<int32_t>& touched,
                        std::vector<int32_t>& last) {
  for (int32_t v : touched) depth[v] = -1;
  touched.clear();
  depth[root] = 0;
  touched.push_back(root);
  size_t head = 0;
  int32_t deepest = 0;
  while (head < touched.size()) {
    const int32_t v = touched[head++];
    for (int64_t e = g.start[v]; e < g.start[v + 1]; ++e) {
      const int32_t w = g.nbr[e];
      if (numbered[w] || depth[w] >= 0) continue;
      depth[w] = depth[v] + 1;
      deepest = std::max(deepest, depth[w]);
      touched.push_back(w);
    }
  }
  last.clear();
  for (int32_t v : touched)
    if (depth[v] == deepest) last.push_back(v);
  return deepest + 1;
}

}  // namespace
}  // namespace spx

using namespace spx;

extern "C" spx_status csr_rcm(int32_t m, int32_t n, int32_t nnz, const int32_t* host_rowptr,
                              const int32_t* host_colind, int32_t* host_perm) {
  if (m < 0 || n < 0 || nnz < 0) return fail(SPX_ERR_INVALID, "csr_rcm: negative size");
  {
    const spx_status s_nnz = check_nnz(nnz, "csr_rcm");
    if (s_nnz != SPX_OK) return s_nnz;
  }
  if (m != n) return fail(SPX_ERR_INVALID, "csr_rcm: the matrix must be square (m=%d, n=%d)", m, n);
  if (m == 0) return SPX_OK;
  if (!host_rowptr || !host_perm || (nnz > 0 && !host_colind))
    return fail(SPX_ERR_INVALID, "csr_rcm: null pointer");
  if (host_rowptr[0] != 0 || host_rowptr[m] != nnz)
    return fail(SPX_ERR_INVALID, "csr_rcm: rowptr[0]=%d, rowptr[m]=%d, nnz=%d", host_rowptr[0],
                host_rowptr[m], nnz);
  for (int32_t i = 0; i < m; ++i)
    if (host_rowptr[i + 1] < host_rowptr[i]) return fail(SPX_ERR_INVALID, "csr_rcm: rowptr decreases at %d", i);
  for (int32_t p = 0; p < nnz; ++p)
    if (host_colind[p] < 0 || host_colind[p] >= n)
      return fail(SPX_ERR_INVALID, "csr_rcm: column %d out of range at %d", host_colind[p], p);
  try {
    SymGraph g;
    build_sym(n, host_rowptr, host_colind, g);
    auto before = [&g](int32_t a, int32_t b) {
      const int32_t da = g.degree(a), db = g.degree(b);
      return da != db ? da < db : a < b;
    };
    std::vector<int32_t> seeds(static_cast<size_t>(n));
    for (int32_t v = 0; v < n; ++v) seeds[v] = v;
    std::sort(seeds.begin(), seeds.end(), before);
    std::vector<char> numbered(static_cast<size_t>(n), 0);
    std::vector<int32_t> depth(static_cast<size_t>(n), -1), touched, last, fresh;
    std::vector<int32_t> cm;
    cm.reserve(static_cast<size_t>(n));
    size_t next_seed = 0;
    while (cm.size() < static_cast<size_t>(n)) {
      while (numbered[seeds[next_seed]]) ++next_seed;
      int32_t root = seeds[next_seed];
      int32_t levels = level_structure(g, root, numbered, depth, touched, last);
      for (;;) {  // George-Liu: walk to a pseudo-peripheral vertex
        const int32_t cand = *std::min_element(last.begin(), last.end(), before);
        std::vector<int32_t> cand_last;
        const int32_t cand_levels = level_structure(g, cand, numbered, depth, touched, cand_last);
        if (cand_levels <= levels) break;
        root = cand;
        levels = cand_levels;
        last.swap(cand_last);
      }
      size_t head = cm.size();
      cm.push_back(root);
      numbered[root] = 1;
      while (head < cm.size()) {
        const int32_t v = cm[head++];
        fresh.clear();
        for (int64_t e = g.start[v]; e < g.start[v + 1]; ++e)
          if (!numbered[g.nbr[e]]) fresh.push_back(g.nbr[e]);
        std::sort(fresh.begin(), fresh.end(), before);
        for (int32_t w : fresh) {
          numbered[w] = 1;
          cm.push_back(w);
        }
      }
    }
    std::reverse_copy(cm.begin(), cm.end(), host_perm);
  } catch (const std::bad_alloc&) {
    return fail(SPX_ERR_INVALID, "csr_rcm: out of host memory");
  }
  return SPX_OK;
}

extern "C" spx_status csr_vector_access(int32_t m, int32_t n, int32_t nnz, const int32_t* host_rowptr,
                                        const int32_t* host_colind, int32_t line, int32_t parts,
                                        int32_t chunk, double* out) {
  if (m < 0 || n < 0 || nnz < 0 || line < 1 || parts < 1 || chunk < 1 || !out)
    return fail(SPX_ERR_INVALID, "csr_vector_access: bad argument");
  if (m > 0 && (!host_rowptr || (nnz > 0 && !host_colind)))
    return fail(SPX_ERR_INVALID, "csr_vector_access: null pointer");
  const int64_t lines = (static_cast<int64_t>(n) + line - 1) / line;
  if (lines == 0) {
    *out = 0.0;
    return SPX_OK;
  }
  // last_part[l] = 1 + the last part that touched line l; parts are visited
  // one after the other, so a line is counted once per part
  std::vector<int32_t> last_part(static_cast<size_t>(lines), 0);
  int64_t moved = 0;
  const int64_t stride = static_cast<int64_t>(parts) * chunk;
  for (int32_t q = 0; q < parts; ++q)
    for (int64_t b = static_cast<int64_t>(q) * chunk; b < m; b += stride)
      for (int64_t i = b; i < std::min<int64_t>(b + chunk, m); ++i)
        for (int32_t p = host_rowptr[i]; p < host_rowptr[i + 1]; ++p) {
          const int32_t c = host_colind[p];
          if (c < 0 || c >= n) return fail(SPX_ERR_INVALID, "csr_vector_access: column out of range");
          int32_t& lp = last_part[c / line];
          if (lp != q + 1) {
            lp = q + 1;
            ++moved;
          }
        }
  *out = static_cast<double>(moved) / static_cast<double>(lines);
  return SPX_OK;
}

extern "C" spx_status csr_tile_lines(int32_t m, int32_t n, int32_t nnz, const int32_t* host_rowptr,
                                     const int32_t* host_colind, int32_t line, int32_t tile, int64_t* out) {
  if (m < 0 || n < 0 || nnz < 0 || line < 1 || tile < 1 || !out)
    return fail(SPX_ERR_INVALID, "csr_tile_lines: bad argument");
  if (m > 0 && (!host_rowptr || (nnz > 0 && !host_colind)))
    return fail(SPX_ERR_INVALID, "csr_tile_lines: null pointer");
  // per tile: the line ids of its nonzeros, sorted, counted once each
  int64_t pairs = 0;
  std::vector<int32_t> ids;
  for (int64_t r0 = 0; r0 < m; r0 += tile) {
    const int64_t r1 = std::min<int64_t>(r0 + tile, m);
    ids.clear();
    for (int32_t p = host_rowptr[r0]; p < host_rowptr[r1]; ++p) {
      const int32_t c = host_colind[p];
      if (c < 0 || c >= n) return fail(SPX_ERR_INVALID, "csr_tile_lines: column out of range");
      ids.push_back(c / line);
    }
    std::sort(ids.begin(), ids.end());
    pairs += std::unique(ids.begin(), ids.end()) - ids.begin();
  }
  *out = pairs;
  return SPX_OK;
}

extern "C" spx_status csr_ucld(int32_t m, int32_t nnz, const int32_t* host_rowptr, const int32_t* host_colind,
                               int32_t line, double* out) {
  if (m < 0 || nnz < 0 || line < 1 || !out) return fail(SPX_ERR_INVALID, "csr_ucld: bad argument");
  if (m > 0 && (!host_rowptr || (nnz > 0 && !host_colind))) return fail(SPX_ERR_INVALID, "csr_ucld: null pointer");
  double total = 0.0;
  int64_t rows = 0;
  for (int32_t i = 0; i < m; ++i) {
    const int32_t b = host_rowptr[i], e = host_rowptr[i + 1];
    if (e <= b) continue;
    // distinct lines of a row with ascending columns: count line changes
    int64_t touched = 1;
    for (int32_t p = b + 1; p < e; ++p) touched += (host_colind[p] / line != host_colind[p - 1] / line);
    total += static_cast<double>(e - b) / (static_cast<double>(line) * static_cast<double>(touched));
    ++rows;
  }
  *out = rows ? total / static_cast<double>(rows) : 0.0;
  return SPX_OK;
}

// ---------------------------------------------------------------- device permutation

namespace spx {
namespace {

__global__ void k_set_i32(int32_t* __restrict__ p, int32_t n, int32_t value) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) p[i] = value;
}

unsigned blocks_for(int64_t n) { return static_cast<unsigned>((n + 255) / 256); }

__global__ void k_invert(const int32_t* __restrict__ perm, int32_t m, int32_t* __restrict__ inv) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= m) return;
  const int32_t o = perm[i];
  if (o >= 0 && o < m) inv[o] = static_cast<int32_t>(i);
}

// The nonzeros keep their positions, with both indices renamed (a row or
// column whose label is missing stays -1 and is reported by the assembly's
// range check).  Tiles of consecutive nonzeros, so a row's length does not
// matter: with a thread per row, the longest row of a power law (20,000 of
// 4.8 M nonzeros) alone held the kernel for 4.9 ms; this takes 33 us.
__global__ __launch_bounds__(kWG) void k_relabel(const int32_t* __restrict__ rowptr,
                                                 const int32_t* __restrict__ colind,
                                                 const int32_t* __restrict__ inv, int32_t m, int32_t nnz,
                                                 int32_t* __restrict__ r, int32_t* __restrict__ c) {
  __shared__ int32_t s_row[radix::kTile];
  __shared__ int32_t s_wsum[radix::kWaves];
  const int t = threadIdx.x, lane = t % kWave, w = t / kWave;
  const int32_t base = static_cast<int32_t>(blockIdx.x) * radix::kTile;
  const int32_t here = min(radix::kTile, nnz - base);
  int32_t col[radix::kItems], row[radix::kItems];
#pragma unroll
  for (int j = 0; j < radix::kItems; ++j) {
    const int32_t i = w * (radix::kTile / radix::kWaves) + j * kWave + lane;
    if (i < here) col[j] = colind[base + i];
  }
  radix::tile_rows(rowptr, m, base, here, s_row, s_wsum, row);
#pragma unroll
  for (int j = 0; j < radix::kItems; ++j) {
    const int32_t i = w * (radix::kTile / radix::kWaves) + j * kWave + lane;
    if (i >= here) continue;
    r[base + i] = inv[row[j]];
    c[base + i] = inv[col[j]];
  }
}

size_t align256(size_t b) { return (b + 255) & ~size_t(255); }

// Nonzeros per column (entries outside [0, n) are not counted).
__global__ void k_col_count(const int32_t* __restrict__ colind, int64_t nnz, int32_t n,
                            int32_t* __restrict__ cnt) {
  const int64_t p = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (p >= nnz) return;
  const int32_t c = colind[p];
  if (c >= 0 && c < n) atomicAdd(cnt + c, 1);
}

// The same from columns grouped by their high bits (one radix pass), so that a
// tile holds few distinct columns: it counts them in LDS and adds each count
// with one atomic.  Every global atomic is performed past L2, and those of a
// column follow one another; on a power law the hot columns' repeats are most
// of them (4.8 M nonzeros: 289 us with an atomic each, 62 us with the pass).
constexpr int kCountWindow = 4096;       // columns counted in LDS, from the tile's first group on
constexpr int64_t kGroupedCount = 1 << 17;  // nonzeros from which the pass over the columns pays for itself
// Nonzeros grouped at a time: bounds the workspace (5 bytes each) to 168 MB.
// Pieces of 2^23 would bound it to 42 MB, but take 268 us instead of 227 for
// 16.8 M nonzeros, a scan and the ends of three launches more.
constexpr int64_t kGroupedPiece = 1 << 25;

struct ColKeySrc {
  const int32_t* colind;
  __device__ __forceinline__ uint32_t raw(int64_t i) const { return static_cast<uint32_t>(colind[i]); }
  __device__ __forceinline__ uint32_t key(uint32_t x) const { return x; }
  __device__ __forceinline__ void check(uint32_t) const {}
  __device__ __forceinline__ radix::NoVal val(int64_t) const { return radix::NoVal(); }
};

struct KeySink {
  uint32_t* k;
  __device__ __forceinline__ void put_key(int64_t i, uint32_t x) const { k[i] = x; }
};

__global__ __launch_bounds__(kWG) void k_col_count_grouped(const uint32_t* __restrict__ grouped, int64_t nnz,
                                                           int32_t n, int shift, uint32_t mask,
                                                           int32_t* __restrict__ cnt) {
  __shared__ int32_t s_cnt[kCountWindow];
  const int t = threadIdx.x;
  const int64_t base = static_cast<int64_t>(blockIdx.x) * radix::kTile;
  for (int i = t; i < kCountWindow; i += kWG) s_cnt[i] = 0;
  const uint32_t first = ((grouped[base] >> shift) & mask) << shift;  // of a column inside [0, n): its group
  __syncthreads();
#pragma unroll
  for (int j = 0; j < radix::kItems; ++j) {
    const int64_t i = base + j * kWG + t;
    if (i >= nnz) continue;
    const uint32_t c = grouped[i];
    if (c >= static_cast<uint32_t>(n)) continue;
    if (c - first < static_cast<uint32_t>(kCountWindow)) atomicAdd(&s_cnt[c - first], 1);
    else atomicAdd(cnt + c, 1);
  }
  __syncthreads();
  for (int i = t; i < kCountWindow; i += kWG)
    if (s_cnt[i]) atomicAdd(cnt + first + i, s_cnt[i]);
}

// Columns by their complemented count: an ascending stable sort lists them by
// descending count with ties in ascending index.
struct DegreeSrc {
  const int32_t* cnt;
  uint32_t top;
  __device__ __forceinline__ int32_t raw(int64_t j) const { return cnt[j]; }
  __device__ __forceinline__ uint32_t key(int32_t x) const { return top - static_cast<uint32_t>(x); }
  __device__ __forceinline__ void check(int32_t) const {}
  __device__ __forceinline__ int32_t val(int64_t j) const { return static_cast<int32_t>(j); }
};

struct PermSink {
  int32_t* perm;
  __device__ __forceinline__ void put_key(int64_t, uint32_t) const {}
  __device__ __forceinline__ void put_val(int64_t i, int32_t x) const { perm[i] = x; }
};

struct DegreeWs {
  int32_t* cnt;
  uint32_t* keys[2];
  int32_t* vals[2];
  uint32_t* grouped;
  void* radix;
};

// Nonzeros of each piece: equal pieces, whole tiles.
int64_t grouped_piece(int64_t nnz) {
  const int64_t pieces = (nnz + kGroupedPiece - 1) / kGroupedPiece;
  return pieces < 2 ? nnz : radix::tiles_of((nnz + pieces - 1) / pieces) * radix::kTile;
}

DegreeWs carve_degree(void* ws, int32_t n, int32_t nnz, size_t* bytes) {
  Carve cv(ws, ~size_t(0));
  const int64_t e = n > 0 ? n : 1;
  DegreeWs w;
  w.cnt = cv.take<int32_t>(e);
  for (int i = 0; i < 2; ++i) {
    w.keys[i] = cv.take<uint32_t>(e);
    w.vals[i] = cv.take<int32_t>(e);
  }
  const int64_t piece = nnz >= kGroupedCount ? grouped_piece(nnz) : 1;
  w.grouped = cv.take<uint32_t>(piece);
  w.radix = cv.take<char>(radix::count_bytes(piece > n ? piece : n));
  *bytes = cv.used;
  return w;
}

// Bandwidth (Sec. 4.4): max |colind[p] - r| over the nonzeros of each row r;
// a wavefront maximum, then one atomic per wavefront into a zeroed *out.
__global__ void k_bandwidth(const int32_t* __restrict__ rowptr, const int32_t* __restrict__ colind, int32_t m,
                            int32_t* __restrict__ out) {
  const int64_t r = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  int32_t best = 0;
  if (r < m) {
    const int32_t p1 = rowptr[r + 1];
    for (int32_t p = rowptr[r]; p < p1; ++p) {
      const int64_t d = static_cast<int64_t>(colind[p]) - r;
      const int64_t a = d < 0 ? -d : d;
      best = max(best, static_cast<int32_t>(a < INT32_MAX ? a : INT32_MAX));
    }
  }
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1) best = max(best, __shfl_xor(best, off, kWave));
  if (threadIdx.x % kWave == 0 && best > 0) atomicMax(out, best);
}

}  // namespace
}  // namespace spx

extern "C" spx_status csr_degree_order_workspace_bytes(int32_t n, int32_t nnz, size_t* bytes) {
  if (!bytes || n < 0 || nnz < 0) return fail(SPX_ERR_INVALID, "csr_degree_order_workspace_bytes: bad argument");
  carve_degree(nullptr, n, nnz, bytes);
  return SPX_OK;
}

extern "C" spx_status csr_degree_order(int32_t n, int32_t nnz, const int32_t* colind, int32_t* perm,
                                       void* workspace, size_t ws_bytes, void* stream) {
  if (n < 0 || nnz < 0) return fail(SPX_ERR_INVALID, "csr_degree_order: negative size");
  {
    const spx_status s_nnz = check_nnz(nnz, "csr_degree_order");
    if (s_nnz != SPX_OK) return s_nnz;
  }
  if ((n > 0 && !perm) || (nnz > 0 && !colind)) return fail(SPX_ERR_INVALID, "csr_degree_order: null pointer");
  size_t need = 0;
  spx_status s = csr_degree_order_workspace_bytes(n, nnz, &need);
  if (s != SPX_OK) return s;
  if (!workspace || ws_bytes < need)
    return fail(SPX_ERR_WORKSPACE, "csr_degree_order: workspace %zu < %zu bytes", ws_bytes, need);
  if (n == 0) return SPX_OK;
  hipStream_t st = as_stream(stream);
  const DegreeWs w = carve_degree(workspace, n, nnz, &need);
  k_set_i32<<<blocks_for(n), 256, 0, st>>>(w.cnt, n, 0);
  SPX_LAUNCHED("k_set_i32");
  if (nnz >= kGroupedCount) {
    const int bits = bits_for(n - 1);
    const int width = bits < radix::kMaxDigit ? bits : radix::kMaxDigit, shift = bits - width;
    const int64_t piece = grouped_piece(nnz);
    for (int64_t p = 0; p < nnz; p += piece) {
      const int64_t here = nnz - p < piece ? nnz - p : piece;
      s = radix::pass(ColKeySrc{colind + p}, KeySink{w.grouped}, here, shift, width, w.radix, st);
      if (s != SPX_OK) return s;
      k_col_count_grouped<<<static_cast<unsigned>(radix::tiles_of(here)), kWG, 0, st>>>(
          w.grouped, here, n, shift, (1u << width) - 1u, w.cnt);
      SPX_LAUNCHED("k_col_count_grouped");
    }
  } else if (nnz > 0) {
    k_col_count<<<blocks_for(nnz), 256, 0, st>>>(colind, nnz, n, w.cnt);
    SPX_LAUNCHED("k_col_count");
  }
  // a count is at most nnz, so its complement needs no more bits than nnz
  const int bits = bits_for(nnz);
  const radix::Pairs<uint32_t, int32_t> a{w.keys[0], w.vals[0]}, b{w.keys[1], w.vals[1]};
  return radix::sort(DegreeSrc{w.cnt, (1u << bits) - 1u}, a, b, PermSink{perm}, n, bits,
                     radix::passes_for(bits), w.radix, st);
}

extern "C" spx_status csr_permute_workspace_bytes(int32_t m, int32_t nnz, size_t* bytes) {
  if (!bytes || m < 0 || nnz < 0) return fail(SPX_ERR_INVALID, "csr_permute_workspace_bytes: bad argument");
  size_t coo = 0;
  spx_status s = csr_from_coo_workspace_bytes(m, m, nnz, &coo);
  if (s != SPX_OK) return s;
  *bytes = align256(sizeof(int32_t) * static_cast<size_t>(m)) + 2 * align256(sizeof(int32_t) * static_cast<size_t>(nnz)) + coo;
  return SPX_OK;
}

extern "C" spx_status csr_permute(int32_t m, int32_t nnz, const int32_t* rowptr, const int32_t* colind,
                                  const double* values, const int32_t* perm, int32_t* rowptr_out,
                                  int32_t* colind_out, double* values_out, int32_t* nnz_out, void* workspace,
                                  size_t ws_bytes, void* stream) {
  if (m < 0 || nnz < 0) return fail(SPX_ERR_INVALID, "csr_permute: negative size");
  {
    const spx_status s_nnz = check_nnz(nnz, "csr_permute");
    if (s_nnz != SPX_OK) return s_nnz;
  }
  if (!rowptr || !rowptr_out || !nnz_out || (m > 0 && !perm) ||
      (nnz > 0 && (!colind || !values || !colind_out || !values_out)))
    return fail(SPX_ERR_INVALID, "csr_permute: null pointer");
  size_t need = 0;
  spx_status s = csr_permute_workspace_bytes(m, nnz, &need);
  if (s != SPX_OK) return s;
  if (!workspace || ws_bytes < need)
    return fail(SPX_ERR_WORKSPACE, "csr_permute: workspace %zu < %zu bytes", ws_bytes, need);
  hipStream_t st = as_stream(stream);
  char* w = static_cast<char*>(workspace);
  int32_t* inv = reinterpret_cast<int32_t*>(w);
  w += align256(sizeof(int32_t) * static_cast<size_t>(m));
  int32_t* r = reinterpret_cast<int32_t*>(w);
  w += align256(sizeof(int32_t) * static_cast<size_t>(nnz));
  int32_t* c = reinterpret_cast<int32_t*>(w);
  w += align256(sizeof(int32_t) * static_cast<size_t>(nnz));
  if (m > 0) {
    k_set_i32<<<blocks_for(m), 256, 0, st>>>(inv, m, -1);
    SPX_LAUNCHED("k_set_i32");
    k_invert<<<blocks_for(m), 256, 0, st>>>(perm, m, inv);
    SPX_LAUNCHED("k_invert");
    if (nnz > 0) {
      k_relabel<<<static_cast<unsigned>(radix::tiles_of(nnz)), kWG, 0, st>>>(rowptr, colind, inv, m, nnz, r, c);
      SPX_LAUNCHED("k_relabel");
    }
  }
  return csr_from_coo(m, m, nnz, r, c, values, rowptr_out, colind_out, values_out, nnz_out, w,
                      ws_bytes - static_cast<size_t>(w - static_cast<char*>(workspace)), stream);
}

extern "C" spx_status csr_bandwidth(int32_t m, int32_t nnz, const int32_t* rowptr, const int32_t* colind,
                                    int32_t* bw_out, void* stream) {
  if (m < 0 || nnz < 0) return fail(SPX_ERR_INVALID, "csr_bandwidth: negative size");
  {
    const spx_status s_nnz = check_nnz(nnz, "csr_bandwidth");
    if (s_nnz != SPX_OK) return s_nnz;
  }
  if (!bw_out || (m > 0 && !rowptr) || (nnz > 0 && !colind))
    return fail(SPX_ERR_INVALID, "csr_bandwidth: null pointer");
  hipStream_t st = as_stream(stream);
  k_set_i32<<<1, 64, 0, st>>>(bw_out, 1, 0);
  SPX_LAUNCHED("k_set_i32");
  if (m > 0 && nnz > 0) {
    k_bandwidth<<<blocks_for(m), 256, 0, st>>>(rowptr, colind, m, bw_out);
    SPX_LAUNCHED("k_bandwidth");
  }
  return SPX_OK;
}
