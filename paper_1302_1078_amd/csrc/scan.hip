// scan.hip -- device-wide exclusive scan.
//
// Used once per sparsity pattern: to assemble CSR from triplets and to bin
// rows.  Tiles are 4096 items (256 threads x 16).  Integer arithmetic only;
// results are deterministic.
#include "device.hpp"
#include "internal.hpp"
#include "radix.hpp"

namespace spx {

namespace {

constexpr int kItems = 16;

__global__ __launch_bounds__(kWG) void k_scan_reduce(const int32_t* __restrict__ in, int64_t n,
                                                     int32_t* __restrict__ sums) {
  const int64_t base = static_cast<int64_t>(blockIdx.x) * kScanTile;
  int32_t s = 0;
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    int64_t i = base + j * kWG + threadIdx.x;
    if (i < n) s += in[i];
  }
  __shared__ int32_t wsum[radix::kWaves];
  int32_t total;
  (void)radix::block_excl_scan(s, wsum, &total);
  if (threadIdx.x == 0) sums[blockIdx.x] = total;
}

// Scan one tile per block with the tile's offset (offs == null: offset 0).
__global__ __launch_bounds__(kWG) void k_scan_apply(const int32_t* in, int32_t* out, int64_t n,
                                                    const int32_t* __restrict__ offs,
                                                    int32_t* total_out) {
  const int64_t base = static_cast<int64_t>(blockIdx.x) * kScanTile + threadIdx.x * kItems;
  int32_t item[kItems];
  int32_t s = 0;
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    int64_t i = base + j;
    item[j] = (i < n) ? in[i] : 0;
    s += item[j];
  }
  __shared__ int32_t wsum[radix::kWaves];
  int32_t total;
  int32_t run = radix::block_excl_scan(s, wsum, &total) + (offs ? offs[blockIdx.x] : 0);
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    int64_t i = base + j;
    if (i < n) out[i] = run;
    run += item[j];
  }
  if (total_out && threadIdx.x == 0) *total_out = total;
}

inline int64_t ntiles(int64_t n) { return (n + kScanTile - 1) / kScanTile; }

}  // namespace

size_t scan_workspace_bytes(int64_t n) {
  size_t b = 0;
  while (n > kScanTile) {
    n = ntiles(n);
    b += align_up(static_cast<size_t>(n) * sizeof(int32_t));
  }
  return b + 256;
}

spx_status exclusive_scan_i32(const int32_t* in, int32_t* out, int64_t n, int32_t* total,
                              void* ws, hipStream_t st) {
  if (n <= 0) {
    if (total) SPX_HIP(hipMemsetAsync(total, 0, sizeof(int32_t), st));
    return SPX_OK;
  }
  if (n <= kScanTile) {
    k_scan_apply<<<1, kWG, 0, st>>>(in, out, n, nullptr, total);
    SPX_LAUNCHED("k_scan_apply");
    return SPX_OK;
  }
  const int64_t nb = ntiles(n);
  int32_t* sums = static_cast<int32_t*>(ws);
  void* rest = static_cast<char*>(ws) + align_up(static_cast<size_t>(nb) * sizeof(int32_t));
  k_scan_reduce<<<static_cast<unsigned>(nb), kWG, 0, st>>>(in, n, sums);
  SPX_LAUNCHED("k_scan_reduce");
  spx_status s = exclusive_scan_i32(sums, sums, nb, total, rest, st);
  if (s != SPX_OK) return s;
  k_scan_apply<<<static_cast<unsigned>(nb), kWG, 0, st>>>(in, out, n, sums, nullptr);
  SPX_LAUNCHED("k_scan_apply");
  return SPX_OK;
}

}  // namespace spx
