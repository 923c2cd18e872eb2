// Exclusive prefix sums (int64 totals) for counts, offsets and index maps,
// of one array or of several of one length in the same launches.  Short ones
// in one launch, a block per array; longer ones in three passes: per-block
// totals, one block scanning the totals, per-block scan plus offset.
// Deterministic (integer) and independent of timing.
#include "internal.hpp"

namespace ibvt {

namespace {

constexpr int kScanThreads = 256;
constexpr int kScanItems = 16;
constexpr int kScanTile = kScanThreads * kScanItems;
constexpr int kSumsThreads = 1024;  // the one block that scans the block totals
// Up to this length one block scans an array: a launch costs the host 4 to 5
// us, and a chain of three short kernels about 20 us on the device, where
// the one block takes 5 to 6.  (Longer arrays need more blocks: the three
// passes take 15 us for 144k items, and one block reads at some 100 GB/s.)
constexpr int kScanShort = kSumsThreads * kScanItems;

// Array y of a launch over several.
struct ScanOuts {
  int64_t* p[3];
};

template <typename Tin>
__global__ __launch_bounds__(kScanThreads) void k_block_sums(const Tin* __restrict__ ins, int64_t n,
                                                            int64_t stride,
                                                            int64_t* __restrict__ bsums) {
  const Tin* in = ins + blockIdx.y * stride;
  int64_t* bsum = bsums + int64_t(blockIdx.y) * gridDim.x;
  __shared__ int64_t red[kScanThreads / kWave];
  const int64_t base = int64_t(blockIdx.x) * kScanTile;
  int64_t s = 0;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    const int64_t i = base + int64_t(k) * kScanThreads + threadIdx.x;
    if (i < n) s += int64_t(in[i]);
  }
  s = wave_sum(s);
  if (lane_id() == 0) red[threadIdx.x / kWave] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    int64_t t = 0;
    for (int w = 0; w < kScanThreads / kWave; ++w) t += red[w];
    bsum[blockIdx.x] = t;
  }
}

// Inclusive scan of one value per thread across the block; returns the
// exclusive prefix and writes the block total to *total.  sh holds one
// entry per wave.
__device__ int64_t block_exclusive(int64_t v, int64_t* sh, int64_t* total) {
  // wave-level inclusive scan
  int64_t x = v;
  const int l = lane_id();
  for (int o = 1; o < kWave; o <<= 1) {
    const int64_t y = __shfl_up(x, o, kWave);
    if (l >= o) x += y;
  }
  const int w = threadIdx.x / kWave;
  if (l == kWave - 1) sh[w] = x;
  __syncthreads();
  int64_t pre = 0, tot = 0;
  for (int k = 0; k < int(blockDim.x) / kWave; ++k) {
    if (k < w) pre += sh[k];
    tot += sh[k];
  }
  __syncthreads();
  *total = tot;
  return pre + x - v;
}

// Exclusive scan of the nb block totals of every array in place, one block
// for each: a thread takes a run of consecutive totals.
__global__ __launch_bounds__(kSumsThreads) void k_scan_sums(int64_t* __restrict__ bsums, int64_t nb,
                                                           ScanOuts outs, int64_t n) {
  __shared__ int64_t sh[kSumsThreads / kWave];
  int64_t* bsum = bsums + int64_t(blockIdx.x) * nb;
  int64_t* out = blockIdx.x == 0 ? outs.p[0] : (blockIdx.x == 1 ? outs.p[1] : outs.p[2]);
  const int64_t per = ceil_div(nb, kSumsThreads);
  const int64_t b0 = int64_t(threadIdx.x) * per;
  const int64_t b1 = min<int64_t>(nb, b0 + per);
  int64_t s = 0;
  for (int64_t b = b0; b < b1; ++b) s += bsum[b];
  int64_t tot;
  int64_t pre = block_exclusive(s, sh, &tot);
  for (int64_t b = b0; b < b1; ++b) {
    const int64_t v = bsum[b];
    bsum[b] = pre;
    pre += v;
  }
  if (threadIdx.x == 0) out[n] = tot;
}

// The whole scan of short arrays, one block for each: a thread takes a run
// of consecutive items, its reads in flight together.
template <typename Tin>
__global__ __launch_bounds__(kSumsThreads) void k_scan_short(const Tin* __restrict__ ins, int n,
                                                            int64_t stride, ScanOuts outs) {
  __shared__ int64_t sh[kSumsThreads / kWave];
  const Tin* in = ins + blockIdx.x * stride;
  int64_t* out = blockIdx.x == 0 ? outs.p[0] : (blockIdx.x == 1 ? outs.p[1] : outs.p[2]);
  const int per = int(ceil_div(n, kSumsThreads));
  const int b0 = int(threadIdx.x) * per;
  int64_t v[kScanItems];
  int64_t s = 0;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) v[k] = k < per && b0 + k < n ? int64_t(in[b0 + k]) : 0;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) s += v[k];
  int64_t tot;
  int64_t pre = block_exclusive(s, sh, &tot);
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    if (k < per && b0 + k < n) out[b0 + k] = pre;
    pre += v[k];
  }
  if (threadIdx.x == 0) out[n] = tot;
}

// Per tile: the items are read with consecutive threads on consecutive
// items into LDS, each thread scans its run of kScanItems there (rows
// padded by one entry against bank conflicts), and the results leave the
// same coalesced way.
__device__ __forceinline__ int scan_slot(int i) { return (i / kScanItems) * (kScanItems + 1) + i % kScanItems; }

template <typename Tin>
__global__ __launch_bounds__(kScanThreads) void k_scan_tiles(const Tin* __restrict__ ins, int64_t n,
                                                            int64_t stride,
                                                            const int64_t* __restrict__ bsums,
                                                            ScanOuts outs) {
  const Tin* in = ins + blockIdx.y * stride;
  const int64_t* bsum = bsums + int64_t(blockIdx.y) * gridDim.x;
  int64_t* out = blockIdx.y == 0 ? outs.p[0] : (blockIdx.y == 1 ? outs.p[1] : outs.p[2]);
  __shared__ int64_t buf[kScanThreads * (kScanItems + 1)];
  __shared__ int64_t sh[kScanThreads / kWave];
  const int64_t base = int64_t(blockIdx.x) * kScanTile;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    const int i = k * kScanThreads + int(threadIdx.x);
    buf[scan_slot(i)] = (base + i < n) ? int64_t(in[base + i]) : 0;
  }
  __syncthreads();
  int64_t* row = buf + threadIdx.x * (kScanItems + 1);
  int64_t s = 0;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) s += row[k];
  int64_t tot;
  int64_t pre = block_exclusive(s, sh, &tot) + bsum[blockIdx.x];
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    const int64_t v = row[k];
    row[k] = pre;
    pre += v;
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    const int i = k * kScanThreads + int(threadIdx.x);
    if (base + i < n) out[base + i] = buf[scan_slot(i)];
  }
}

template <typename Tin>
int scan_impl(ibvt_coupling* c, const Tin* in, int64_t stride, const ScanOuts& outs, int m,
              int64_t n, hipStream_t s) {
  if (n <= kScanShort) {
    k_scan_short<Tin><<<unsigned(m), kSumsThreads, 0, s>>>(in, int(n), stride, outs);
    return hip_check(hipGetLastError(), "scan launch");
  }
  const int64_t nb = ceil_div(n, kScanTile);
  int st = ensure(c, c->scan_tmp, size_t(m * nb) * sizeof(int64_t));
  if (st) return st;
  int64_t* bsum = c->scan_tmp.as<int64_t>();
  const dim3 grid{unsigned(nb), unsigned(m)};
  k_block_sums<Tin><<<grid, kScanThreads, 0, s>>>(in, n, stride, bsum);
  k_scan_sums<<<unsigned(m), kSumsThreads, 0, s>>>(bsum, nb, outs, n);
  k_scan_tiles<Tin><<<grid, kScanThreads, 0, s>>>(in, n, stride, bsum, outs);
  return hip_check(hipGetLastError(), "scan launch");
}

}  // namespace

int scan_i64(ibvt_coupling* c, const int64_t* in, int64_t* out, int64_t n, hipStream_t s) {
  return scan_impl<int64_t>(c, in, 0, ScanOuts{{out, nullptr, nullptr}}, 1, n, s);
}

int scan_i64_rows(ibvt_coupling* c, const int64_t* in, int64_t* const* out, int m, int64_t n,
                  hipStream_t s) {
  ScanOuts o{};
  for (int k = 0; k < m; ++k) o.p[k] = out[k];
  return scan_impl<int64_t>(c, in, n, o, m, n, s);
}

int scan_i32_to_i64(ibvt_coupling* c, const int32_t* in, int64_t* out, int64_t n, hipStream_t s) {
  return scan_impl<int32_t>(c, in, 0, ScanOuts{{out, nullptr, nullptr}}, 1, n, s);
}

}  // namespace ibvt
