// B^dT over the touched fluid nodes (the force transfer's operator).
//
// Rows of B^dT are the fluid nodes that occur as columns of B^d, in
// ascending node order, each listing its vertices in ascending order.  Large
// operators go through buckets of kBucketNodes consecutive lattice nodes:
//   k_bucket_count    blocks of kBucketRows rows of B^d take their nonzeros
//                     in rounds of kRound; within a wave the nonzeros of one
//                     bucket come in runs (a row's columns ascend), and each
//                     run's head adds its count into an LDS hash table, so
//                     one global atomic per (round, bucket) sums them; every
//                     nonzero marks its node (a byte per lattice node).
//   k_bucket_tiles,   per tile of buckets and then before each bucket: its
//   _scan, _list      offsets in B^dT (from the counts), row offsets (from the
//                     marked nodes) and the list of nonempty buckets.
//   k_bucket_scatter  the same rounds reserve a range per (round, bucket);
//                     run heads take their runs' places in it and every
//                     nonzero writes its (value, vertex, node) record.
//   k_bucket_sort     nonempty buckets, a block each: a counting sort of its
//                     records by node in LDS, then each record's place in its
//                     node's row is the number of that row's vertices below
//                     its own (a row's vertices are distinct); the block
//                     writes the bucket's columns, values, row pointers and
//                     row map.
// The components go through these together while they are not too large.
// Small operators take a counting sort over the whole lattice instead,
// together as well:
//   k_tcount          nonzeros per lattice node.
//   k_tsums, k_tscan  per tile of nodes: its touched nodes and its nonzeros,
//                     and their prefix sums.
//   k_ttiles          row map, row pointers and each node's end in B^dT.
//   k_tscatter        every nonzero takes a slot of its row.
//   k_trow_order      each row of B^dT put in vertex order by ranking.
// Atomics only reserve space; every position follows from the (node, vertex)
// order, so the result is deterministic either way.
#include <algorithm>
#include <climits>
#include <cstdlib>
#include <type_traits>

#include "internal.hpp"

namespace ibvt {

namespace {

// A nonzero carried through the counting sort: its value and its row.
template <typename T>
using ValRow = std::conditional_t<std::is_same<T, float>::value, SortVal32, SortVal64>;

constexpr int kKeyLanes = 16;  // lanes per row of B^d in the counting sort's scatter

// Counting sort for small operators, where the bucket path's fixed launches
// dominate (use_buckets): one component of a launch.  The components share
// every launch and the counts stay on the device: bound by launches and the
// reading of the lattice's counters, 32 us for a 144-tet beam on 32^3 cells,
// where component by component with marks, two scans and a read-back for each
// it was 201.
template <typename T>
struct TOne {
  const int64_t* rowptr;  // B^d
  const int32_t* col;
  const T* val;
  int64_t nnz;
  int32_t* node;          // per lattice node (whole tiles): count, then end in B^dT
  uint64_t* sum;          // per tile of nodes: touched nodes << 32 | nonzeros, then before it
  int64_t tiles;
  int64_t tile0;          // its first tile among the launch's
  int64_t* touched;
  int64_t* trowptr;       // B^dT
  int32_t* rowmap;
  int32_t* tcol;
  T* tval;
  ValRow<T>* vr;
};
template <typename T>
struct TBatch {
  TOne<T> c[3];
  int n;
};

constexpr unsigned kTOrderBlocks = 4096;  // four rows each, then the next
constexpr int kTThreads = 256;
constexpr int kTItems = 16;
constexpr int kTTile = kTThreads * kTItems;

// (grid.y: the component)
template <typename T>
__global__ __launch_bounds__(256) void k_tcount(TBatch<T> b) {
  const TOne<T>& c = blockIdx.y == 0 ? b.c[0] : (blockIdx.y == 1 ? b.c[1] : b.c[2]);
  const int64_t k = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (k < c.nnz) atomicAdd(&c.node[c.col[k]], 1);
}

template <typename T>
__device__ __forceinline__ const TOne<T>& tile_component(const TBatch<T>& b) {
  const int64_t t = blockIdx.x;
  return b.n > 2 && t >= b.c[2].tile0 ? b.c[2] : (b.n > 1 && t >= b.c[1].tile0 ? b.c[1] : b.c[0]);
}

// A thread's kTItems consecutive nodes of tile t.
__device__ __forceinline__ void tile_nodes(const int32_t* node, int64_t t, int32_t (&v)[kTItems]) {
  load_row<kTItems>(node + t * kTTile + int64_t(threadIdx.x) * kTItems, v);
}
__device__ __forceinline__ uint64_t nodes_sum(const int32_t (&v)[kTItems]) {
  uint64_t s = 0;
#pragma unroll
  for (int k = 0; k < kTItems; ++k) s += v[k] > 0 ? (uint64_t(1) << 32) + uint32_t(v[k]) : 0;
  return s;
}

template <typename T>
__global__ __launch_bounds__(kTThreads) void k_tsums(TBatch<T> b) {
  __shared__ uint64_t red[kTThreads / kWave];
  const TOne<T>& c = tile_component(b);
  const int64_t t = int64_t(blockIdx.x) - c.tile0;
  int32_t v[kTItems];
  tile_nodes(c.node, t, v);
  const int64_t s = wave_sum(int64_t(nodes_sum(v)));
  if (lane_id() == 0) red[threadIdx.x / kWave] = uint64_t(s);
  __syncthreads();
  if (threadIdx.x == 0) {
    uint64_t x = 0;
    for (int w = 0; w < kTThreads / kWave; ++w) x += red[w];
    c.sum[t] = x;
  }
}

// Exclusive prefix of one value per thread across the block, and the total.
template <int THREADS>
__device__ __forceinline__ uint64_t block_prefix(uint64_t v, uint64_t (&sh)[THREADS / kWave],
                                                 uint64_t& total) {
  uint64_t x = v;
  const int l = lane_id(), w = threadIdx.x / kWave;
  for (int o = 1; o < kWave; o <<= 1) {
    const uint64_t y = __shfl_up((unsigned long long)x, o, kWave);
    if (l >= o) x += y;
  }
  if (l == kWave - 1) sh[w] = x;
  __syncthreads();
  uint64_t pre = 0;
  total = 0;
  for (int k = 0; k < THREADS / kWave; ++k) {
    if (k < w) pre += sh[k];
    total += sh[k];
  }
  __syncthreads();
  return pre + x - v;
}

// One block per component scans its tiles' sums in place (fewer than 2^31
// nonzeros and lattice nodes: the halves of a sum do not overflow).
template <typename T>
__global__ __launch_bounds__(1024) void k_tscan(TBatch<T> b) {
  __shared__ uint64_t sh[1024 / kWave];
  const TOne<T>& c = blockIdx.x == 0 ? b.c[0] : (blockIdx.x == 1 ? b.c[1] : b.c[2]);
  const int64_t per = ceil_div(c.tiles, 1024);
  const int64_t b0 = int64_t(threadIdx.x) * per, b1 = min<int64_t>(c.tiles, b0 + per);
  uint64_t s = 0;
  for (int64_t t = b0; t < b1; ++t) s += c.sum[t];
  uint64_t total;
  uint64_t pre = block_prefix<1024>(s, sh, total);
  for (int64_t t = b0; t < b1; ++t) {
    const uint64_t v = c.sum[t];
    c.sum[t] = pre;
    pre += v;
  }
  if (threadIdx.x == 0) *c.touched = int64_t(total >> 32);
}

template <typename T>
__global__ __launch_bounds__(kTThreads) void k_ttiles(TBatch<T> b) {
  __shared__ uint64_t sh[kTThreads / kWave];
  const TOne<T>& c = tile_component(b);
  const int64_t t = int64_t(blockIdx.x) - c.tile0;
  int32_t v[kTItems];
  tile_nodes(c.node, t, v);
  uint64_t total;
  uint64_t at = c.sum[t] + block_prefix<kTThreads>(nodes_sum(v), sh, total);
  const int64_t n0 = t * kTTile + int64_t(threadIdx.x) * kTItems;
  if (t == 0 && threadIdx.x == 0) c.trowptr[*c.touched] = c.nnz;
#pragma unroll
  for (int k = 0; k < kTItems; ++k) {
    if (v[k] > 0) {
      const uint32_t row = uint32_t(at >> 32), q = uint32_t(at);
      c.rowmap[row] = int32_t(n0 + k);
      c.trowptr[row] = int64_t(q);
      c.node[n0 + k] = int32_t(q + uint32_t(v[k]));
      at += (uint64_t(1) << 32) + uint32_t(v[k]);
    }
  }
}

// Every nonzero (i, j) of B^d takes a slot of node j's row of B^dT by
// counting its end down (the slot order depends on timing; k_trow_order puts
// each row in vertex order afterwards).
template <typename T>
__global__ __launch_bounds__(256) void k_tscatter(TBatch<T> b, int64_t n_rows) {
  const TOne<T>& c = blockIdx.y == 0 ? b.c[0] : (blockIdx.y == 1 ? b.c[1] : b.c[2]);
  const int64_t i = (int64_t(blockIdx.x) * blockDim.x + threadIdx.x) / kKeyLanes;
  const int lane = threadIdx.x % kKeyLanes;
  if (i >= n_rows) return;
  const int64_t end = c.rowptr[i + 1];
  for (int64_t k = c.rowptr[i] + lane; k < end; k += kKeyLanes) {
    ValRow<T> x;
    x.v = c.val[k];
    x.r = int32_t(i);
    c.vr[atomicSub(&c.node[c.col[k]], 1) - 1] = x;
  }
}

// One wave per row of B^dT: the row's vertices are distinct, so an entry's
// place in ascending vertex order is the number of the row's entries with a
// smaller vertex.  The row is read in tiles of kWave entries whose vertices
// are broadcast lane by lane.  Positions do not depend on the slot order
// k_tscatter left, so the result is deterministic.  The number of rows is
// on the device: the waves loop over them.
template <typename T>
__global__ __launch_bounds__(256) void k_trow_order(TBatch<T> bt) {
  const TOne<T>& c = blockIdx.y == 0 ? bt.c[0] : (blockIdx.y == 1 ? bt.c[1] : bt.c[2]);
  const int lane = lane_id();
  const int64_t rows = *c.touched, step = int64_t(gridDim.x) * (blockDim.x / kWave);
  for (int64_t r = (int64_t(blockIdx.x) * blockDim.x + threadIdx.x) / kWave; r < rows; r += step) {
    const int64_t b = c.trowptr[r];
    const int L = __builtin_amdgcn_readfirstlane(int(c.trowptr[r + 1] - b));
    for (int c0 = 0; c0 < L; c0 += kWave) {
      const bool mine = c0 + lane < L;
      ValRow<T> x;
      x.v = T(0);
      x.r = INT_MAX;
      if (mine) x = c.vr[b + c0 + lane];
      int rank = 0;
      for (int m0 = 0; m0 < L; m0 += kWave) {
        const int y = (m0 + lane < L) ? c.vr[b + m0 + lane].r : INT_MAX;
        const int nm = L - m0 < kWave ? L - m0 : kWave;
        for (int m = 0; m < nm; ++m) rank += __builtin_amdgcn_readlane(y, m) < x.r ? 1 : 0;
      }
      if (mine) {
        c.tcol[b + rank] = x.r;
        c.tval[b + rank] = x.v;
      }
    }
  }
}

// ---- bucket transpose (large operators) ----

constexpr int kBucketBits = 5;
constexpr int kBucketNodes = 1 << kBucketBits;  // consecutive lattice nodes per bucket
constexpr int kBucketRows = 64;                 // rows of B^d per block (count, scatter)
constexpr int kBucketThreads = 256;
constexpr int kRound = 2048;                    // nonzeros per round (8 per thread)
constexpr int kTableBits = 12;
constexpr int kTable = 1 << kTableBits;         // hash slots per round (>= 2 x kRound)
constexpr int kSortCap = 4096;                  // records a bucket sorts in LDS
static_assert(kRound % kBucketThreads == 0 && 2 * kRound <= kTable, "round and table sizes");

// A nonzero of B^d on its way into B^dT: value, and vertex (its row of B^d)
// with the node within the bucket in one word (vertices below 2^27).
template <typename T>
struct BucketRec {
  T v;
  uint32_t rn;  // vertex << kBucketBits | node
  __device__ __forceinline__ int32_t r() const { return int32_t(rn >> kBucketBits); }
  __device__ __forceinline__ int nl() const { return int(rn & (kBucketNodes - 1)); }
};
constexpr int64_t kBucketMaxVert = int64_t(1) << (32 - kBucketBits);

// A nonempty bucket as the sort takes it: its first record (= its first
// place in B^dT), its first row of B^dT, the bucket and its record count.
struct BucketSpan {
  int64_t a, t;
  int32_t b, n;
};

// Sums over buckets: nonzeros, touched nodes, nonempty buckets.
struct BucketSums {
  int64_t nnz, touched, full;
  __device__ __forceinline__ void add(const BucketSums& o) {
    nnz += o.nnz;
    touched += o.touched;
    full += o.full;
  }
};

// One component of a launch.
template <typename T>
struct BOne {
  const int64_t* rowptr;  // B^d
  const int32_t* col;
  const T* val;
  int64_t nnz;
  int64_t nb;             // buckets
  int32_t* bcount;        // per bucket: nonzeros
  int32_t* bfill;         // places taken
  uint8_t* mark;          // a byte per node (whole buckets)
  int32_t* boff;          // first place
  BucketSpan* list;       // nonempty buckets
  BucketRec<T>* rec;
  BucketSums* sum;        // per tile of buckets, then before it
  int64_t tiles, tile0;   // (tile0: its first among the launch's)
  int64_t* touched;
  int64_t* trowptr;       // B^dT
  int32_t* rowmap;
  int32_t* tcol;
  T* tval;
};
template <typename T>
struct BBatch {
  BOne<T> c[3];
  int n;
};
constexpr int64_t kBatchRecords = int64_t(32) << 20;  // (0.25 GiB in float)
constexpr int kBTile = 4 * kBucketThreads;  // buckets of a tile

// Slot of bucket b in a round's table (open addressing; a round has at most
// kRound distinct buckets, so a free slot always exists).
__device__ __forceinline__ int table_slot(int32_t* key, int32_t b) {
  int h = int((uint32_t(b) * 2654435761u) >> (32 - kTableBits));
  for (;;) {
    const int32_t prev = atomicCAS(&key[h], -1, b);
    if (prev == -1 || prev == b) return h;
    h = (h + 1) & (kTable - 1);
  }
}

// Row block of this workgroup.  Workgroups are dispatched to the 8 XCDs in
// turn; handing each XCD a contiguous run of row blocks keeps the bucket
// ranges one XCD writes away from the others' (whole cache lines per L2).
// The grid has 8 * per blocks.
__device__ __forceinline__ int64_t xcd_row_block(int64_t per) {
  return int64_t(blockIdx.x % 8) * per + int64_t(blockIdx.x / 8);
}

// Runs of one bucket among a wave's consecutive nonzeros (a row's columns
// ascend, so its buckets come in runs): a run starts where the bucket
// differs from the previous lane's, or at lane 0.  The valid lanes are a
// prefix of the wave.  Gives the lane's run start and run end (one past).
struct WaveRun {
  int head, end;
  bool is_head;
};
__device__ __forceinline__ WaveRun wave_run(int32_t bucket, bool valid) {
  const int l = lane_id();
  const int32_t prev = __shfl_up(bucket, 1, kWave);
  WaveRun w;
  w.is_head = valid && (l == 0 || prev != bucket);
  const uint64_t heads = ballot64(w.is_head);
  const uint64_t n_valid = uint64_t(popc64(ballot64(valid)));
  const uint64_t upto = (2ull << l) - 1ull;  // lanes 0..l (all lanes when l = 63)
  const uint64_t below = heads & upto, above = heads & ~upto;
  w.head = below ? 63 - __builtin_clzll(below) : 0;
  w.end = above ? __builtin_ctzll(above) : int(n_valid);
  return w;
}

// Per bucket: nonzero count (only run heads touch the round's table), and
// a byte per node that occurs (plain stores: every writer stores 1).
template <typename T>
__global__ __launch_bounds__(kBucketThreads) void k_bucket_count(BBatch<T> bt, int64_t n_rows,
                                                                 int64_t per) {
  const BOne<T>& c = blockIdx.y == 0 ? bt.c[0] : (blockIdx.y == 1 ? bt.c[1] : bt.c[2]);
  const int64_t* __restrict__ rowptr = c.rowptr;
  const int32_t* __restrict__ col = c.col;
  int32_t* __restrict__ bcount = c.bcount;
  uint8_t* __restrict__ mark = c.mark;
  __shared__ int32_t key[kTable];
  __shared__ int32_t cnt[kTable];
  const int64_t r0 = xcd_row_block(per) * kBucketRows;
  if (r0 >= n_rows) return;
  const int64_t r1 = min<int64_t>(n_rows, r0 + kBucketRows);
  const int64_t k0 = rowptr[r0], k1 = rowptr[r1];
  const int l = lane_id();
  for (int64_t kb = k0; kb < k1; kb += kRound) {
    for (int h = threadIdx.x; h < kTable; h += kBucketThreads) {
      key[h] = -1;
      cnt[h] = 0;
    }
    __syncthreads();
    constexpr int J = kRound / kBucketThreads;
    int32_t nodes[J];
#pragma unroll
    for (int j = 0; j < J; ++j) {  // all loads first
      const int64_t k = kb + j * kBucketThreads + threadIdx.x;
      nodes[j] = k < k1 ? col[k] : 0;
    }
#pragma unroll
    for (int j = 0; j < J; ++j) {
      const bool valid = kb + j * kBucketThreads + threadIdx.x < k1;
      const int32_t node = nodes[j];
      const WaveRun w = wave_run(node >> kBucketBits, valid);
      if (valid) mark[node] = 1;
      if (w.is_head) atomicAdd(&cnt[table_slot(key, node >> kBucketBits)], w.end - l);
    }
    __syncthreads();
    for (int h = threadIdx.x; h < kTable; h += kBucketThreads) {
      const int32_t b = key[h];
      if (b >= 0) atomicAdd(&bcount[b], cnt[h]);
    }
    __syncthreads();
  }
}

template <typename T>
__device__ __forceinline__ const BOne<T>& tile_component(const BBatch<T>& b) {
  const int64_t t = blockIdx.x;
  return b.n > 2 && t >= b.c[2].tile0 ? b.c[2] : (b.n > 1 && t >= b.c[1].tile0 ? b.c[1] : b.c[0]);
}

// Bucket b's sums (its touched nodes are its marked ones).
template <typename T>
__device__ __forceinline__ BucketSums bucket_sums(const BOne<T>& c, int64_t b) {
  BucketSums x{0, 0, 0};
  if (b < c.nb) {
    const uint4* m = reinterpret_cast<const uint4*>(c.mark + b * kBucketNodes);
    const uint4 p = m[0], q = m[1];
    x.nnz = c.bcount[b];
    x.touched = __popc(p.x) + __popc(p.y) + __popc(p.z) + __popc(p.w) + __popc(q.x) + __popc(q.y) +
                __popc(q.z) + __popc(q.w);
    x.full = x.touched != 0;
  }
  return x;
}

// Exclusive prefix of the threads' sums across the block, and the total.
template <int THREADS>
__device__ __forceinline__ BucketSums sums_prefix(const BucketSums& v, BucketSums (&sh)[THREADS / kWave],
                                                  BucketSums& total) {
  BucketSums x = v;
  const int l = lane_id(), w = threadIdx.x / kWave;
  for (int o = 1; o < kWave; o <<= 1) {
    const BucketSums y{__shfl_up(x.nnz, o, kWave), __shfl_up(x.touched, o, kWave),
                       __shfl_up(x.full, o, kWave)};
    if (l >= o) x.add(y);
  }
  if (l == kWave - 1) sh[w] = x;
  __syncthreads();
  BucketSums pre{0, 0, 0};
  total = pre;
  for (int k = 0; k < THREADS / kWave; ++k) {
    if (k < w) pre.add(sh[k]);
    total.add(sh[k]);
  }
  __syncthreads();
  pre.add(BucketSums{x.nnz - v.nnz, x.touched - v.touched, x.full - v.full});
  return pre;
}

template <typename T>
__global__ __launch_bounds__(kBucketThreads) void k_bucket_tiles(BBatch<T> bt) {
  __shared__ BucketSums sh[kBucketThreads / kWave];
  const BOne<T>& c = tile_component(bt);
  const int64_t t = int64_t(blockIdx.x) - c.tile0;
  BucketSums x{0, 0, 0}, total;
#pragma unroll
  for (int k = 0; k < 4; ++k) x.add(bucket_sums(c, t * kBTile + threadIdx.x * 4 + k));
  sums_prefix<kBucketThreads>(x, sh, total);
  if (threadIdx.x == 0) c.sum[t] = total;
}

// One block per component: its tiles' sums scanned in place, the totals.
template <typename T>
__global__ __launch_bounds__(1024) void k_bucket_scan(BBatch<T> bt) {
  __shared__ BucketSums sh[1024 / kWave];
  const BOne<T>& c = blockIdx.x == 0 ? bt.c[0] : (blockIdx.x == 1 ? bt.c[1] : bt.c[2]);
  const int64_t per = ceil_div(c.tiles, 1024);
  const int64_t b0 = int64_t(threadIdx.x) * per, b1 = min<int64_t>(c.tiles, b0 + per);
  BucketSums x{0, 0, 0}, total;
  for (int64_t t = b0; t < b1; ++t) x.add(c.sum[t]);
  BucketSums pre = sums_prefix<1024>(x, sh, total);
  for (int64_t t = b0; t < b1; ++t) {
    const BucketSums v = c.sum[t];
    c.sum[t] = pre;
    pre.add(v);
  }
  if (threadIdx.x == 0) {
    c.touched[0] = total.touched;
    c.touched[1] = total.full;
  }
}

// Every bucket's first place, and the nonempty ones in ascending order.
template <typename T>
__global__ __launch_bounds__(kBucketThreads) void k_bucket_list(BBatch<T> bt) {
  __shared__ BucketSums sh[kBucketThreads / kWave];
  const BOne<T>& c = tile_component(bt);
  const int64_t t = int64_t(blockIdx.x) - c.tile0, b0 = t * kBTile + threadIdx.x * 4;
  BucketSums v[4], x{0, 0, 0}, total;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    v[k] = bucket_sums(c, b0 + k);
    x.add(v[k]);
  }
  if (t == 0 && threadIdx.x == 0) c.trowptr[c.touched[0]] = c.nnz;
  BucketSums at = sums_prefix<kBucketThreads>(x, sh, total);
  at.add(c.sum[t]);
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if (b0 + k < c.nb) c.boff[b0 + k] = int32_t(at.nnz);
    if (v[k].full) c.list[at.full] = BucketSpan{at.nnz, at.touched, int32_t(b0 + k), int32_t(v[k].nnz)};
    at.add(v[k]);
  }
}

// The same rounds as k_bucket_count: each (round, bucket) reserves a range
// of the bucket, run heads take their runs' places in it, and every
// nonzero writes its record there.
template <typename T>
__global__ __launch_bounds__(kBucketThreads) void k_bucket_scatter(BBatch<T> bt, int64_t n_rows,
                                                                   int64_t per) {
  const BOne<T>& c = blockIdx.y == 0 ? bt.c[0] : (blockIdx.y == 1 ? bt.c[1] : bt.c[2]);
  const int64_t* __restrict__ rowptr = c.rowptr;
  const int32_t* __restrict__ col = c.col;
  const T* __restrict__ val = c.val;
  const int32_t* __restrict__ boff = c.boff;
  int32_t* __restrict__ bfill = c.bfill;
  BucketRec<T>* __restrict__ rec = c.rec;
  __shared__ int32_t key[kTable];
  __shared__ int32_t cnt[kTable];  // then the slot's first position in the records
  __shared__ int64_t srp[kBucketRows + 1];
  const int64_t r0 = xcd_row_block(per) * kBucketRows;
  if (r0 >= n_rows) return;
  const int nr = int(min<int64_t>(n_rows - r0, kBucketRows));
  for (int i = threadIdx.x; i <= nr; i += kBucketThreads) srp[i] = rowptr[r0 + i];
  __syncthreads();
  const int64_t k0 = srp[0], k1 = srp[nr];
  const int l = lane_id();
  constexpr int J = kRound / kBucketThreads;
  for (int64_t kb = k0; kb < k1; kb += kRound) {
    for (int h = threadIdx.x; h < kTable; h += kBucketThreads) {
      key[h] = -1;
      cnt[h] = 0;
    }
    __syncthreads();
    int slot[J], rank[J];
    int32_t node[J];
    T v[J];
#pragma unroll
    for (int j = 0; j < J; ++j) {  // all loads first
      const int64_t k = kb + j * kBucketThreads + threadIdx.x;
      node[j] = k < k1 ? col[k] : 0;
      v[j] = k < k1 ? val[k] : T(0);
    }
#pragma unroll
    for (int j = 0; j < J; ++j) {
      const bool valid = kb + j * kBucketThreads + threadIdx.x < k1;
      const WaveRun w = wave_run(node[j] >> kBucketBits, valid);
      int h = 0, r = 0;
      if (w.is_head) {
        h = table_slot(key, node[j] >> kBucketBits);
        r = atomicAdd(&cnt[h], w.end - l);
      }
      slot[j] = valid ? __shfl(h, w.head, kWave) : -1;
      rank[j] = __shfl(r, w.head, kWave) + (l - w.head);
    }
    __syncthreads();
    for (int h = threadIdx.x; h < kTable; h += kBucketThreads) {
      const int32_t b = key[h];
      if (b >= 0) cnt[h] = boff[b] + atomicAdd(&bfill[b], cnt[h]);
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < J; ++j) {
      if (slot[j] < 0) continue;
      const int64_t k = kb + j * kBucketThreads + threadIdx.x;
      // row of nonzero k: srp[lo] <= k < srp[lo + 1] (empty rows skipped)
      int lo = 0, hi = nr;
      while (hi - lo > 1) {
        const int m = (lo + hi) >> 1;
        if (srp[m] <= k) lo = m;
        else hi = m;
      }
      BucketRec<T> x;
      x.v = v[j];
      x.rn = (uint32_t(r0 + lo) << kBucketBits) | uint32_t(node[j] & (kBucketNodes - 1));
      rec[cnt[slot[j]] + rank[j]] = x;
    }
    __syncthreads();
  }
}

// A block takes nonempty buckets in turn (each owns its ranges of B^dT): row
// pointers and row map of its nodes, then its records in (node, vertex)
// order.  A bucket that fits the LDS is read once into registers; counting
// a record's node also gives it a slot among that node's records, the LDS
// holds the vertices grouped by node, and each record is ranked from its
// registers.
template <typename T>
__global__ __launch_bounds__(kBucketThreads, sizeof(T) == sizeof(float) ? 5 : 4) void k_bucket_sort(BBatch<T> bt) {
  const BOne<T>& c = blockIdx.y == 0 ? bt.c[0] : (blockIdx.y == 1 ? bt.c[1] : bt.c[2]);
  const BucketSpan* __restrict__ list = c.list;
  BucketRec<T>* __restrict__ rec = c.rec;
  int32_t* __restrict__ tcol = c.tcol;
  T* __restrict__ tval = c.tval;
  int64_t* __restrict__ trowptr = c.trowptr;
  int32_t* __restrict__ rowmap = c.rowmap;
  constexpr int R = kSortCap / kBucketThreads;
  __shared__ int32_t ncnt[kBucketNodes], noff[kBucketNodes], nfill[kBucketNodes];
  __shared__ int32_t sr[kSortCap];
  const int64_t full = c.touched[1];
  for (int64_t at = blockIdx.x; at < full; at += gridDim.x) {
    const BucketSpan e = list[at];
    const int64_t a = e.a;
    const int n = e.n;
    const int t = threadIdx.x;
    const bool fits = n <= kSortCap;
    if (t < kBucketNodes) {
      ncnt[t] = 0;
      nfill[t] = 0;
    }
    BucketRec<T> x[R];
    int slot[R];
    if (fits) {
#pragma unroll
      for (int i = 0; i < R; ++i)
        if (t + i * kBucketThreads < n) x[i] = rec[a + t + i * kBucketThreads];
    }
    __syncthreads();
    if (fits) {
#pragma unroll
      for (int i = 0; i < R; ++i)
        if (t + i * kBucketThreads < n) slot[i] = atomicAdd(&ncnt[x[i].nl()], 1);
    } else {
      for (int j = t; j < n; j += kBucketThreads) atomicAdd(&ncnt[rec[a + j].nl()], 1);
    }
    __syncthreads();
    if (t < kWave) {  // the first wave: node offsets, and the touched nodes' rows
      const int cn = t < kBucketNodes ? ncnt[t] : 0;
      int y = cn;
      for (int o = 1; o < kBucketNodes; o <<= 1) {
        const int z = __shfl_up(y, o, kWave);
        if (t >= o) y += z;
      }
      const uint64_t m = ballot64(cn > 0);
      if (t < kBucketNodes) noff[t] = y - cn;
      if (cn > 0) {
        const int64_t row = e.t + rank_below(m);
        trowptr[row] = a + (y - cn);
        rowmap[row] = (e.b << kBucketBits) | t;
      }
    }
    __syncthreads();
    if (fits) {
#pragma unroll
      for (int i = 0; i < R; ++i)
        if (t + i * kBucketThreads < n) sr[noff[x[i].nl()] + slot[i]] = x[i].r();
      __syncthreads();
      // a record's place in its row: the row's vertices below its own
#pragma unroll
      for (int i = 0; i < R; ++i) {
        if (t + i * kBucketThreads >= n) continue;
        const int nl = x[i].nl();
        const int s0 = noff[nl], s1 = s0 + ncnt[nl];
        const int32_t r = x[i].r();
        int rank = 0, u = s0;
        for (; u + 8 <= s1; u += 8) {  // eight reads in flight
          int32_t y[8];
#pragma unroll
          for (int k = 0; k < 8; ++k) y[k] = sr[u + k];
#pragma unroll
          for (int k = 0; k < 8; ++k) rank += y[k] < r ? 1 : 0;
        }
        for (; u < s1; ++u) rank += sr[u] < r ? 1 : 0;
        tcol[a + s0 + rank] = r;
        tval[a + s0 + rank] = x[i].v;
      }
    } else {
      // more records than the LDS holds: group them by node in B^dT's arrays,
      // copy the grouped records back over the bucket's (consumed) ones, then
      // rank each node's records against its row, kSortCap of the row's
      // vertices at a time through LDS
      for (int j = t; j < n; j += kBucketThreads) {
        const BucketRec<T> g = rec[a + j];
        const int64_t q = a + noff[g.nl()] + atomicAdd(&nfill[g.nl()], 1);
        tcol[q] = g.r();
        tval[q] = g.v;
      }
      __syncthreads();
      for (int j = t; j < n; j += kBucketThreads) {
        BucketRec<T> g;
        g.v = tval[a + j];
        g.rn = uint32_t(tcol[a + j]) << kBucketBits;
        rec[a + j] = g;
      }
      for (int nl = 0; nl < kBucketNodes; ++nl) {
        const int L = ncnt[nl];
        const int64_t s0 = a + noff[nl];
        for (int q0 = 0; q0 < L; q0 += kBucketThreads) {
          const int q = q0 + t;
          BucketRec<T> g;
          g.v = T(0);
          g.rn = 0;
          int rank = 0;
          for (int c0 = 0; c0 < L; c0 += kSortCap) {
            const int m = min(kSortCap, L - c0);
            __syncthreads();  // the grouped records are written; sr is free
            if (c0 == 0 && q < L) g = rec[s0 + q];
            for (int u = t; u < m; u += kBucketThreads) sr[u] = rec[s0 + c0 + u].r();
            __syncthreads();
            if (q < L)
              for (int u = 0; u < m; ++u) rank += sr[u] < g.r() ? 1 : 0;
          }
          if (q < L) {
            tcol[s0 + rank] = g.r();
            tval[s0 + rank] = g.v;
          }
        }
      }
    }
    __syncthreads();  // the LDS is free for the next bucket
  }
}

// Whether B^d is transposed through the buckets: from 2^18 nonzeros, with
// fewer than 4,096 rows (whose blocks of 64 rows leave most of the card idle)
// from 2^22; or from IBVT_BUCKET_NNZ nonzeros (the environment, a positive
// integer; small values put small operators through the bucket path, as the
// tests do).  Both paths give the same B^dT.  Microseconds for three
// components through the buckets / the counting sort (double within 5 % of
// float), by rows, nonzeros and lattice nodes of each:
//      63,   8k, 0.03M:  82 /  36       63,  95k,  2.1M: 868 / 195
//     756,  40k, 0.1M:   69 /  44      756, 491k,  7.1M: 463 / 158
//   1,519,  82k, 0.3M:   75 /  60    1,519, 774k, 11.3M: 426 / 197
//   3,321, 129k, 0.3M:   72 /  90    3,321, 778k,  7.1M: 208 / 169
//   3,969, 367k, 2.1M:  109 / 143    3,969, 1.0M, 11.3M: 252 / 225
//   9,648, 432k, 0.9M:   95 / 123    9,648, 1.4M, 11.3M: 182 / 288
//   9,648, 576k, 2.1M:  100 / 265   37,544, 2.4M,  7.1M: 216 / 427
// The buckets take 55 us and 0.55 for each nonzero of a row (a block's rounds
// follow one another), the counting sort 35 us and some 14 for each million
// nodes: below the lines the one or the other wins by up to a third, by its
// lattice and its rows' length, past them the buckets.
bool use_buckets(int64_t nnz, int64_t n_rows) {
  if (const char* e = std::getenv("IBVT_BUCKET_NNZ")) {
    char* end = nullptr;
    const long long v = std::strtoll(e, &end, 10);
    if (end != e && *end == '\0' && v > 0) return nnz >= int64_t(v);
  }
  return nnz >= (n_rows < 4096 ? int64_t(1) << 22 : int64_t(1) << 18);
}

inline unsigned blocks_for(int64_t n, int threads) {
  return unsigned(ceil_div(n > 0 ? n : 1, threads));
}

// Where B^dT's row pointers and row maps go: its rows are counted on the
// device, and waiting for the counts costs some 45 us of a step.  They cannot
// exceed the nonzeros or the lattice's nodes, but may be tens of times fewer
// (200k tets in 192^3 cells: 83 MB by that bound, 3 by the rows), and the
// arrays live as long as the handle.  So they are allocated by the bound only
// where that is little; otherwise the rows go to scratch, which
// coupling_release_scratch gives back, and are copied once the counts have
// been read with the assembly's others (transpose_done); and where the
// components do not go through the buckets together (kBatchRecords; three
// bodies of 4.5M tets: 1.2 GB), or their scratch is never given back (planar
// and tet backgrounds), the counts are waited for.
constexpr int64_t kLooseRows = int64_t(32) << 20, kStagedRows = int64_t(384) << 20;  // bytes
int64_t rows_bound(const ibvt_coupling* c, int d) {
  return std::min<int64_t>(c->B[d].nnz, c->n_fluid[d]);
}

// For all components of an assembly together; wait: the counts are to be
// waited for.
int stage_rows(ibvt_coupling* c, int n, bool& wait) {
  constexpr int64_t per_row = sizeof(int64_t) + sizeof(int32_t);
  int64_t all = 0;
  for (int d = 0; d < n; ++d) {
    all += rows_bound(c, d) + 2;
    c->trows_from[d] = ibvt_coupling::StagedRows{};
  }
  const bool little = all * per_row <= kLooseRows;
  const bool scratch = all * per_row <= kStagedRows && c->dim == 3 && !c->unstructured;
  wait = !little && !scratch;
  if (little || wait) return IBVT_OK;
  if (int st = ensure(c, c->trows, size_t(all * per_row))) return st;
  int64_t* rp = c->trows.as<int64_t>();
  int32_t* rm = reinterpret_cast<int32_t*>(rp + all);
  for (int d = 0; d < n; ++d) {
    c->trows_from[d] = {rp, rm};
    rp += rows_bound(c, d) + 2;
    rm += rows_bound(c, d) + 2;
  }
  return IBVT_OK;
}

// The row arrays of the components of one launch, their counts enqueued.
template <typename One>
int transpose_rows(ibvt_coupling* c, const int* ds, int n, bool wait, One* one, hipStream_t s) {
  int64_t rows[3];
  const int64_t* src[3];
  int st;
  for (int k = 0; k < n; ++k) {
    rows[k] = rows_bound(c, ds[k]);
    src[k] = one[k].touched;
  }
  if (wait && (st = read_counts(c, src, n, rows, s))) return st;
  for (int k = 0; k < n; ++k) {
    Csr& Bt = c->Bt[ds[k]];
    one[k].trowptr = c->trows_from[ds[k]].rowptr;
    one[k].rowmap = c->trows_from[ds[k]].rowmap;
    if (one[k].trowptr) continue;
    if ((st = ensure(c, Bt.rowptr, size_t(rows[k] + 1) * sizeof(int64_t)))) return st;
    if ((st = ensure(c, Bt.rowmap, size_t(rows[k] + 1) * sizeof(int32_t)))) return st;
    one[k].trowptr = Bt.rowptr.template as<int64_t>();
    one[k].rowmap = Bt.rowmap.template as<int32_t>();
  }
  return IBVT_OK;
}

// Staged rows into the arrays of B^dT (blockIdx.y: the component).
struct RowCopies {
  const int64_t* rp[3];
  const int32_t* rm[3];
  int64_t* to_rp[3];
  int32_t* to_rm[3];
  int64_t rows[3];
};
__global__ __launch_bounds__(256) void k_copy_rows(RowCopies r) {
  const int d = blockIdx.y;
  const int64_t n = d == 0 ? r.rows[0] : (d == 1 ? r.rows[1] : r.rows[2]);
  const int64_t* rp = d == 0 ? r.rp[0] : (d == 1 ? r.rp[1] : r.rp[2]);
  const int32_t* rm = d == 0 ? r.rm[0] : (d == 1 ? r.rm[1] : r.rm[2]);
  int64_t* to_rp = d == 0 ? r.to_rp[0] : (d == 1 ? r.to_rp[1] : r.to_rp[2]);
  int32_t* to_rm = d == 0 ? r.to_rm[0] : (d == 1 ? r.to_rm[1] : r.to_rm[2]);
  const int64_t k = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (k <= n) to_rp[k] = rp[k];
  if (k < n) to_rm[k] = rm[k];
}

// Counting sort over the whole lattice (small operators; nnz == 0 too) of
// the n components in ds.  The counts of touched nodes stay on the device,
// in touched.
template <typename T>
int transpose_counting(ibvt_coupling* c, const int* ds, int n, bool wait, const int64_t** touched,
                       hipStream_t s) {
  TBatch<T> b{};
  b.n = n;
  int64_t tiles = 0, nnz = 0, nnz_max = 0, rows_max = 0;
  for (int k = 0; k < n; ++k) {
    b.c[k].tile0 = tiles;
    b.c[k].tiles = ceil_div(c->n_fluid[ds[k]], kTTile);
    tiles += b.c[k].tiles;
  }
  int st;
  const size_t node_b = size_t(tiles) * kTTile * sizeof(int32_t);
  if ((st = ensure(c, c->mark, node_b + size_t(tiles) * sizeof(uint64_t)))) return st;
  if ((st = ensure(c, c->tcnt, 6 * sizeof(int64_t)))) return st;
  for (int k = 0; k < n; ++k) {
    const Csr& B = c->B[ds[k]];
    Csr& Bt = c->Bt[ds[k]];
    TOne<T>& o = b.c[k];
    const int64_t rows = std::min<int64_t>(B.nnz, c->n_fluid[ds[k]]);
    Bt.nnz = B.nnz;
    if ((st = ensure(c, Bt.col, size_t(B.nnz + 1) * sizeof(int32_t)))) return st;
    if ((st = ensure(c, Bt.val, size_t(B.nnz + 1) * sizeof(T)))) return st;
    o.rowptr = B.rowptr.template as<int64_t>();
    o.col = B.col.template as<int32_t>();
    o.val = B.val.template as<T>();
    o.nnz = B.nnz;
    o.node = c->mark.as<int32_t>() + o.tile0 * kTTile;
    o.sum = reinterpret_cast<uint64_t*>(c->mark.as<char>() + node_b) + o.tile0;
    o.touched = c->tcnt.as<int64_t>() + 2 * ds[k];
    o.tcol = Bt.col.template as<int32_t>();
    o.tval = Bt.val.template as<T>();
    touched[ds[k]] = o.touched;
    nnz += B.nnz;
    nnz_max = std::max(nnz_max, B.nnz);
    rows_max = std::max(rows_max, rows);
  }
  if ((st = ensure(c, c->tbuf, size_t(nnz) * sizeof(ValRow<T>)))) return st;
  for (int64_t k = 0, at = 0; k < n; at += b.c[k++].nnz) b.c[k].vr = c->tbuf.as<ValRow<T>>() + at;
  if ((st = hip_check(hipMemsetAsync(c->mark.p, 0, node_b, s), "memset"))) return st;
  const unsigned un = unsigned(n);
  if (nnz_max) k_tcount<T><<<dim3(blocks_for(nnz_max, 256), un), 256, 0, s>>>(b);
  k_tsums<T><<<unsigned(tiles), kTThreads, 0, s>>>(b);
  k_tscan<T><<<un, 1024, 0, s>>>(b);
  if ((st = transpose_rows(c, ds, n, wait, b.c, s))) return st;
  k_ttiles<T><<<unsigned(tiles), kTThreads, 0, s>>>(b);
  if (nnz_max) {
    k_tscatter<T><<<dim3(blocks_for(c->n_vert * kKeyLanes, 256), un), 256, 0, s>>>(b, c->n_vert);
    k_trow_order<T><<<dim3(std::min(blocks_for(rows_max * kWave, 256), kTOrderBlocks), un), 256, 0,
                      s>>>(b);
  }
  return hip_check(hipGetLastError(), "transpose launch");
}

// Bucket transpose of the n components in ds; the counts as in
// transpose_counting.
template <typename T>
int transpose_buckets(ibvt_coupling* c, const int* ds, int n, bool wait, const int64_t** touched,
                      hipStream_t s) {
  BBatch<T> b{};
  b.n = n;
  auto al = [](size_t x) { return (x + 255) & ~size_t(255); };
  int st;
  if ((st = ensure(c, c->tcnt, 6 * sizeof(int64_t)))) return st;
  size_t zero = 0, rest = 0;
  int64_t tiles = 0, nb_max = 0, nnz_max = 0;
  size_t zero_at[3], rest_at[3];
  for (int k = 0; k < n; ++k) {
    const Csr& B = c->B[ds[k]];
    Csr& Bt = c->Bt[ds[k]];
    BOne<T>& o = b.c[k];
    const int64_t nf = c->n_fluid[ds[k]];
    Bt.nnz = B.nnz;
    if ((st = ensure(c, Bt.col, size_t(B.nnz + 1) * sizeof(int32_t)))) return st;
    if ((st = ensure(c, Bt.val, size_t(B.nnz + 1) * sizeof(T)))) return st;
    o.rowptr = B.rowptr.template as<int64_t>();
    o.col = B.col.template as<int32_t>();
    o.val = B.val.template as<T>();
    o.nnz = B.nnz;
    o.nb = ceil_div(nf, kBucketNodes);
    o.tiles = ceil_div(o.nb, kBTile);
    o.tile0 = tiles;
    tiles += o.tiles;
    nb_max = std::max(nb_max, o.nb);
    nnz_max = std::max(nnz_max, o.nnz);
    o.touched = c->tcnt.as<int64_t>() + 2 * ds[k];
    touched[ds[k]] = o.touched;
    o.tcol = Bt.col.template as<int32_t>();
    o.tval = Bt.val.template as<T>();
    zero_at[k] = zero;
    rest_at[k] = rest;
    zero += 2 * al(size_t(o.nb) * sizeof(int32_t)) + al(size_t(o.nb) * kBucketNodes);
    rest += al(size_t(B.nnz) * sizeof(BucketRec<T>)) + al(size_t(o.nb) * sizeof(int32_t)) +
            al(size_t(o.nb) * sizeof(BucketSpan)) + al(size_t(o.tiles) * sizeof(BucketSums));
  }
  if ((st = ensure(c, c->tbuf, zero + rest))) return st;
  for (int k = 0; k < n; ++k) {
    BOne<T>& o = b.c[k];
    char* p = c->tbuf.as<char>() + zero_at[k];
    const size_t i32 = al(size_t(o.nb) * sizeof(int32_t));
    o.bcount = reinterpret_cast<int32_t*>(p);
    o.bfill = reinterpret_cast<int32_t*>(p + i32);
    o.mark = reinterpret_cast<uint8_t*>(p + 2 * i32);
    p = c->tbuf.as<char>() + zero + rest_at[k];
    o.rec = reinterpret_cast<BucketRec<T>*>(p);
    p += al(size_t(o.nnz) * sizeof(BucketRec<T>));
    o.boff = reinterpret_cast<int32_t*>(p);
    p += i32;
    o.list = reinterpret_cast<BucketSpan*>(p);
    o.sum = reinterpret_cast<BucketSums*>(p + al(size_t(o.nb) * sizeof(BucketSpan)));
  }
  if ((st = hip_check(hipMemsetAsync(c->tbuf.p, 0, zero, s), "memset"))) return st;
  const int64_t n_rows = c->n_vert;
  const int64_t per = ceil_div(ceil_div(n_rows, kBucketRows), 8);
  const unsigned un = unsigned(n);
  const dim3 grid(unsigned(8 * per), un);
  k_bucket_count<T><<<grid, kBucketThreads, 0, s>>>(b, n_rows, per);
  k_bucket_tiles<T><<<unsigned(tiles), kBucketThreads, 0, s>>>(b);
  k_bucket_scan<T><<<un, 1024, 0, s>>>(b);
  if ((st = transpose_rows(c, ds, n, wait, b.c, s))) return st;
  k_bucket_list<T><<<unsigned(tiles), kBucketThreads, 0, s>>>(b);
  k_bucket_scatter<T><<<grid, kBucketThreads, 0, s>>>(b, n_rows, per);
  // (the number of nonempty buckets is on the device: a block for 512
  // nonzeros, the blocks loop)
  const int64_t sort_blocks = std::min<int64_t>({nb_max, 65536, nnz_max / 512 + 64});
  k_bucket_sort<T><<<dim3(unsigned(sort_blocks), un), kBucketThreads, 0, s>>>(b);
  return hip_check(hipGetLastError(), "transpose launch");
}

}  // namespace

// Components with fewer nonzeros than the bucket transpose is for go through
// the counting sort together, the others through the buckets: together while
// their records are few, else one after the other in the same scratch.
// Large ones that have too many vertices for the buckets take the counting
// sort one by one.
template <typename T>
int transposes(ibvt_coupling* c, int n, const int64_t** touched, hipStream_t s) {
  int small[3], large[3], ns = 0, nl = 0, st;
  int64_t records = 0;
  bool wait;
  if ((st = stage_rows(c, n, wait))) return st;
  for (int d = 0; d < n; ++d) {
    if (!use_buckets(c->B[d].nnz, c->n_vert)) {
      small[ns++] = d;
    } else if (c->n_vert < kBucketMaxVert) {
      large[nl++] = d;
      records += c->B[d].nnz;
    } else if ((st = transpose_counting<T>(c, &d, 1, wait, touched, s))) {
      return st;
    }
  }
  if (nl && records <= kBatchRecords) {
    if ((st = transpose_buckets<T>(c, large, nl, wait, touched, s))) return st;
  } else {
    for (int k = 0; k < nl; ++k)
      if ((st = transpose_buckets<T>(c, large + k, 1, wait, touched, s))) return st;
  }
  return ns ? transpose_counting<T>(c, small, ns, wait, touched, s) : IBVT_OK;
}

int transpose_done(ibvt_coupling* c, int n, const int64_t* rows, hipStream_t s) {
  RowCopies r{};
  int64_t most = -1;
  int st;
  for (int d = 0; d < n; ++d) {
    Csr& Bt = c->Bt[d];
    Bt.nrows = rows[d];
    r.rows[d] = -1;  // nothing to copy
    const auto from = c->trows_from[d];
    if (!from.rowptr) continue;
    if ((st = ensure(c, Bt.rowptr, size_t(rows[d] + 1) * sizeof(int64_t)))) return st;
    if ((st = ensure(c, Bt.rowmap, size_t(rows[d] + 1) * sizeof(int32_t)))) return st;
    r.rows[d] = rows[d];
    r.rp[d] = from.rowptr;
    r.rm[d] = from.rowmap;
    r.to_rp[d] = Bt.rowptr.as<int64_t>();
    r.to_rm[d] = Bt.rowmap.as<int32_t>();
    most = std::max(most, rows[d]);
  }
  if (most < 0) return IBVT_OK;
  k_copy_rows<<<dim3(blocks_for(most + 1, 256), unsigned(n)), 256, 0, s>>>(r);
  return hip_check(hipGetLastError(), "transpose rows launch");
}

template int transposes<float>(ibvt_coupling*, int, const int64_t**, hipStream_t);
template int transposes<double>(ibvt_coupling*, int, const int64_t**, hipStream_t);

}  // namespace ibvt
