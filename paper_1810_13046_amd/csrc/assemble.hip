// Assembly of the mortar matrices B^d (Section 2.3, steps (I)-(IV)).
//
//  k_tet_prep      per tet: bounding box -> cell index range on each
//                  component's lattice (replaces the tree search: on a
//                  rectilinear grid the overlap candidates of a tet are an
//                  index box), volume, geometry record, validity checks.
//  scan            candidate (tet, component, cell) pair offsets.
//  k_order_count / k_order_scatter
//                  per chunk: the pairs' 16-byte descriptors in clip
//                  order (key: the cell planes the tet straddles, in
//                  classes by cut count: vertex slots 10, 12, 16), counted
//                  and placed per (tet, key) group from the cell ranges.
//  k_pieces        (FP64, the items within the limits of moments.hpp) the
//                  pieces' moments and the 32 values ∫ λ_i N_j per pair from
//                  boundary integrals, without clipped polyhedra; the
//                  order, k_clip and k_integrate serve the others.
//  k_clip<T,MAXV>  one lane per pair: clip the tet by the straddled cell
//                  planes in double (vertex graph in LDS), fan the piece
//                  into sub-tetrahedra and store them as records.
//  k_integrate<T>  one lane per record: its 32 cell-local moments, summed
//                  per pair; then one lane per pair turns them into the 32
//                  values ∫ λ_i N_j.
//  k_row_box / k_rows<T> / k_rows_compact<T>
//                  each (solid vertex, component) row gathered in an LDS
//                  node box after each chunk's integration (rows whose
//                  pairs span chunks keep double partial sums between
//                  chunks), pairs added in a fixed order (deterministic,
//                  no value atomics outside LDS), written column-sorted,
//                  then compacted into CSR.
//  transpose       B^dT over the touched fluid nodes (transpose.hip).
//  masses          lumped m_i = Σ_{T∋i} |T|/4 and the consistent P1 mass
//                  matrix |T|(1+δ_il)/20 (Section 2.1), per vertex in
//                  incident-tet order.

#include "internal.hpp"
#include "moments.hpp"

#include <climits>
#include <cstdlib>

namespace ibvt {

namespace {

constexpr int kRowNodes = 640;  // LDS box nodes of a wave's rows per pass in k_rows

__device__ __forceinline__ int upper_bound_d(const double* L, int n, double x) {
  int lo = 0, hi = n;  // first index with L[idx] > x
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (L[mid] <= x) lo = mid + 1; else hi = mid;
  }
  return lo;
}

__device__ __forceinline__ int lower_bound_d(const double* L, int n, double x) {
  int lo = 0, hi = n;  // first index with L[idx] >= x
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (L[mid] < x) lo = mid + 1; else hi = mid;
  }
  return lo;
}

// ---------------------------------------------------------------------------
// topology: vertex -> incident tets
// ---------------------------------------------------------------------------

// K vertices per element: 4 (tetrahedra) or 3 (triangles, the planar case).
template <int K>
__global__ void k_vt_count(int64_t n_t, int64_t n_v, const int32_t* __restrict__ tets,
                           unsigned long long* __restrict__ deg, unsigned* flags) {
  const int64_t t = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (t >= n_t) return;
  int v[K];
  bool bad = false;
  for (int k = 0; k < K; ++k) {
    v[k] = tets[K * t + k];
    bad |= (v[k] < 0) || (int64_t(v[k]) >= n_v);
  }
  for (int a = 0; a < K; ++a)
    for (int b = a + 1; b < K; ++b) bad |= (v[a] == v[b]);
  if (bad) {
    atomicOr(flags, kFlagValence);
    return;
  }
  for (int k = 0; k < K; ++k) atomicAdd(&deg[v[k]], 1ull);
}

template <int K>
__global__ void k_vt_fill(int64_t n_t, const int32_t* __restrict__ tets,
                          const int64_t* __restrict__ vt_ptr, unsigned long long* __restrict__ cur,
                          int32_t* __restrict__ vt_tet) {
  const int64_t t = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (t >= n_t) return;
  for (int k = 0; k < K; ++k) {
    const int v = tets[K * t + k];
    const int64_t pos = vt_ptr[v] + int64_t(atomicAdd(&cur[v], 1ull));
    vt_tet[pos] = int32_t(t);
  }
}

__global__ void k_sort_segments_i32(int64_t n, const int64_t* __restrict__ ptr,
                                    int32_t* __restrict__ key) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int64_t b = ptr[i], e = ptr[i + 1];
  for (int64_t k = b + 1; k < e; ++k) {
    const int32_t x = key[k];
    int64_t j = k - 1;
    while (j >= b && key[j] > x) {
      key[j + 1] = key[j];
      --j;
    }
    key[j + 1] = x;
  }
}

// Consistent-mass pattern: distinct vertices of the incident elements.
template <int K, bool FILL>
__global__ void k_mass_pattern(int64_t n_v, const int64_t* __restrict__ vt_ptr,
                               const int32_t* __restrict__ vt_tet, const int32_t* __restrict__ tets,
                               int64_t* __restrict__ rowcnt, const int64_t* __restrict__ rowptr,
                               int32_t* __restrict__ col) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= n_v) return;
  const int64_t b = vt_ptr[i], e = vt_ptr[i + 1];
  int cur = -1;
  int64_t cnt = 0;
  int64_t pos = FILL ? rowptr[i] : 0;
  for (;;) {
    int nxt = INT_MAX;
    for (int64_t k = b; k < e; ++k) {
      const int64_t t = vt_tet[k];
      for (int q = 0; q < K; ++q) {
        const int v = tets[K * t + q];
        if (v > cur && v < nxt) nxt = v;
      }
    }
    if (nxt == INT_MAX) break;
    if (FILL) col[pos++] = nxt;
    ++cnt;
    cur = nxt;
  }
  if (!FILL) rowcnt[i] = cnt;
}

// ---------------------------------------------------------------------------
// per-tet preparation
// ---------------------------------------------------------------------------

// clipped (or null): set for the (component, tet) items whose pieces are
// clipped, not integrated over their boundary (moments.hpp).
__global__ void k_tet_prep(int64_t n_t, const double* __restrict__ X,
                           const int32_t* __restrict__ tets, const double* __restrict__ lat,
                           LatDesc ld, double* __restrict__ tetvol, CellRange* __restrict__ rng,
                           int64_t* __restrict__ cnt, double* __restrict__ tetrec,
                           double* __restrict__ tetgrad, uint8_t* __restrict__ clipped,
                           unsigned* flags, unsigned long long* counters) {
  const int64_t t = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  bool zero = false;
  uint32_t to_clip = 0;  // pairs of the items marked in `clipped`
  if (t < n_t) {
    double P[4][3];
    bool finite = true;
    for (int k = 0; k < 4; ++k) {
      const int64_t v = tets[4 * t + k];
      for (int e = 0; e < 3; ++e) {
        P[k][e] = X[3 * v + e];
        finite &= isfinite(P[k][e]);
      }
    }
    double mn[3], mx[3];
    for (int e = 0; e < 3; ++e) {
      mn[e] = fmin(fmin(P[0][e], P[1][e]), fmin(P[2][e], P[3][e]));
      mx[e] = fmax(fmax(P[0][e], P[1][e]), fmax(P[2][e], P[3][e]));
    }
    double a[3], b[3], c[3];
    for (int e = 0; e < 3; ++e) {
      a[e] = P[1][e] - P[0][e];
      b[e] = P[2][e] - P[0][e];
      c[e] = P[3][e] - P[0][e];
    }
    const double det = a[0] * (b[1] * c[2] - b[2] * c[1]) - a[1] * (b[0] * c[2] - b[2] * c[0]) +
                       a[2] * (b[0] * c[1] - b[1] * c[0]);
    const double vol = fabs(det) / 6.0;
    tetvol[t] = finite ? vol : 0.0;
    double range;
    {
      TetGeom G;
      for (int k = 0; k < 4; ++k)
        for (int e = 0; e < 3; ++e) G.V[k][e] = P[k][e];
      tet_geom(G);
      double r[kTetRec];
      store_tet_rec(G, r);
      store_row<kTetRec>(tetrec + t * kTetRec, r);
      double g[12];
      for (int k = 0; k < 4; ++k)
        for (int e = 0; e < 3; ++e) g[3 * k + e] = G.g[k][e];
      store_row<12>(tetgrad + t * 12, g);
      range = hat_range(G.g, mn, mx);
    }
    zero = finite && (vol == 0.0);
    if (!finite) atomicOr(flags, kFlagNonFinite);
    for (int d = 0; d < 3; ++d) {
      CellRange r;
      bool ok = finite && !zero;
      for (int e = 0; e < 3; ++e) {
        const double* L = lat + ld.off[3 * d + e];
        const int n = ld.n[3 * d + e];
        if (!(mn[e] >= L[0] && mx[e] <= L[n - 1])) {
          if (finite) atomicOr(flags, kFlagOutOfGrid);
          ok = false;
          r.lo[e] = 0;
          r.n[e] = 0;
          continue;
        }
        int lo = upper_bound_d(L, n, mn[e]) - 1;
        lo = min(max(lo, 0), n - 2);
        int hi = lower_bound_d(L, n, mx[e]) - 1;
        hi = min(max(hi, lo), n - 2);
        r.lo[e] = lo;
        r.n[e] = hi - lo + 1;
      }
      if (!ok) r.n[0] = r.n[1] = r.n[2] = 0;
      rng[d * n_t + t] = r;
      cnt[d * n_t + t] = int64_t(r.n[0]) * r.n[1] * r.n[2];
      if (int64_t(r.n[0]) * r.n[1] * r.n[2] > kMaxTetCells) atomicOr(flags, kFlagTetSpan);
      if (clipped) {
        bool cl = max(r.n[0], max(r.n[1], r.n[2])) > kOctantCells || !(range <= kOctantRange);
        if (ok && !cl) {
          double product = 1.0;
          for (int e = 0; e < 3; ++e) {
            const double x = axis_reach(lat + ld.off[3 * d + e] + r.lo[e], r.n[e], mn[e], mx[e]);
            product *= x;
            cl |= !(x <= kOctantReach);
          }
          cl |= !(product <= kOctantProduct);
        }
        clipped[d * n_t + t] = cl ? 1 : 0;
        if (cl) to_clip += uint32_t(r.n[0]) * uint32_t(r.n[1]) * uint32_t(r.n[2]);
      }
    }
  }
  const uint64_t zm = ballot64(zero);
  if (lane_id() == 0 && zm) atomicAdd(&counters[kCntZeroTets], (unsigned long long)popc64(zm));
  if (clipped) {
    const unsigned long long n = wave_sum((unsigned long long)to_clip);
    if (lane_id() == 0 && n) atomicAdd(&counters[kCntToClip], n);
  }
}

// ---------------------------------------------------------------------------
// clip + integrate, one lane per (tet, component, cell) pair
// ---------------------------------------------------------------------------

// The clip order of a chunk, from the cell ranges alone.  Which of the six
// cell planes a pair's tet straddles follows from indices: the low plane of
// cell ci cuts the tet iff ci > the first cell of the tet's range along that
// axis, the high plane iff ci < the last.  Sort key = class · 64 + pattern
// (the straddled planes, two bits per axis), class 0: <= 3 cuts, 1: 4,
// 2: >= 5 (classes need 10, 12, 16 vertex slots); ordering the pairs by
// key gives every wave the same sequence of clips.  Along an axis with n
// cells the pairs fall into at most three runs (first cell, inner cells,
// last cell), so a (component, tet) item's pairs form at most 27 groups of
// one key each, counted and placed per group:
//   k_order_count    per block of kOrderItems items: pairs per key (LDS
//                    integer atomics) → hist[key][block];
//   scan             → the first place of each (key, block), key-major, so
//                    entry 64·k·blocks is where class k starts;
//   k_order_scatter  each item takes chunk-local places for its groups
//                    from its block's running offsets (LDS atomics: the
//                    order within a key depends on timing, which changes no
//                    result: a pair's clip and its records depend on the
//                    pair alone) and writes the groups' descriptors
//                    (pair_desc's fields), and the owner (the item's index)
//                    of each of its pairs.
// Items not marked in `clipped` (null: all are clipped) are left out.
constexpr int kOrderItems = 256;

struct AxisRuns {
  int n;          // runs along the axis (1, 2 or 3)
  int start[3];   // first cell of each run (range-relative)
  int count[3];   // cells in each run
  int bits[3];    // straddled planes of the run's cells: 1 low, 2 high
};

__device__ __forceinline__ AxisRuns axis_runs(int n) {
  AxisRuns a;
  if (n <= 1) {
    a.n = 1;
    a.start[0] = 0; a.count[0] = n; a.bits[0] = 0;
  } else {
    a.n = n > 2 ? 3 : 2;
    a.start[0] = 0; a.count[0] = 1; a.bits[0] = 2;
    a.start[1] = n - 1; a.count[1] = 1; a.bits[1] = 1;
    a.start[2] = 1; a.count[2] = n - 2; a.bits[2] = 3;
  }
  return a;
}

__device__ __forceinline__ int order_key(int pattern) {
  const int cuts = __popc(pattern);
  return (cuts <= 3 ? 0 : (cuts == 4 ? 1 : 2)) * 64 + pattern;
}

__global__ __launch_bounds__(kOrderItems) void k_order_count(int64_t tc0, int64_t n_items,
                                                             const CellRange* __restrict__ rng,
                                                             const uint8_t* __restrict__ clipped,
                                                             int32_t* __restrict__ hist) {
  __shared__ int32_t h[256];
  const int64_t nb = gridDim.x;
  h[threadIdx.x] = 0;
  __syncthreads();
  const int64_t w = int64_t(blockIdx.x) * kOrderItems + threadIdx.x;
  if (w < n_items && (!clipped || clipped[tc0 + w])) {
    const CellRange r = rng[tc0 + w];
    if (int64_t(r.n[0]) * r.n[1] * r.n[2] > 0) {
      const AxisRuns ax = axis_runs(r.n[0]), ay = axis_runs(r.n[1]), az = axis_runs(r.n[2]);
      for (int c = 0; c < az.n; ++c)
        for (int b = 0; b < ay.n; ++b)
          for (int a = 0; a < ax.n; ++a) {
            const int cnt = ax.count[a] * ay.count[b] * az.count[c];
            if (cnt > 0)
              atomicAdd(&h[order_key(ax.bits[a] | (ay.bits[b] << 2) | (az.bits[c] << 4))], cnt);
          }
    }
  }
  __syncthreads();
  hist[int64_t(threadIdx.x) * nb + blockIdx.x] = h[threadIdx.x];
}

__global__ __launch_bounds__(kOrderItems) void k_order_scatter(
    int64_t tc0, int64_t n_items, int64_t n_t, const CellRange* __restrict__ rng,
    const uint8_t* __restrict__ clipped, const int64_t* __restrict__ pair_off,
    const int64_t* __restrict__ first,
    PairDesc* __restrict__ order, int32_t* __restrict__ owner) {
  __shared__ unsigned long long cur[256];
  const int64_t nb = gridDim.x;
  cur[threadIdx.x] = (unsigned long long)first[int64_t(threadIdx.x) * nb + blockIdx.x];
  __syncthreads();
  const int64_t w = int64_t(blockIdx.x) * kOrderItems + threadIdx.x;
  if (w >= n_items) return;
  const int64_t tc = tc0 + w;
  if (clipped && !clipped[tc]) return;
  const CellRange r = rng[tc];
  if (int64_t(r.n[0]) * r.n[1] * r.n[2] == 0) return;
  const int d = (tc >= n_t) + (tc >= 2 * n_t);
  const uint32_t td = uint32_t(tc - int64_t(d) * n_t) | (uint32_t(d) << 30);
  const int64_t pb = pair_off[tc];
  const int64_t cnt_all = int64_t(r.n[0]) * r.n[1] * r.n[2];
  for (int64_t q = 0; q < cnt_all; ++q) owner[pb + q] = int32_t(tc);
  const AxisRuns ax = axis_runs(r.n[0]), ay = axis_runs(r.n[1]), az = axis_runs(r.n[2]);
  for (int c = 0; c < az.n; ++c)
    for (int b = 0; b < ay.n; ++b)
      for (int a = 0; a < ax.n; ++a) {
        const int cnt = ax.count[a] * ay.count[b] * az.count[c];
        if (cnt == 0) continue;
        const int key = order_key(ax.bits[a] | (ay.bits[b] << 2) | (az.bits[c] << 4));
        int64_t pos = int64_t(atomicAdd(&cur[key], (unsigned long long)cnt));
        for (int z = az.start[c]; z < az.start[c] + az.count[c]; ++z)
          for (int y = ay.start[b]; y < ay.start[b] + ay.count[b]; ++y)
            for (int x = ax.start[a]; x < ax.start[a] + ax.count[a]; ++x) {
              PairDesc o;
              o.p = int32_t(pb + x + int64_t(r.n[0]) * (y + int64_t(r.n[1]) * z));
              o.td = td;
              o.cell = uint64_t(uint32_t(r.lo[0] + x)) |
                       (uint64_t(uint32_t(r.lo[1] + y)) << kCellBits) |
                       (uint64_t(uint32_t(r.lo[2] + z)) << (2 * kCellBits));
              order[pos++] = o;  // chunk-local place
            }
      }
}

// Clip every (tet, component, cell) pair in double, one lane per pair, and
// store the fan sub-tetrahedra of the piece.  The pairs come as descriptors
// in clip order (pattern-sorted).  The grid is sized to the resident waves
// and each wave loops over batches of 64 pairs.  A wave takes store space in
// chunks of `chunk` records (one atomic per chunk, not per batch:
// same-address atomics serialise device-wide) and hands each batch a
// contiguous block of its chunk, so every pair's records are contiguous and
// in fan order; the unused tail of a chunk is left empty.  The counters are
// summed per wave and added once at the end.
//
// Bound: vector and scalar issue, with the LDS (28 bytes per slot and lane)
// holding two waves a SIMD where the graph is kept.  The first three planes
// that cut are looked up (clip_piece_box): with 10 slots no graph is kept or
// walked and ten waves fit a CU instead of eight; with 12 and 16 slots the
// graph is written once, after the third, and walked from there.  On 84.4M
// pairs all classes took 19.7 ms with the walks nested by vertex and
// neighbour, 17.0 with one step or cut of every lane per round, 11.0 with 10
// slots looked up and take 10.7 with the look-up in all classes; on the
// graded 397k-tet plate with its many pairs of four and more planes 3.65
// became 3.07 by the last step.  A piece without a record, where rounding
// has split a plane's inside or outside, is clipped again by the graph walk
// (with 10 slots its neighbour words are in the lane's own memory).
template <typename T, int MAXV>
__global__ __launch_bounds__(kWave) void k_clip(
    ClipTables tab, const int64_t* __restrict__ cls_first, const int64_t* __restrict__ cls_end,
    const PairDesc* __restrict__ desc_all, const double* __restrict__ tetrec,
    const double* __restrict__ lat, LatDesc ld, double drop_rel, T* __restrict__ pool,
    int64_t pool_cap, uint64_t* __restrict__ pinfo, unsigned long long* pool_used,
    unsigned* flags, unsigned long long* counters) {
  constexpr bool kTable = MAXV == 10;
  __shared__ double sv[3 * MAXV * kWave];
  __shared__ uint32_t snb[kTable ? 1 : MAXV * kWave];
  uint32_t own[kTable ? MAXV : 1];
  const int lane = threadIdx.x;
  // this class's stretch of the pair order (read here, so the host needs
  // no class sizes); chunk ~ 1/8 of a wave's expected records (about 3 per
  // pair), so the unused chunk tails stay a few percent of the store
  const int64_t first = *cls_first;
  const int64_t n_list = *cls_end - first;
  const PairDesc* __restrict__ desc = desc_all + first;
  const int chunk = int(min<int64_t>(
      2048, max<int64_t>(1, (3 * n_list) / (8 * int64_t(gridDim.x)))));
  const PolyView P = slots_view<MAXV>(sv + lane, snb + lane, own);
  unsigned long long nk = 0, nd = 0, ns = 0;
  ClipCount cc;
  unsigned long long cbase = 0;  // next free record of the wave's chunk
  int cleft = 0;                 // records left in it
  bool fail = false;
  for (int64_t p0 = int64_t(blockIdx.x) * kWave; p0 < n_list; p0 += int64_t(gridDim.x) * kWave) {
    const bool active = p0 + lane < n_list;
    TetGeom G;
    double lo[3], hi[3];
    int64_t p = 0;
    Piece<MAXV> o;
    if (active) {
      int d, ci[3];
      int64_t t;
      desc_cell(desc[p0 + lane], lat, ld, p, d, t, ci, lo, hi);
      double r[kTetRec];
      load_row<kTetRec>(tetrec + t * kTetRec, r);
      load_tet_box(G, r);
      clip_piece_box<MAXV>(P, tab, G, lo, hi, o, &cc);
    }
    const int want = o.want;
    int incl = want;
    for (int s = 1; s < kWave; s <<= 1) {
      const int y = __shfl_up(incl, s, kWave);
      if (lane >= s) incl += y;
    }
    const int wave_total = __shfl(incl, kWave - 1, kWave);
    if (wave_total > cleft) {
      const int take = wave_total > chunk ? wave_total : chunk;
      unsigned long long b = 0;
      if (lane == 0) b = atomicAdd(pool_used, (unsigned long long)take);
      cbase = __shfl(b, 0, kWave);
      cleft = take;
    }
    const unsigned long long wbase = cbase;
    cbase += unsigned(wave_total);
    cleft -= wave_total;
    if (active) {
      const int64_t my = int64_t(wbase) + (incl - want);
      const bool fits = my + want <= pool_cap;
      double vol6 = 0.0;
      int nsub = 0;
      bool ok = o.ok;
      if (ok && want > 0) {
        T* rec = pool + my * kRecord;
        ok = fan_local<MAXV>(P, o, lo, hi,
                             [&](const double* a, const double* b, const double* c,
                                 const double* d, double) IBVT_INLINE {
                               T r[kRecord];
#pragma unroll
                               for (int e = 0; e < 3; ++e) {
                                 r[e] = T(a[e]);
                                 r[3 + e] = T(b[e]);
                                 r[6 + e] = T(c[e]);
                                 r[9 + e] = T(d[e]);
                               }
                               if (fits && nsub < want)
                                 store_row<kRecord>(rec + int64_t(nsub) * kRecord, r);
                               ++nsub;
                             },
                             vol6);
      }
      if (ok && nsub != want) ok = false;
      ns += unsigned(nsub);
      if (!ok) {
        fail = true;
        pinfo[p] = 0;
      } else {
        const double cv = (hi[0] - lo[0]) * (hi[1] - lo[1]) * (hi[2] - lo[2]);
        const double vol = vol6 * cv / 6.0;
        const bool kp = vol > drop_rel * (fabs(G.det) / 6.0);
        // records past the store's end were not written: the pair reads as
        // empty, and the host sees the overflow and runs the clip again
        pinfo[p] = (kp && fits) ? ((uint64_t(my) << 8) | uint64_t(nsub)) : 0;
        if (kp) ++nk;
        else if (vol > 0.0) ++nd;
      }
    }
  }
  nk = wave_sum(nk);
  nd = wave_sum(nd);
  ns = wave_sum(ns);
  const unsigned long long ndist = wave_sum((unsigned long long)cc.dist);
  const unsigned long long ncut = wave_sum((unsigned long long)cc.cuts);
  const unsigned long long npl = wave_sum((unsigned long long)cc.planes);
  const uint64_t fm = ballot64(fail);
  if (lane == 0) {
    if (npl) atomicAdd(&counters[kCntPlanes], npl);
    if (nk) atomicAdd(&counters[kCntPieces], nk);
    if (nd) atomicAdd(&counters[kCntDropped], nd);
    if (ns) atomicAdd(&counters[kCntSubtets], ns);
    if (ndist) atomicAdd(&counters[kCntDist], ndist);
    if (ncut) atomicAdd(&counters[kCntCutPts], ncut);
    if (fm) atomicOr(flags, kFlagCapacity);
  }
}

// One wave per group of 64 consecutive pairs, whose records are contiguous:
// records are taken one per lane (balanced whatever the count per pair) and
// summed per pair in record order through LDS (deterministic).  Returns,
// for the group's dense record index s, the owning lane (largest j with
// excl_j <= s, excl = exclusive prefix of the per-pair counts).
__device__ __forceinline__ int owner_lane(int excl, int s) {
  int lo = 0, hi = kWave - 1;
#pragma unroll
  for (int it = 0; it < 6; ++it) {
    const int mid = (lo + hi + 1) >> 1;
    const int e = __shfl(excl, mid, kWave);
    if (e <= s) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

// (III) integrate every stored sub-tetrahedron: its 32 moments (cell-local,
// centred) with the 11-point degree-4 rule, summed per pair in record order through
// LDS (deterministic) into pmom[pair][m] (rows of kMomPad).  Then each lane
// turns its pair's moments into the 4 x 8 values ∫ λ_i N_j, written to
// pval[i][pair - p_begin][j] (the chunk's pairs only; local-vertex major:
// each vertex row of a pair is 8 contiguous values, planes of plane_pairs
// pairs).  Without ALL, pairs of items not marked in `clipped` are passed by
// (a template parameter: asking for it at run time took the float kernel from
// 732 to 772 us on 200k tets).
template <typename T, bool ALL>
__global__ __launch_bounds__(kWave) void k_integrate(
    int64_t plane_pairs, int64_t p_begin, int64_t p_end, int64_t n_t,
    const uint8_t* __restrict__ clipped, const uint64_t* __restrict__ pinfo,
    const T* __restrict__ pool, const int32_t* __restrict__ owner,
    const int64_t* __restrict__ pair_off, const CellRange* __restrict__ rng,
    const double* __restrict__ tetrec, const double* __restrict__ lat, LatDesc ld,
    uint8_t* __restrict__ keep, T* __restrict__ pval, T* __restrict__ pmom, int dual) {
  __shared__ __align__(16) T red[kWave][kMomLds];  // a record's moments per row, padded
  const int lane = threadIdx.x;
  const int64_t g0 = p_begin + int64_t(blockIdx.x) * kWave;
  const int64_t pj = g0 + lane;
  int cnt = 0;
  int64_t beg = 0;
  const bool mine = pj < p_end && (ALL || clipped[owner[pj]]);
  if (!ALL && ballot64(mine) == 0) return;  // (the block is one wave)
  if (mine) {
    const uint64_t pi = pinfo[pj];
    cnt = int(pi & 0xff);
    beg = int64_t(pi >> 8);
    keep[pj] = cnt > 0 ? 1 : 0;
  }
  int incl = cnt;
  for (int o = 1; o < kWave; o <<= 1) {
    const int y = __shfl_up(incl, o, kWave);
    if (lane >= o) incl += y;
  }
  const int excl = incl - cnt;
  const int total = __shfl(incl, kWave - 1, kWave);
  T run = T(0);
  for (int s0 = 0; s0 < total; s0 += kWave) {
    const int s = s0 + lane;
    const int j = owner_lane(excl, s);
    const int ex_j = __shfl(excl, j, kWave);
    const int in_j = __shfl(incl, j, kWave);
    const long long bj = __shfl((long long)beg, j, kWave);
    T M[kMom];
#pragma unroll
    for (int k = 0; k < kMom; ++k) M[k] = T(0);
    if (s < total) {
      T r[kRecord];
      load_row<kRecord>(pool + (int64_t(bj) + (s - ex_j)) * kRecord, r);
      T y[4][3];
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int e = 0; e < 3; ++e) y[v][e] = r[v * 3 + e];
      subtet_moments<T>(y, subtet_det<T>(y[0], y[1], y[2], y[3]), M);
    }
    {
      T Mp[kMomLds];
#pragma unroll
      for (int k = 0; k < kMom; ++k) Mp[k] = M[k];
#pragma unroll
      for (int k = kMom; k < kMomLds; ++k) Mp[k] = T(0);
      store_row<kMomLds>(&red[lane][0], Mp);  // 16-byte LDS writes
    }
    // the record that ends each pair, and each record's pair, are uniform
    // across the wave: a ballot and lane reads (no LDS)
    const uint64_t last = ballot64((s < total) && (s + 1 == in_j));
    __syncthreads();
    if (lane < kMom) {
      const int rows = min(kWave, total - s0);
      for (int r = 0; r < rows; ++r) {
        run += red[r][lane];
        if ((last >> r) & 1ull) {
          pmom[(g0 + __builtin_amdgcn_readlane(j, r)) * kMomPad + lane] = run;
          run = T(0);
        }
      }
    }
    __syncthreads();
  }
  // the block barrier above orders these reads after the other lanes' writes
  if (cnt > 0) {
    T M[kMomPad];
    load_row<kMomPad>(pmom + pj * kMomPad, M);
    int d, ci[3];
    int64_t t;
    double lo[3], hi[3];
    pair_cell(pj, n_t, owner, pair_off, rng, lat, ld, d, t, ci, lo, hi);
    double rec[kTetRec];
    load_row<kTetRec>(tetrec + t * kTetRec, rec);
    T LA[4], LG[4][3];
    rec_cell_lambda<T>(rec, lo, hi, LA, LG);
    const T sc = T(-(hi[0] - lo[0]) * (hi[1] - lo[1]) * (hi[2] - lo[2]) / 6.0);
    const int64_t plane = plane_pairs * 8;
    T b[4][8];
    mom_to_b<T>(M, LA, LG, [&](int i, int jj, T v) { b[i][jj] = sc * v; });
    if (dual) {
      // dual multipliers ψ_i = 5λ_i − Σ_k λ_k: ∫ ψ_i N_j = 5 b_ij − Σ_k b_kj
#pragma unroll
      for (int jj = 0; jj < 8; ++jj) {
        const T sum = b[0][jj] + b[1][jj] + b[2][jj] + b[3][jj];
#pragma unroll
        for (int i = 0; i < 4; ++i) b[i][jj] = T(5) * b[i][jj] - sum;
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) store_row<8>(pval + i * plane + (pj - p_begin) * 8, b[i]);
  }
}

// ---------------------------------------------------------------------------
// pieces by boundary integrals: candidate test, moments and values in one
// kernel
// ---------------------------------------------------------------------------

// The owner ((component, tet) item) of every pair.
__global__ __launch_bounds__(256) void k_owner(int64_t n_items,
                                               const int64_t* __restrict__ pair_off,
                                               int32_t* __restrict__ owner) {
  const int64_t w = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (w >= n_items) return;
  const int64_t e = pair_off[w + 1];
  for (int64_t p = pair_off[w]; p < e; ++p) owner[p] = int32_t(w);
}

// Offset of (component d, axis e) by selects on d (a variable index into the
// kernel argument would copy it to scratch).
__device__ __forceinline__ int lattice_offset(const LatDesc& ld, int d, int e) {
  return d == 0 ? ld.off[e] : (d == 1 ? ld.off[3 + e] : ld.off[6 + e]);
}

// A candidate pair's item and its cell's place k[] in the item's range (no
// axis longer than kOctantCells: quotients below 216 by float reciprocals).
struct PairPlace {
  int d;
  int64_t t;
  CellRange r;
  int k[3];
};

__device__ __forceinline__ void pair_item(int64_t p, int64_t n_t, const int32_t* owner,
                                          const CellRange* rng, PairPlace& o) {
  const int64_t tc = owner[p];
  o.d = (tc >= n_t) + (tc >= 2 * n_t);
  o.t = tc - int64_t(o.d) * n_t;
  o.r = rng[tc];
}

__device__ __forceinline__ int small_div(int q, int n) {
  return int((float(q) + 0.5f) * __builtin_amdgcn_rcpf(float(n)));
}

// Octant terms of a candidate pair, 0 if the cell surely misses the tet: a
// barycentric coordinate is negative on all of the cell's part of the tet's
// box.  The coordinates are affine with gradients good to about κ² ulps, κ =
// box volume / |det|, which is at most kOctantRange³ here (the determinant
// of the gradients times the box's sides, and each of them sums to at most
// kOctantRange), so the test asks for a margin of 1e-8 (far above κ² ulps;
// what it lets through is integrated and dropped by its volume).
__device__ __forceinline__ int candidate_terms(const PairPlace& o, const double* tetrec,
                                               const double* tetgrad, const double* lat,
                                               const LatDesc& ld, int& cuts) {
  double rec[kTetRec], g[12];
  load_row<kTetRec>(tetrec + o.t * kTetRec, rec);
  load_row<12>(tetgrad + o.t * 12, g);
  int terms = 1;
  cuts = 0;
  double top[4] = {1.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int e = 0; e < 3; ++e) {
    const double* L = lat + lattice_offset(ld, o.d, e) + o.r.lo[e] + o.k[e];
    const double mn = fmin(fmin(rec[e], rec[3 + e]), fmin(rec[6 + e], rec[9 + e]));
    const double mx = fmax(fmax(rec[e], rec[3 + e]), fmax(rec[6 + e], rec[9 + e]));
    const double a = fmax(mn, L[0]) - rec[e];
    const double b = fmin(mx, L[1]) - rec[e];
#pragma unroll
    for (int i = 0; i < 4; ++i) top[i] += fmax(g[3 * i + e] * a, g[3 * i + e] * b);
    terms <<= axis_two(o.k[e], o.r.n[e]) ? 1 : 0;
    cuts += (o.k[e] > 0) + (o.k[e] < o.r.n[e] - 1);
  }
  const double least = fmin(fmin(top[0], top[1]), fmin(top[2], top[3]));
  return least < -1e-8 ? 0 : terms;
}

// A queued octant term: its pair relative to the block's first (11 bits),
// the cell's place (3 bits an axis), the term's index among the pair's and
// their number less one.
constexpr int kPieceRange = 2048;  // most candidate pairs of one block
__device__ __forceinline__ uint32_t term_pack(int rel, const int k[3], int j, int n) {
  return uint32_t(rel) | uint32_t(k[0] | (k[1] << 3) | (k[2] << 6)) << 11 | uint32_t(j) << 20 |
         uint32_t(n - 1) << 23;
}

__device__ __forceinline__ int64_t queued_pair(uint32_t e, int64_t b0, int64_t n_t,
                                               const int32_t* owner, const CellRange* rng,
                                               PairPlace& o) {
  const int64_t p = b0 + int64_t(e & 0x7ffu);
  pair_item(p, n_t, owner, rng, o);
  o.k[0] = int((e >> 11) & 7u);
  o.k[1] = int((e >> 14) & 7u);
  o.k[2] = int((e >> 17) & 7u);
  return p;
}

// Writes the 16 values of every lane's row of the stage to memory, 128
// bytes of eight rows at a time (one lane, one row: each 16-byte store is
// a request of its own to the L2).  rel[s]: where row 8 s + lane / 8 goes
// (times `stride` from `out`, this lane's place in it), or negative.  No
// load may be pending here: waiting for one waits for the stores before it.
constexpr int kStageRow = 17;
__device__ __forceinline__ void store_stage(const double* stage, const int rel[8], double* out,
                                            int stride) {
  const int lane = threadIdx.x;
  const double* src = stage + (lane >> 3) * kStageRow + 2 * (lane & 7);
  wave_lds_sync();
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    const double v[2] = {src[8 * s * kStageRow], src[8 * s * kStageRow + 1]};
    if (rel[s] >= 0) store_row_nt<2>(out + int64_t(rel[s]) * stride, v);
  }
  wave_lds_sync();
}

// (II)-(III) of an FP64 coupling's items that are not marked in `clipped`
// (null: none is).  One wave per `range` candidate pairs: 64 candidates at a
// time are tested against the tet's faces, the octant terms of those left
// are queued, and whole batches of 64 terms are integrated, one lane each
// (moments.hpp), so the lanes stay filled although a fifth of the candidates
// is empty.  A pair's terms are consecutive; its
// first lane adds them in order and turns the 32 moments into the values
// ∫ λ_i N_j, so a pair's results depend on the pair alone.
//
// Measured on 84.4M pairs (4.5M tets on 512 x 256 x 256): 17.7 ms, where the
// pair order, the clip and the integration of its sub-tetrahedra take 36 (a
// step 43.4 ms for 61.6).  Bound: 5.1e9 VALU instructions (702 a face, 576 of
// them FP64; 8.2 ms of issue) and 32.5 GB written and 8.3 read (8 ms at a
// copy's rate), neither hidden behind the other at two waves a SIMD (207
// registers).  Three waves (168 registers) spill and take 0.5 ms more; stores
// of 16 bytes a lane to lines of their own 0.4 ms.
__global__ __launch_bounds__(kWave, 2) void k_pieces(
    int64_t plane_pairs, int64_t p_begin, int64_t p_end, int range, int64_t n_t,
    const uint8_t* __restrict__ clipped, const int32_t* __restrict__ owner,
    const int64_t* __restrict__ pair_off, const CellRange* __restrict__ rng,
    const double* __restrict__ tetrec, const double* __restrict__ tetgrad,
    const double* __restrict__ tetvol, const double* __restrict__ lat, LatDesc ld,
    double drop_rel, uint8_t* __restrict__ keep, double* __restrict__ pval,
    double* __restrict__ pmom, int dual, unsigned long long* counters) {
  constexpr int kQueue = 9 * kWave;
  // rows 0..11: the tet in octant coordinates; 12..17: the octant's signs
  // and shifts (here while the faces need the registers); then the stage
  __shared__ double lds[18 * kWave];
  __shared__ uint32_t queue[kQueue];
  static_assert(kWave * kStageRow <= 18 * kWave, "stage");
  const int lane = threadIdx.x;
  const int64_t b0 = p_begin + int64_t(blockIdx.x) * range;
  const int64_t b1 = min<int64_t>(b0 + range, p_end);
  int filled = 0;
  uint32_t nk = 0, nd = 0, np = 0;
  int64_t next = b0;
  while (next < b1 || filled > 0) {
    if (filled < kWave && next < b1) {
      const int64_t p = next + lane;
      next += kWave;
      int terms = 0;
      PairPlace o;
      if (p < b1) {
        pair_item(p, n_t, owner, rng, o);
        const int64_t tc = int64_t(o.d) * n_t + o.t;
        if (!clipped || !clipped[tc]) {
          const int q = int(p - pair_off[tc]);
          const int qy = small_div(q, o.r.n[0]), qz = small_div(qy, o.r.n[1]);
          o.k[0] = q - qy * o.r.n[0];
          o.k[1] = qy - qz * o.r.n[1];
          o.k[2] = qz;
          int cuts;
          terms = candidate_terms(o, tetrec, tetgrad, lat, ld, cuts);
          if (terms == 0) keep[p] = 0;
          else np += unsigned(cuts);
        }
      }
      int incl = terms;
      for (int o2 = 1; o2 < kWave; o2 <<= 1) {
        const int y = __shfl_up(incl, o2, kWave);
        if (lane >= o2) incl += y;
      }
      for (int j = 0; j < terms; ++j)
        queue[filled + incl - terms + j] = term_pack(int(p - b0), o.k, j, terms);
      filled += __shfl(incl, kWave - 1, kWave);
      wave_lds_sync();
      continue;
    }
    // up to 64 terms, whole pairs only
    int take = min(filled, kWave);
    if (filled > kWave) {
      const uint32_t e = queue[kWave - 1];
      const int j = int((e >> 20) & 7u), n = int(e >> 23) + 1;
      if (j + 1 < n) take = kWave - 1 - j;
    }
    // lanes past the batch repeat its first term: every lane runs the same
    // code on a term of its own, and what it may write is masked
    const bool active = lane < take;
    const uint32_t e = queue[active ? lane : 0];
    const int term = int((e >> 20) & 7u), terms = int(e >> 23) + 1;
    double M[kMom];
#pragma unroll
    for (int k = 0; k < kMom; ++k) M[k] = 0.0;
    double sign = 6.0;  // of the term, times 6
    {
      PairPlace o;
      queued_pair(e, b0, n_t, owner, rng, o);
      double rec[kTetRec];
      load_row<kTetRec>(tetrec + o.t * kTetRec, rec);
      int bit = 0;
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        const double* L = lat + lattice_offset(ld, o.d, a) + o.r.lo[a] + o.k[a];
        const double lo = L[0], hi = L[1];
        const double mn = fmin(fmin(rec[a], rec[3 + a]), fmin(rec[6 + a], rec[9 + a]));
        const bool two = axis_two(o.k[a], o.r.n[a]);
        const AxisOctant x =
            axis_octant(o.k[a], o.r.n[a], lo, hi, mn, two && ((term >> bit) & 1));
        bit += two ? 1 : 0;
        const double sih = x.sg * recip(hi - lo);
#pragma unroll
        for (int v = 0; v < 4; ++v) lds[(3 * v + a) * kWave + lane] = sih * (rec[3 * v + a] - x.c);
        lds[(12 + a) * kWave + lane] = x.sg;
        lds[(15 + a) * kWave + lane] = sih * (x.c - lo) - 0.5 * x.sg;
        sign = x.minus ? -sign : sign;
      }
    }
    wave_lds_sync();
#pragma unroll 1
    for (int f = 0; f < 4; ++f) {
      // faces (1,2,3), (0,3,2), (0,1,3), (0,2,1)
      const int ia = f == 0 ? 1 : 0, ib = f == 1 ? 3 : (f == 2 ? 1 : 2),
                ic = f == 1 ? 2 : (f == 3 ? 1 : 3);
      add_face([&](int v, int a) { return lds[(3 * v + a) * kWave + lane]; }, ia, ib, ic, M);
    }
    wave_lds_sync();
    {
      const double sg[3] = {lds[12 * kWave + lane], lds[13 * kWave + lane], lds[14 * kWave + lane]};
      const double sh[3] = {lds[15 * kWave + lane], lds[16 * kWave + lane], lds[17 * kWave + lane]};
      // M[0] > 0 for a positively oriented tet in octant coordinates; the
      // stored moments are −6 ∫ s^α
      centre_moments(M, sg, sh, M[0] > 0.0 ? -sign : sign);
    }
    // a pair's terms are consecutive: its first lane adds the others' in order
    const int most = wave_max(active ? terms : 1);
#pragma unroll 1
    for (int j = 1; j < most; ++j) {
      const double on = term == 0 && j < terms ? 1.0 : 0.0;
#pragma unroll
      for (int k = 0; k < kMom; ++k) M[k] = fma(on, __shfl_down(M[k], j, kWave), M[k]);
    }
    // the pair again (read again: kept through the faces it would cost
    // registers, and two waves a SIMD leave none)
    uint32_t e2 = e;
    asm volatile("" : "+v"(e2));
    PairPlace o;
    const int64_t p = queued_pair(e2, b0, n_t, owner, rng, o);
    double lo[3], h[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const double* L = lat + lattice_offset(ld, o.d, a) + o.r.lo[a] + o.k[a];
      lo[a] = L[0];
      h[a] = L[1] - L[0];
    }
    const double cv = h[0] * h[1] * h[2] * (-1.0 / 6.0);
    // λ_i in centred coordinates (dual: ψ_i = 5 λ_i − Σ_k λ_k = 5 λ_i − 1),
    // times the cell's volume
    double lc[4], lg[4][3];
    {
      double g[12], v0[4];
      load_row<12>(tetgrad + o.t * 12, g);
      load_row<4>(tetrec + o.t * kTetRec, v0);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        lc[i] = i == 0 ? 1.0 : 0.0;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          lc[i] += g[3 * i + a] * ((lo[a] - v0[a]) + 0.5 * h[a]);
          lg[i][a] = g[3 * i + a] * h[a] * (dual ? 5.0 * cv : cv);
        }
        lc[i] = (dual ? 5.0 * lc[i] - 1.0 : lc[i]) * cv;
      }
    }
    const double vol = M[0] * cv;
    const bool lead = active && term == 0;
    const double tv = tetvol[o.t];
    const bool kp = lead && vol > drop_rel * tv;
    if (lead) keep[p] = kp ? 1 : 0;
    nk += kp ? 1 : 0;
    // (below a tenth of that a volume may be the roundings of an empty cell)
    nd += lead && !kp && vol > 0.1 * drop_rel * tv ? 1 : 0;
    const uint64_t rows = ballot64(kp);
    double* stage = lds;
    int rel[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const int row = 8 * s + (lane >> 3);
      rel[s] = (rows >> row) & 1ull ? int(queue[row] & 0x7ffu) : -1;
    }
    // (opaque, so that the addresses below are made here and not kept, and
    // spilled, through the loop)
    int q = lane & 7;
    asm volatile("" : "+v"(q));
#pragma unroll
    for (int half = 0; half < 2; ++half) {
#pragma unroll
      for (int k = 0; k < 16; ++k) stage[lane * kStageRow + k] = M[16 * half + k];
      store_stage(stage, rel, pmom + b0 * kMomPad + 16 * half + 2 * q, kMomPad);
    }
#pragma unroll
    for (int k = 0; k < kMom; ++k) finish(M[k]);
    double F[4][8];
    mom_hats<double>(M, F);
#pragma unroll
    for (int half = 0; half < 2; ++half) {
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int v = 2 * half + i;
#pragma unroll
        for (int j = 0; j < 8; ++j)
          stage[lane * kStageRow + 8 * i + j] =
              lc[v] * F[0][j] + lg[v][0] * F[1][j] + lg[v][1] * F[2][j] + lg[v][2] * F[3][j];
      }
      store_stage(stage, rel,
                  pval + ((2 * half + (q >> 2)) * plane_pairs + (b0 - p_begin)) * 8 + 2 * (q & 3), 8);
#pragma unroll
      for (int f = 0; f < 4; ++f)
#pragma unroll
        for (int j = 0; j < 8; ++j) finish(F[f][j]);
    }
    // the rest of the queue moves to its front
    const int rest = filled - take;
    for (int k = 0; k < rest; k += kWave) {
      const uint32_t x = k + lane < rest ? queue[take + k + lane] : 0;
      wave_lds_sync();
      if (k + lane < rest) queue[k + lane] = x;
      wave_lds_sync();
    }
    filled = rest;
  }
  const uint32_t sk = wave_sum(nk), sd = wave_sum(nd), sp = wave_sum(np);
  if (lane == 0) {
    if (sk) atomicAdd(&counters[kCntPieces], (unsigned long long)sk);
    if (sd) atomicAdd(&counters[kCntDropped], (unsigned long long)sd);
    if (sp) atomicAdd(&counters[kCntPlanes], (unsigned long long)sp);
  }
}

// ---------------------------------------------------------------------------
// row gather: one wavefront per (vertex, component)
// ---------------------------------------------------------------------------

// Node box of row (vertex i, component d): the union of the cell ranges of
// the incident tets, as lo[3] and extent[3] (nodes); its size bounds the row.
// chunks = first | last << 8: the pair chunks holding the row's pairs (0xff:
// the row has none).
struct RowBox {
  int32_t lo[3];
  int32_t n[3];
  int32_t chunks;
};

// The (component, tet) ranges of the pair chunks: chunk k holds the items
// [at[k], at[k + 1]).
struct ChunkBounds {
  int64_t at[kMaxChunks + 1];
  int n;
};

__device__ __forceinline__ int chunk_of(const ChunkBounds& cb, int64_t tc) {
  int k = 0;
  for (int j = 1; j < cb.n; ++j) k += tc >= cb.at[j] ? 1 : 0;
  return k;
}

// kBoxG lanes per row: each takes every kBoxG-th incident tet, then the
// group reduces its bounds with lane shuffles.  Also the row's first and
// last pair chunk; a row without pairs gets rownnz = 0 here (no chunk
// gathers it).
constexpr int kBoxG = 16;

__global__ __launch_bounds__(256) void k_row_box(int64_t n_v, int64_t n_t, ChunkBounds cb,
                                                 const int64_t* __restrict__ vt_ptr,
                                                 const int32_t* __restrict__ vt_tet,
                                                 const CellRange* __restrict__ rng,
                                                 RowBox* __restrict__ box,
                                                 int64_t* __restrict__ cap,
                                                 int64_t* __restrict__ rownnz) {
  const int64_t w = (int64_t(blockIdx.x) * blockDim.x + threadIdx.x) / kBoxG;
  const int g = threadIdx.x % kBoxG;
  const bool active = w < 3 * n_v;
  int bmin[3] = {INT_MAX, INT_MAX, INT_MAX}, bmax[3] = {INT_MIN, INT_MIN, INT_MIN};
  int cmin = INT_MAX, cmax = INT_MIN;
  if (active) {
    const int d = int(w / n_v);
    const int64_t i = w - int64_t(d) * n_v;
    for (int64_t k = vt_ptr[i] + g; k < vt_ptr[i + 1]; k += kBoxG) {
      const int64_t tc = int64_t(d) * n_t + vt_tet[k];
      const CellRange r = rng[tc];
      if (int64_t(r.n[0]) * r.n[1] * r.n[2] == 0) continue;
      for (int e = 0; e < 3; ++e) {
        bmin[e] = min(bmin[e], r.lo[e]);
        bmax[e] = max(bmax[e], r.lo[e] + r.n[e]);
      }
      const int ch = chunk_of(cb, tc);
      cmin = min(cmin, ch);
      cmax = max(cmax, ch);
    }
  }
#pragma unroll
  for (int o = kBoxG / 2; o > 0; o >>= 1) {
    for (int e = 0; e < 3; ++e) {
      bmin[e] = min(bmin[e], __shfl_xor(bmin[e], o, kWave));
      bmax[e] = max(bmax[e], __shfl_xor(bmax[e], o, kWave));
    }
    cmin = min(cmin, __shfl_xor(cmin, o, kWave));
    cmax = max(cmax, __shfl_xor(cmax, o, kWave));
  }
  if (!active || g != 0) return;
  RowBox b;
  int64_t sz = 1;
  for (int e = 0; e < 3; ++e) {
    b.lo[e] = bmin[e] <= bmax[e] ? bmin[e] : 0;
    b.n[e] = bmin[e] <= bmax[e] ? bmax[e] - bmin[e] + 1 : 0;
    sz *= b.n[e];
  }
  b.chunks = cmin <= cmax ? (cmin | (cmax << 8)) : (0xff | (0xff << 8));
  box[w] = b;
  cap[w] = sz;
  if (cmin > cmax) rownnz[w] = 0;
}

// Spill capacity of each row: its box size if its pairs lie in more than one
// chunk (the partial sums wait between the chunks), else 0 (in place).
__global__ void k_row_spill_cap(int64_t n_rows, const RowBox* __restrict__ box,
                                int64_t* __restrict__ cap) {
  const int64_t w = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (w >= n_rows) return;
  const int ch = box[w].chunks;
  if ((ch & 0xff) == 0xff || (ch & 0xff) == (ch >> 8)) cap[w] = 0;
}

// Exact floor(q / n) for q < 2^16 and 1 <= n < 2^16 as a multiply-high by
// m = ceil(2^32 / n): with m n = 2^32 + e, 0 <= e < n, the error term q e / 2^32
// stays below 1.  n = 1 (m = 2^32) is coded as m = 0.
__device__ __forceinline__ uint32_t magic_div(uint32_t n) {
  return n <= 1u ? 0u : 0xFFFFFFFFu / n + 1u;
}
__device__ __forceinline__ uint32_t div_magic(uint32_t q, uint32_t m) {
  return m ? __umulhi(q, m) : q;
}

// Maximum of x over the row groups of a wavefront (lanes hl, hl + H, ...),
// for loop bounds common to all of them.
template <int H>
__device__ __forceinline__ int64_t rows_max(int64_t x) {
  for (int o = H; o < kWave; o <<= 1) x = max(x, __shfl_xor(x, o, kWave));
  return x;
}

// Gather the pieces of the incident tets into the row's node box, kept in
// LDS 640 / RPW nodes at a time.  Each wavefront serves RPW rows, H = 64 / RPW
// lanes each, so the memory latency of one row's steps overlaps the others'.
// The row's incident tets are taken in ascending order; for each, the lanes
// take its pairs (cells), H at a time, each lane loading its pair's 8 values
// of this vertex at once, and the values are added eight cells after eight
// cells, corner by corner: for one corner the cells of one tet are distinct,
// so are the nodes they add to, and every node sums its contributions in
// the order (tet, eight cells, corner) whatever the timing and RPW
// (deterministic, no value atomics outside LDS).  Per batch of H incident
// tets, each tet's offsets are set up once in LDS.  Touched nodes are written
// column-sorted at tmp_off[w].
//
// One launch per pair chunk ch (items [tc_lo, tc_hi), pairs from p_base,
// values in pval planes of plane_pairs pairs), over the rows w_begin ..
// w_begin + n_rows - 1: a row takes the incident tets of the chunk.  A row
// whose pairs lie in several chunks starts from zero in its first chunk,
// keeps its node sums (double) and touched flags in its spill space between
// the chunks, and is written in its last; the chunks come in tet order, so
// every node still sums in that order.
//
// Bound: with few or wide rows the chain of a row's steps (a load and eight
// LDS adds each, and again for every 640 / RPW nodes of its box); with many
// rows the LDS adds.  rows_per_wave chooses.
template <typename T, int RPW>
__global__ __launch_bounds__(256) void k_rows(
    int64_t n_v, int64_t n_t, int ch, int64_t tc_lo, int64_t tc_hi, int64_t p_base,
    int64_t plane_pairs, int64_t w_begin, int64_t n_rows, const int64_t* __restrict__ vt_ptr,
    const int32_t* __restrict__ vt_tet, const int32_t* __restrict__ tets,
    const CellRange* __restrict__ rng, const int64_t* __restrict__ pair_off,
    const uint8_t* __restrict__ keep, const T* __restrict__ pval, LatDesc ld,
    const RowBox* __restrict__ box, const int64_t* __restrict__ tmp_off,
    int32_t* __restrict__ tmp_col, T* __restrict__ tmp_val, int64_t* __restrict__ rownnz,
    const int64_t* __restrict__ spill_off, double* __restrict__ spill_acc,
    uint8_t* __restrict__ spill_flg) {
  constexpr int H = kWave / RPW;   // lanes per row
  constexpr int RB = 4 * RPW;      // rows per block
  constexpr int NODES = kRowNodes / RPW;
  __shared__ double s_acc[RB][NODES];  // summed in double in both precisions
  __shared__ uint8_t s_flag[RB][NODES];
  __shared__ int4 s_m0[RB][H], s_m1[RB][H];
  const int lane = lane_id();
  const int h = lane / H, hl = lane % H;
  const int slot = RPW * (threadIdx.x / kWave) + h;  // this row's LDS slot
  const int64_t wl =
      RPW * ((int64_t(blockIdx.x) * blockDim.x + threadIdx.x) / kWave) + h;
  const int64_t w = w_begin + wl;
  double* acc = s_acc[slot];
  uint8_t* flg = s_flag[slot];
  int4* M0 = s_m0[slot];
  int4* M1 = s_m1[slot];
  RowBox b{};
  if (wl < n_rows) b = box[w];
  // rows of this chunk: first <= ch <= last
  const int cf = b.chunks & 0xff, cl = (b.chunks >> 8) & 0xff;
  const bool live = wl < n_rows && cf != 0xff && cf <= ch && ch <= cl;
  const bool first = cf == ch, last = cl == ch;
  const int64_t so = (live && !(first && last)) ? spill_off[w] : 0;
  const int d = live ? int(w / n_v) : 0;
  const int64_t i = live ? w - int64_t(d) * n_v : 0;
  const int bn0 = b.n[0], bn1 = b.n[1];
  const int64_t total = live ? int64_t(bn0) * bn1 * b.n[2] : 0;
  int64_t outpos = live ? tmp_off[w] : 0;
  const int64_t start = outpos;
  const int64_t NX = ld.n[3 * d + 0], NY = ld.n[3 * d + 1];
  const int64_t beg = live ? vt_ptr[i] : 0, end = live ? vt_ptr[i + 1] : 0;
  // box-linear offsets of the 8 corners of a cell
  int coff[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) coff[j] = (j & 1) + bn0 * (((j >> 1) & 1) + bn1 * (j >> 2));
  const int64_t vplane = plane_pairs * 8;
  // loop bounds common to the row groups of the wave (each masks its own work)
  const int64_t total_max = rows_max<H>(total);
  const int64_t ntet = end - beg;
  const int64_t ntet_max = rows_max<H>(ntet);
  for (int64_t c0 = 0; c0 < total_max; c0 += NODES) {
    const int span = int(max<int64_t>(0, min<int64_t>(NODES, total - c0)));
    for (int k = hl; k < span; k += H) {
      acc[k] = first ? 0.0 : spill_acc[so + c0 + k];
      flg[k] = first ? 0 : spill_flg[so + c0 + k];
    }
    for (int64_t kb0 = 0; kb0 < ntet_max; kb0 += H) {
      const int nk = int(max<int64_t>(0, min<int64_t>(H, ntet - kb0)));
      wave_lds_sync();
      if (hl < nk) {
        const int64_t t = vt_tet[beg + kb0 + hl];
        const int64_t tc = int64_t(d) * n_t + t;
        const CellRange r = rng[tc];
        const int4 tv = *reinterpret_cast<const int4*>(tets + 4 * t);
        const int li =
            (tv.y == int32_t(i)) ? 1 : (tv.z == int32_t(i)) ? 2 : (tv.w == int32_t(i)) ? 3 : 0;
        const int64_t kbase = pair_off[tc];  // pair of cell 0
        // box-linear offset of the tet's first cell in this pass
        const int off0 = int(int64_t(r.lo[0] - b.lo[0]) +
                             int64_t(bn0) * ((r.lo[1] - b.lo[1]) +
                                             int64_t(bn1) * (r.lo[2] - b.lo[2])) -
                             c0);
        // tets of other chunks add nothing here
        const int cnt = (tc >= tc_lo && tc < tc_hi) ? r.n[0] * r.n[1] * r.n[2] : 0;
        M0[hl] = make_int4(int(kbase & 0xffffffffll), int(kbase >> 32), li, cnt);
        M1[hl] = make_int4(r.n[0] | (r.n[1] << 16), off0,
                           int(magic_div(uint32_t(max(r.n[0], 1)))),
                           int(magic_div(uint32_t(max(r.n[1], 1)))));
      }
      wave_lds_sync();
      const int nk_max = int(rows_max<H>(int64_t(nk)));
      for (int kk = 0; kk < nk_max; ++kk) {
        int4 m0 = make_int4(0, 0, 0, 0), m1 = make_int4(0, 0, 0, 0);
        if (kk < nk) {
          m0 = M0[kk];
          m1 = M1[kk];
        }
        const int cnt = m0.w;
        const int cnt_max = int(rows_max<H>(int64_t(cnt)));
        const int64_t kbase = int64_t((unsigned long long)(unsigned)m0.x |
                                      ((unsigned long long)(unsigned)m0.y << 32));
        const uint32_t n0 = uint32_t(m1.x) & 0xffffu, n1 = uint32_t(m1.x) >> 16;
        for (int q0 = 0; q0 < cnt_max; q0 += H) {
          const int q = q0 + hl;
          bool add = false;
          int base = 0;
          T v[8];
          if (q < cnt) {
            const uint32_t qy = div_magic(uint32_t(q), uint32_t(m1.z));
            const int ix = int(uint32_t(q) - qy * n0);
            const uint32_t iz = div_magic(qy, uint32_t(m1.w));
            const int iy = int(qy - iz * n1);
            base = m1.y + ix + bn0 * (iy + bn1 * int(iz));
            const int64_t ko = kbase + q;
            add = keep[ko] != 0;
            load_row<8>(pval + int64_t(m0.z) * vplane + (ko - p_base) * 8, v);
          }
          // eight cells after eight cells, corner by corner: the cells of one
          // tet are distinct, so one corner's adds go to distinct nodes
          for (int g = 0; g < H / 8 && q0 + 8 * g < cnt_max; ++g)
            if (H == 8 || hl / 8 == g) {
#pragma unroll
              for (int j = 0; j < 8; ++j) {
                const int lin = base + coff[j];
                if (add && lin >= 0 && lin < span) {
                  __hip_atomic_fetch_add(&acc[lin], double(v[j]), __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_WAVEFRONT);
                  flg[lin] = 1;
                }
              }
            }
        }
      }
    }
    wave_lds_sync();
    if (!last)
      for (int k = hl; k < span; k += H) {
        spill_acc[so + c0 + k] = acc[k];
        spill_flg[so + c0 + k] = flg[k];
      }
    const int span_max = int(rows_max<H>(int64_t(span)));
    for (int k0 = 0; k0 < span_max; k0 += H) {
      const int k = k0 + hl;
      const bool tch = last && k < span && flg[k] != 0;
      const uint64_t m = (ballot64(tch) >> (H * h)) & (~uint64_t(0) >> (kWave - H));
      if (tch) {
        // the box lies inside the lattice, whose node count fits int32
        const uint32_t lin = uint32_t(c0 + k);
        const uint32_t r = lin / uint32_t(bn0);
        const uint32_t zq = r / uint32_t(bn1);
        const int64_t gx = b.lo[0] + int64_t(lin - r * uint32_t(bn0));
        const int64_t gy = b.lo[1] + int64_t(r - zq * uint32_t(bn1));
        const int64_t gz = b.lo[2] + int64_t(zq);
        const int64_t pos = outpos + popc64(m & ((uint64_t(1) << hl) - 1));
        tmp_col[pos] = int32_t(gx + NX * (gy + NY * gz));
        tmp_val[pos] = T(acc[k]);
      }
      outpos += popc64(m);
    }
    wave_lds_sync();
  }
  if (live && last && hl == 0) rownnz[w] = outpos - start;
}

// Rows a wave of k_rows serves.  The LDS of a block lets 20 waves live on a
// CU, about 5,000 on the card: while the rows are few, or a tet's cells more
// than a group's lanes, more lanes for each row shorten its chain of steps.
// Microseconds with 8 / 4 / 2 / 1 rows a wave, by rows and cells per
// (component, tet):
//      189, 26:  248 / 126 /  68 /  61       3,240,  9:   99 /  51 /  46 /   43
//    5,733, 19:  208 / 118 /  63 /  87       5,586, 38:  619 / 304 / 183 /  135
//    8,064,  9:  108 /  55 /  52 /  75      15,900, 36:  760 / 350 / 266 /  288
//   16,500, 16:  169 /  88 / 125 / 180      21,417,  5:   48 /  57 /  72 /  121
//   28,944, 10:  243 / 172 / 172 / 249      56,025,  8:  144 / 155 / 218 /  359
//  112,632, 10:  440 / 368 / 523 / 861     242,208, 14: 1216 / 896 / 1264 / 2129
//  2,497,551, 6: 5.30 / 6.85 / 10.6 / 17.4 ms
int rows_per_wave(int64_t n_rows, int64_t n_pairs, int64_t n_items) {
  const bool wide = n_pairs > 32 * n_items;
  if (n_rows <= 3500 || (wide && n_rows <= 6000)) return 1;
  if (n_rows <= 10000 || (wide && n_rows <= 20000)) return 2;
  return n_rows <= 20000 || n_pairs > 9 * n_items ? 4 : 8;
}

// Copy each row from the box-capacity scratch into the CSR arrays.
constexpr int kCompactLanes = 16;
template <typename T>
__global__ __launch_bounds__(256) void k_rows_compact(
    int64_t n_v, const int64_t* __restrict__ tmp_off, const int32_t* __restrict__ tmp_col,
    const T* __restrict__ tmp_val, const int64_t* __restrict__ rp0,
    const int64_t* __restrict__ rp1, const int64_t* __restrict__ rp2, int32_t* __restrict__ c0,
    int32_t* __restrict__ c1, int32_t* __restrict__ c2, T* __restrict__ v0, T* __restrict__ v1,
    T* __restrict__ v2) {
  // kCompactLanes lanes per row
  const int64_t w = (int64_t(blockIdx.x) * blockDim.x + threadIdx.x) / kCompactLanes;
  const int lane = threadIdx.x % kCompactLanes;
  if (w >= 3 * n_v) return;
  const int d = int(w / n_v);
  const int64_t i = w - int64_t(d) * n_v;
  const int64_t* rp = d == 0 ? rp0 : (d == 1 ? rp1 : rp2);
  int32_t* col = d == 0 ? c0 : (d == 1 ? c1 : c2);
  T* val = d == 0 ? v0 : (d == 1 ? v1 : v2);
  const int64_t src = tmp_off[w], dst = rp[i], n = rp[i + 1] - rp[i];
  for (int64_t k = lane; k < n; k += kCompactLanes) {
    col[dst + k] = tmp_col[src + k];
    val[dst + k] = tmp_val[src + k];
  }
}

// ---------------------------------------------------------------------------
// masses
// ---------------------------------------------------------------------------

template <typename T>
__global__ void k_lumped(int64_t n_v, const int64_t* __restrict__ vt_ptr,
                         const int32_t* __restrict__ vt_tet, const double* __restrict__ tetvol,
                         double* __restrict__ m, T* __restrict__ minv) {
  const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= n_v) return;
  double s = 0.0;
  for (int64_t k = vt_ptr[i]; k < vt_ptr[i + 1]; ++k) s += tetvol[vt_tet[k]];
  s *= 0.25;
  m[i] = s;
  minv[i] = (s > 0.0) ? T(1.0 / s) : T(0);
}

// Consistent mass rows M_il = Σ_{T ∋ i, l} |T|(1 + δ_il)/20, kMassLanes
// lanes per vertex (rows hold ~15 columns): lane k holds column k of the
// row, and the incident tets are broadcast one at a time within the lane
// group (sum order = incident-tet order).
constexpr int kMassLanes = 16;
__global__ __launch_bounds__(256) void k_mass_values(
    int64_t n_v, const int64_t* __restrict__ vt_ptr, const int32_t* __restrict__ vt_tet,
    const int32_t* __restrict__ tets, const double* __restrict__ tetvol,
    const int64_t* __restrict__ rowptr, const int32_t* __restrict__ col,
    double* __restrict__ val, float* __restrict__ val32, double* __restrict__ dinv) {
  constexpr int H = kMassLanes;
  const int64_t i = (int64_t(blockIdx.x) * blockDim.x + threadIdx.x) / H;
  const int hl = threadIdx.x % H;
  if (i >= n_v) return;  // whole lane groups leave together
  const int64_t rb = rowptr[i], re = rowptr[i + 1];
  const int64_t tb = vt_ptr[i], te = vt_ptr[i + 1];
  double diag = 0.0;
  for (int64_t c0 = rb; c0 < re; c0 += H) {
    const bool has = c0 + hl < re;
    const int l = has ? col[c0 + hl] : -1;
    double a = 0.0;
    for (int64_t k0 = tb; k0 < te; k0 += H) {
      const int nk = int(min<int64_t>(H, te - k0));
      int4 tv = make_int4(-1, -1, -1, -1);
      double w = 0.0;
      if (hl < nk) {
        const int64_t t = vt_tet[k0 + hl];
        tv = *reinterpret_cast<const int4*>(tets + 4 * t);
        w = tetvol[t] / 20.0;
      }
      for (int k = 0; k < nk; ++k) {
        const int v0 = __shfl(tv.x, k, H), v1 = __shfl(tv.y, k, H), v2 = __shfl(tv.z, k, H),
                  v3 = __shfl(tv.w, k, H);
        const double wk = __shfl(w, k, H);
        if (l == v0 || l == v1 || l == v2 || l == v3) a += (int64_t(l) == i) ? 2.0 * wk : wk;
      }
    }
    if (has) {
      val[c0 + hl] = a;
      if (val32) val32[c0 + hl] = float(a);
      if (int64_t(l) == i) diag = a;
    }
  }
  for (int o = H / 2; o > 0; o >>= 1) diag += __shfl_xor(diag, o, H);
  if (hl == 0) dinv[i] = (diag > 0.0) ? 1.0 / diag : 0.0;
}

inline unsigned blocks_for(int64_t n, int threads) {
  return unsigned(ceil_div(n > 0 ? n : 1, threads));
}

// Blocks of one wave each that the device keeps resident for kernel f
// (grid of a persistent launch).
template <typename F>
int resident_blocks(F f) {
  int dev = 0, cus = 0, per_cu = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, f, kWave, 0) != hipSuccess ||
      cus <= 0 || per_cu <= 0) {
    (void)hipGetLastError();  // a failed query must not read as a launch error
    return 1 << 16;
  }
  return cus * per_cu;
}

}  // namespace

int read_back(ibvt_coupling* c, void* host, const void* dev, size_t bytes, hipStream_t s) {
  (void)c;
  int st = hip_check(hipMemcpyAsync(host, dev, bytes, hipMemcpyDeviceToHost, s), "read back");
  if (st) return st;
  return hip_check(hipStreamSynchronize(s), "stream sync");
}

int flags_status(unsigned f) {
  if (f & kFlagNonFinite) return set_error(IBVT_E_INVALID, "non-finite vertex coordinate");
  if (f & kFlagValence) return set_error(IBVT_E_INVALID, "tet vertex index out of range or repeated");
  if (f & kFlagOutOfGrid)
    return set_error(IBVT_E_OUT_OF_GRID, "a tet's bounding box leaves a velocity lattice's node hull");
  if (f & kFlagCapacity)
    return set_error(IBVT_E_CAPACITY, "clipped piece exceeded the 16-vertex capacity");
  if (f & kFlagTetSpan)
    return set_error(IBVT_E_CAPACITY, "an element spans more than 65535 cells of one lattice");
  return IBVT_OK;
}

int check_flags(ibvt_coupling* c, hipStream_t s) {
  unsigned f = 0;
  int st = read_back(c, &f, c->flags_dev.p, sizeof(unsigned), s);
  if (st) return st;
  return flags_status(f);
}

namespace {
struct CountSrc {
  const int64_t* p[kMaxCounts];
};
__global__ void k_gather_counts(CountSrc src, int n, const unsigned* __restrict__ flags,
                                int64_t* __restrict__ out) {
  const int k = threadIdx.x;
  if (k < n) out[k] = *src.p[k];
  if (k == 0) out[kMaxCounts] = int64_t(*flags);
}
}  // namespace

int read_counts(ibvt_coupling* c, const int64_t* const* srcs, int n, int64_t* out, hipStream_t s) {
  if (n < 0 || n > kMaxCounts) return set_error(IBVT_E_INVALID, "read_counts: too many values");
  int st = host_block(c);
  if (st) return st;
  CountSrc src{};
  for (int k = 0; k < n; ++k) src.p[k] = srcs[k];
  // straight to the host: a copy would be one more launch to wait for
  k_gather_counts<<<1, 64, 0, s>>>(src, n, c->flags_dev.as<unsigned>(), c->host_rb_dev);
  if ((st = hip_check(hipGetLastError(), "count gather launch"))) return st;
  if ((st = hip_check(hipStreamSynchronize(s), "stream sync"))) return st;
  for (int k = 0; k < n; ++k) out[k] = c->host_rb[k];
  c->host_flags = unsigned(c->host_rb[kMaxCounts]);
  return IBVT_OK;
}

namespace {

// (Component, tet) items per pair chunk: 3 · 2^19 (about 10M pairs at the
// three-body workload's density), or IBVT_CHUNK_ITEMS from the environment
// (a positive integer; small values put small meshes through the chunked
// path, as the tests do).  At most kMaxChunks chunks either way.
int64_t chunk_items() {
  if (const char* e = std::getenv("IBVT_CHUNK_ITEMS")) {
    char* end = nullptr;
    const long long v = std::strtoll(e, &end, 10);
    if (end != e && *end == '\0' && v > 0) return int64_t(v);
  }
  return int64_t(3) << 19;
}

// Without stored matrices (IBVT_NO_STORE_B): after the overlap candidates,
// only the solid masses and the per-(component, tet) buffer of the
// matrix-free products (3 n_t x 4 values) are built.
template <typename T>
int finish_matfree(ibvt_coupling* c, hipStream_t s) {
  int st;
  if ((st = ensure(c, c->pval, size_t(3 * c->n_tet + 1) * 4 * sizeof(T)))) return st;
  for (int d = 0; d < 3; ++d) {
    c->B[d].nnz = 0;
    c->Bt[d].nrows = 0;
    c->Bt[d].nnz = 0;
  }
  if ((st = solid_masses(c, s))) return st;
  if ((st = matfree_order(c, s))) return st;
  int64_t zero = 0;
  {
    const int64_t* src[1] = {
        reinterpret_cast<const int64_t*>(c->counters.as<unsigned long long>() + kCntZeroTets)};
    if ((st = read_counts(c, src, 1, &zero, s))) return st;
  }
  if ((st = flags_status(c->host_flags))) return st;
  const int64_t done = c->stats.assemblies + 1;
  c->stats = AsmStats{};
  c->stats.pairs = c->n_pairs;
  c->stats.zero_tets = zero;
  c->stats.assemblies = done;
  c->mom_valid = false;
  return IBVT_OK;
}

template <typename T>
int assemble_typed(ibvt_coupling* c, hipStream_t s) {
  const int64_t n_t = c->n_tet, n_v = c->n_vert;
  int st;
  unsigned* flags = c->flags_dev.as<unsigned>();
  auto* counters = c->counters.as<unsigned long long>();
  if ((st = hip_check(hipMemsetAsync(flags, 0, sizeof(unsigned), s), "memset"))) return st;
  if ((st = hip_check(hipMemsetAsync(counters, 0, kCntSlots * sizeof(unsigned long long), s),
                      "memset")))
    return st;
  // FP64 items are marked for the clip or for the boundary integrals
  uint8_t* to_clip = nullptr;
  if (sizeof(T) == sizeof(double) && !c->matrix_free) {
    if ((st = ensure(c, c->clipped, size_t(3 * n_t + 1)))) return st;
    to_clip = c->clipped.as<uint8_t>();
  }
  // (I) overlap candidates
  {
    ProfScope ps("tet_prep", s);
  k_tet_prep<<<blocks_for(n_t, 256), 256, 0, s>>>(
      n_t, c->X.as<double>(), c->tets.as<int32_t>(), c->lat.as<double>(), c->ld,
      c->tetvol.as<double>(), c->rng.as<CellRange>(), c->cnt.as<int64_t>(), c->tetrec.as<double>(),
      c->tetgrad.as<double>(), to_clip, flags, counters);
  }
  if ((st = hip_check(hipGetLastError(), "prep launch"))) return st;
  if ((st = scan_i64(c, c->cnt.as<int64_t>(), c->pair_off.as<int64_t>(), 3 * n_t, s))) return st;
  // The pairs are clipped and integrated in chunks of consecutive (component,
  // tet) ranges: the piece store holds one chunk's sub-tetrahedra, and a
  // chunk's tet records stay in the caches while its pairs are clipped.
  const int64_t n_tc = 3 * n_t;
  const int nchunk =
      int(std::min<int64_t>(kMaxChunks, std::max<int64_t>(1, n_tc / chunk_items())));
  ChunkBounds cb{};
  cb.n = nchunk;
  for (int k = 0; k <= nchunk; ++k) cb.at[k] = n_tc * k / nchunk;
  const int64_t* tc_at = cb.at;
  // (IV, set-up) each row's node box and its first and last chunk: from the
  // cell ranges alone.  Rows gather their pairs after each chunk's
  // integration, so the per-pair values are held for one chunk only; a row
  // whose pairs lie in several chunks keeps its partial sums in spill space
  // of its box size.
  if (!c->matrix_free) {
    if ((st = ensure(c, c->rowbox, size_t(3 * n_v + 1) * sizeof(RowBox)))) return st;
    if ((st = ensure(c, c->rowcap, size_t(3 * n_v + 1) * sizeof(int64_t)))) return st;
    if ((st = ensure(c, c->rowtmpoff, size_t(3 * n_v + 1) * sizeof(int64_t)))) return st;
    if ((st = ensure(c, c->rowspilloff, size_t(3 * n_v + 1) * sizeof(int64_t)))) return st;
    if ((st = ensure(c, c->rownnz, size_t(3 * n_v + 1) * sizeof(int64_t)))) return st;
    {
      ProfScope ps("rows_box", s);
      k_row_box<<<blocks_for(3 * n_v * kBoxG, 256), 256, 0, s>>>(
          n_v, n_t, cb, c->vt_ptr.as<int64_t>(), c->vt_tet.as<int32_t>(), c->rng.as<CellRange>(),
          c->rowbox.as<RowBox>(), c->rowcap.as<int64_t>(), c->rownnz.as<int64_t>());
    }
    if ((st = hip_check(hipGetLastError(), "row box launch"))) return st;
    if ((st = scan_i64(c, c->rowcap.as<int64_t>(), c->rowtmpoff.as<int64_t>(), 3 * n_v, s)))
      return st;
    if (nchunk > 1) {  // (in one chunk no row is spilled)
      k_row_spill_cap<<<blocks_for(3 * n_v, 256), 256, 0, s>>>(3 * n_v, c->rowbox.as<RowBox>(),
                                                              c->rowcap.as<int64_t>());
      if ((st = hip_check(hipGetLastError(), "row spill launch"))) return st;
      if ((st = scan_i64(c, c->rowcap.as<int64_t>(), c->rowspilloff.as<int64_t>(), 3 * n_v, s)))
        return st;
    }
  }
  // read-back 1: the chunks' first pairs (the last entry is the pair count),
  // the row scratch size, the pairs to clip, the spill size, and status flags
  int64_t pat[kMaxChunks + 4];
  {
    const int64_t* src[kMaxChunks + 4];
    for (int k = 0; k <= nchunk; ++k) src[k] = c->pair_off.as<int64_t>() + tc_at[k];
    int nsrc = nchunk + 1;
    if (!c->matrix_free) {
      src[nsrc++] = c->rowtmpoff.as<int64_t>() + 3 * n_v;
      src[nsrc++] = reinterpret_cast<const int64_t*>(counters + kCntToClip);
      if (nchunk > 1) src[nsrc++] = c->rowspilloff.as<int64_t>() + 3 * n_v;
    }
    if ((st = read_counts(c, src, nsrc, pat, s))) return st;
  }
  if ((st = flags_status(c->host_flags))) return st;
  const int64_t n_pairs = pat[nchunk];
  if (n_pairs >= (int64_t(1) << 31) - 1)
    return set_error(IBVT_E_CAPACITY, "2^31 or more (tet, cell) pairs");
  c->n_pairs = n_pairs;
  if (c->matrix_free) return finish_matfree<T>(c, s);
  const int64_t tmp_total = pat[nchunk + 1], spill_total = nchunk > 1 ? pat[nchunk + 3] : 0;
  // Boundary integrals (k_pieces) or clipping: the items of an FP64 coupling
  // within the limits of moments.hpp take the former (a step of the three-body
  // mesh takes 43.4 ms so and 61.6 clipped, of 47,916 tets 1.51 and 2.12), the
  // others are clipped, each into its own pairs' places.  Mixed couplings are clipped
  // throughout: the boundary integrals would take a three-body step from 40 to
  // 33 ms, and be no further off, but move every float result in its last
  // digits (g_X by 3e-7 to 5e-6 of its norm), and a caller who compares a run
  // with a stored one gets the same bits.
  const int64_t clip_pairs = to_clip ? pat[nchunk + 2] : n_pairs;
  const bool clips = clip_pairs > 0, octants = clip_pairs < n_pairs;
  if (!octants) to_clip = nullptr;  // all items
  int64_t chunk_max = 0;
  for (int k = 0; k < nchunk; ++k) chunk_max = std::max(chunk_max, pat[k + 1] - pat[k]);
  if ((st = ensure(c, c->owner, size_t(n_pairs + 1) * sizeof(int32_t)))) return st;
  if ((st = ensure(c, c->keep, size_t(n_pairs + 1)))) return st;
  // one chunk's values: 4 planes (local vertex) of chunk_max pairs x 8
  if ((st = ensure(c, c->pval, size_t(chunk_max + 1) * 32 * sizeof(T)))) return st;
  if ((st = ensure(c, c->rowtmpcol, size_t(tmp_total + 1) * sizeof(int32_t)))) return st;
  if ((st = ensure(c, c->rowtmpval, size_t(tmp_total + 1) * sizeof(T)))) return st;
  const size_t spill_acc_bytes = (size_t(spill_total + 1) * sizeof(double) + 255) & ~size_t(255);
  if ((st = ensure(c, c->rowspill, spill_acc_bytes + size_t(spill_total + 1)))) return st;
  double* spill_acc = c->rowspill.as<double>();
  uint8_t* spill_flg = c->rowspill.as<uint8_t>() + spill_acc_bytes;
  if ((st = ensure(c, c->pmom, size_t(n_pairs + 1) * kMomPad * sizeof(T)))) return st;
  if ((st = side_stream(c))) return st;
  bool masses_done = false;
  // (IV) the rows of B^d that take pairs of chunk ch: the rows of the
  // components its items belong to (on this stream: beside the next chunk's
  // pieces they slow them by more than they take)
  auto gather_rows = [&](int ch) -> int {
    ProfScope ps("rows_gather", s);
    const int64_t d_lo = tc_at[ch] / n_t, d_hi = (tc_at[ch + 1] - 1) / n_t;
    const int64_t w_begin = d_lo * n_v, n_rows = (d_hi - d_lo + 1) * n_v;
    const int rpw = rows_per_wave(n_rows, n_pairs, n_tc);
    const auto rows = rpw == 1 ? k_rows<T, 1>
                               : (rpw == 2 ? k_rows<T, 2> : (rpw == 4 ? k_rows<T, 4> : k_rows<T, 8>));
    rows<<<blocks_for(ceil_div(n_rows, rpw) * kWave, 256), 256, 0, s>>>(
        n_v, n_t, ch, tc_at[ch], tc_at[ch + 1], pat[ch], chunk_max, w_begin, n_rows,
        c->vt_ptr.as<int64_t>(), c->vt_tet.as<int32_t>(), c->tets.as<int32_t>(),
        c->rng.as<CellRange>(), c->pair_off.as<int64_t>(), c->keep.as<uint8_t>(),
        c->pval.as<T>(), c->ld, c->rowbox.as<RowBox>(), c->rowtmpoff.as<int64_t>(),
        c->rowtmpcol.as<int32_t>(), c->rowtmpval.as<T>(), c->rownnz.as<int64_t>(),
        c->rowspilloff.as<int64_t>(), spill_acc, spill_flg);
    return hip_check(hipGetLastError(), "rows launch");
  };
  // row pointers of B^d; their last entries are the nonzeros
  auto count_rows = [&]() -> int {
    int64_t* out[3];
    for (int d = 0; d < 3; ++d) {
      c->B[d].nrows = n_v;
      out[d] = c->B[d].rowptr.as<int64_t>();
    }
    return scan_i64_rows(c, c->rownnz.as<int64_t>(), out, 3, n_v, s);
  };
  // the solid masses need only the tet volumes: on the second stream beside
  // the first chunk's pieces, joined after them
  auto fork_masses = [&]() -> int {
    if (masses_done) return IBVT_OK;
    masses_done = true;
    return solid_masses(c, c->side.stream);
  };
  int32_t* ohist = nullptr;
  int64_t* ofirst = nullptr;
  const int64_t clip_max = std::min(chunk_max, clip_pairs);  // most pairs a chunk clips
  if (clips) {
    if ((st = ensure(c, c->pinfo, size_t(n_pairs + 1) * sizeof(uint64_t)))) return st;
    // the clip order of one chunk at a time, as pair descriptors
    if ((st = ensure(c, c->order, size_t(clip_max + 1) * sizeof(PairDesc)))) return st;
    // per chunk: the pair descriptors in clip order (k_order_count, scan,
    // k_order_scatter); the scanned key counts give the clip launches their
    // class stretches on the device
    int64_t items_max = 1;
    for (int k = 0; k < nchunk; ++k) items_max = std::max(items_max, tc_at[k + 1] - tc_at[k]);
    const int64_t ob_max = ceil_div(items_max, kOrderItems);
    const size_t hb = (size_t(256 * ob_max) * sizeof(int32_t) + 255) & ~size_t(255);
    if ((st = ensure(c, c->pscan, hb + size_t(256 * ob_max + 1) * sizeof(int64_t)))) return st;
    ohist = c->pscan.as<int32_t>();
    ofirst = reinterpret_cast<int64_t*>(c->pscan.as<char>() + hb);
  }
  if (octants) {
    k_owner<<<blocks_for(n_tc, 256), 256, 0, s>>>(n_tc, c->pair_off.as<int64_t>(),
                                                  c->owner.as<int32_t>());
    if ((st = hip_check(hipGetLastError(), "owner launch"))) return st;
  }
  // Chunks with pairs, in order.  Per chunk: the clip's classes 12 and 16
  // run on the side stream beside class 10 (they fill its tail), and the
  // next chunk's pair order is made on the side stream while this chunk
  // integrates (the order and the sort scratch are free once the clip has
  // read them; the store is reused only after the integration).
  int live[kMaxChunks];
  int n_live = 0;
  for (int ch = 0; ch < nchunk; ++ch)
    if (pat[ch + 1] > pat[ch]) live[n_live++] = ch;
  auto order_chunk = [&](int ch, hipStream_t q) -> int {
    // the next chunk's order runs beside the integration: its span is
    // shared with it
    ProfScope ps(q == s ? "pair_order" : "pair_order_beside_integrate", q);
    const int64_t tc0 = tc_at[ch], items = tc_at[ch + 1] - tc_at[ch];
    const int64_t ob = ceil_div(items, kOrderItems);
    k_order_count<<<unsigned(ob), kOrderItems, 0, q>>>(tc0, items, c->rng.as<CellRange>(), to_clip,
                                                       ohist);
    int r = hip_check(hipGetLastError(), "order count launch");
    if (r) return r;
    if ((r = scan_i32_to_i64(c, ohist, ofirst, 256 * ob, q))) return r;
    k_order_scatter<<<unsigned(ob), kOrderItems, 0, q>>>(
        tc0, items, n_t, c->rng.as<CellRange>(), to_clip, c->pair_off.as<int64_t>(), ofirst,
        c->order.as<PairDesc>(), c->owner.as<int32_t>());
    return hip_check(hipGetLastError(), "order scatter launch");
  };
  int64_t nnzs[3];
  for (int attempt = 0; attempt < 2; ++attempt) {
    if (clips) {
      const int64_t want = std::max<int64_t>(int64_t(3.25 * double(clip_max)) + 1024,
                                             c->pool_needed + c->pool_needed / 32 + 1024);
      if (int64_t(c->pool.cap / (kRecord * sizeof(T))) < want &&
          (st = ensure(c, c->pool, size_t(want) * kRecord * sizeof(T))))
        return st;
      c->pool_cap = int64_t(c->pool.cap / (kRecord * sizeof(T)));
    }
    // again: clear the clip's counters (the zero-tet count of the preparation
    // stays)
    if (attempt > 0) {
      for (int k : {int(kCntPieces), int(kCntDropped), int(kCntSubtets), int(kCntDist),
                    int(kCntCutPts), int(kCntPlanes)})
        if ((st = hip_check(hipMemsetAsync(counters + k, 0, sizeof(unsigned long long), s),
                            "memset")))
          return st;
      if ((st = hip_check(hipMemsetAsync(counters + kCntChunkPool, 0,
                                         kMaxChunks * sizeof(unsigned long long), s),
                          "memset")))
        return st;
    }
    if (clips && n_live > 0 && (st = order_chunk(live[0], s))) return st;
    for (int li = 0; li < n_live; ++li) {
      const int ch = live[li];
      const int64_t p0 = pat[ch], nc = pat[ch + 1] - pat[ch];
      const int64_t* cls_start = ofirst;  // key-major: class k starts at 64 k blocks
      const int64_t ntiles = ceil_div(tc_at[ch + 1] - tc_at[ch], kOrderItems);
      const bool fork = clips || !masses_done;
      if (fork && ((st = hip_check(hipEventRecord(c->side.fork, s), "event")) ||
                   (st = hip_check(hipStreamWaitEvent(c->side.stream, c->side.fork, 0),
                                   "stream wait")) ||
                   (st = fork_masses())))
        return st;
      if (clips) {
        // (II) clip the chunk's pairs, one launch per cut class (fewer vertex
        // slots per lane, more resident waves); each launch reads its
        // class's stretch of the order from the prefix sum of the key counts
        ProfScope ps("clip", s);
        ClipTables tab;
        if ((st = clip_tables(tab))) return st;
        for (int k = 2; k >= 0; --k) {
          hipStream_t ks = k == 0 ? s : c->side.stream;
          const int resident =
              k == 0 ? resident_blocks(k_clip<T, 10>)
                     : (k == 1 ? resident_blocks(k_clip<T, 12>) : resident_blocks(k_clip<T, kMaxV>));
          const int64_t nb = std::min<int64_t>(ceil_div(std::min(nc, clip_pairs), kWave), resident);
#define IBVT_CLIP_ARGS                                                                          \
  tab, cls_start + 64 * k * ntiles, cls_start + 64 * (k + 1) * ntiles, c->order.as<PairDesc>(), \
      c->tetrec.as<double>(), c->lat.as<double>(), c->ld, 1e-14, c->pool.as<T>(), c->pool_cap,  \
      c->pinfo.as<uint64_t>(), counters + kCntChunkPool + ch, flags, counters
          if (k == 0) k_clip<T, 10><<<dim3(unsigned(nb)), kWave, 0, ks>>>(IBVT_CLIP_ARGS);
          else if (k == 1) k_clip<T, 12><<<dim3(unsigned(nb)), kWave, 0, ks>>>(IBVT_CLIP_ARGS);
          else k_clip<T, kMaxV><<<dim3(unsigned(nb)), kWave, 0, ks>>>(IBVT_CLIP_ARGS);
#undef IBVT_CLIP_ARGS
        }
        if ((st = hip_check(hipGetLastError(), "clip launch"))) return st;
      }
      if constexpr (sizeof(T) == sizeof(double)) {
        if (octants) {
          // (II)-(III) the other pairs' pieces from their boundary integrals
          ProfScope ps("pieces", s);
          // candidates per block: about eight rounds of the resident waves, at
          // most kPieceRange (a block's last, partly filled batch then weighs
          // little), at least one batch
          const int64_t range = std::min<int64_t>(
              kPieceRange, std::max<int64_t>(1, nc / (16384 * kWave)) * kWave);
          k_pieces<<<dim3(unsigned(ceil_div(nc, range))), kWave, 0, s>>>(
              chunk_max, p0, p0 + nc, int(range), n_t, clips ? to_clip : nullptr,
              c->owner.as<int32_t>(), c->pair_off.as<int64_t>(), c->rng.as<CellRange>(),
              c->tetrec.as<double>(), c->tetgrad.as<double>(), c->tetvol.as<double>(),
              c->lat.as<double>(), c->ld, 1e-14, c->keep.as<uint8_t>(), c->pval.as<T>(),
              c->pmom.as<T>(), c->dual ? 1 : 0, counters);
          if ((st = hip_check(hipGetLastError(), "pieces launch"))) return st;
        }
      }
      if (fork && ((st = hip_check(hipEventRecord(c->side.join, c->side.stream), "event")) ||
                   (st = hip_check(hipStreamWaitEvent(s, c->side.join, 0), "stream wait"))))
        return st;
      const bool next = clips && li + 1 < n_live;
      if (next) {
        if ((st = hip_check(hipEventRecord(c->side.fork, s), "event")) ||
            (st = hip_check(hipStreamWaitEvent(c->side.stream, c->side.fork, 0), "stream wait")) ||
            (st = order_chunk(live[li + 1], c->side.stream)) ||
            (st = hip_check(hipEventRecord(c->side.sorted, c->side.stream), "event")))
          return st;
      }
      if (clips) {
        // (III) integrate the chunk's sub-tetrahedra, summed per pair (pairs
        // whose records did not fit the store read as empty)
        ProfScope ps("integrate", s);
        constexpr bool kMixed = sizeof(T) == sizeof(double);
        const auto integrate =
            kMixed && octants ? k_integrate<T, !kMixed> : k_integrate<T, true>;
        integrate<<<dim3(unsigned(ceil_div(nc, kWave))), kWave, 0, s>>>(
            chunk_max, p0, p0 + nc, n_t, to_clip, c->pinfo.as<uint64_t>(), c->pool.as<T>(),
            c->owner.as<int32_t>(), c->pair_off.as<int64_t>(), c->rng.as<CellRange>(),
            c->tetrec.as<double>(), c->lat.as<double>(), c->ld, c->keep.as<uint8_t>(),
            c->pval.as<T>(), c->pmom.as<T>(), c->dual ? 1 : 0);
        if ((st = hip_check(hipGetLastError(), "integrate launch"))) return st;
      }
      if ((st = gather_rows(ch))) return st;
      if (next && (st = hip_check(hipStreamWaitEvent(s, c->side.sorted, 0), "stream wait")))
        return st;
    }
    // read-back 2: records each chunk asked for, nonzeros of the three
    // components, flags
    if ((st = count_rows())) return st;
    int64_t rb2[kMaxChunks + 3];
    {
      const int64_t* src[kMaxChunks + 3];
      for (int k = 0; k < nchunk; ++k)
        src[k] = reinterpret_cast<const int64_t*>(counters + kCntChunkPool + k);
      for (int d = 0; d < 3; ++d) src[nchunk + d] = c->B[d].rowptr.as<int64_t>() + n_v;
      if ((st = read_counts(c, src, nchunk + 3, rb2, s))) return st;
    }
    if ((st = flags_status(c->host_flags))) return st;
    c->pool_needed = 0;
    for (int k = 0; k < nchunk; ++k) c->pool_needed = std::max(c->pool_needed, rb2[k]);
    for (int d = 0; d < 3; ++d) nnzs[d] = rb2[nchunk + d];
    if (c->pool_needed <= c->pool_cap) break;
    if (attempt == 1) return set_error(IBVT_E_CAPACITY, "piece store could not be sized");
  }
  // (IV) global assembly: rows of B^d (gathered per chunk above)
  for (int d = 0; d < 3; ++d) {
    const int64_t nnz = nnzs[d];
    c->B[d].nnz = nnz;
    if (nnz >= (int64_t(1) << 31) - 1)
      return set_error(IBVT_E_CAPACITY, "more than 2^31 nonzeros in one component of B");
    if ((st = ensure(c, c->B[d].col, size_t(nnz + 1) * sizeof(int32_t)))) return st;
    if ((st = ensure(c, c->B[d].val, size_t(nnz + 1) * sizeof(T)))) return st;
  }
  {
    ProfScope ps("rows_compact", s);
    k_rows_compact<T><<<blocks_for(3 * n_v * kCompactLanes, 256), 256, 0, s>>>(
        n_v, c->rowtmpoff.as<int64_t>(), c->rowtmpcol.as<int32_t>(), c->rowtmpval.as<T>(),
        c->B[0].rowptr.as<int64_t>(), c->B[1].rowptr.as<int64_t>(), c->B[2].rowptr.as<int64_t>(),
        c->B[0].col.as<int32_t>(), c->B[1].col.as<int32_t>(), c->B[2].col.as<int32_t>(),
        c->B[0].val.as<T>(), c->B[1].val.as<T>(), c->B[2].val.as<T>());
  }
  if ((st = hip_check(hipGetLastError(), "rows compact launch"))) return st;
  const int64_t* touched[3];
  {
    ProfScope ps("transpose", s);
    if ((st = transposes<T>(c, 3, touched, s))) return st;
  }
  // masses, unless they ran beside the first clip (no pairs at all)
  if (!masses_done && (st = solid_masses(c, s))) return st;
  // read-back 3: the counters of the assembly, the rows of B^dT, flags
  int64_t cnt[kCntSlots + 3];
  {
    const int64_t* src[kCntSlots + 3];
    for (int k = 0; k < kCntSlots; ++k) src[k] = reinterpret_cast<const int64_t*>(counters + k);
    for (int d = 0; d < 3; ++d) src[kCntSlots + d] = touched[d];
    if ((st = read_counts(c, src, kCntSlots + 3, cnt, s))) return st;
  }
  if ((st = transpose_done(c, 3, cnt + kCntSlots, s))) return st;
  c->stats.pairs = n_pairs;
  c->stats.pieces = cnt[kCntPieces];
  c->stats.dropped = cnt[kCntDropped];
  c->stats.zero_tets = cnt[kCntZeroTets];
  c->stats.subtets = cnt[kCntSubtets];
  c->stats.dist_evals = cnt[kCntDist];
  c->stats.cut_points = cnt[kCntCutPts];
  c->stats.plane_cuts = cnt[kCntPlanes];
  c->stats.assemblies += 1;
  if ((st = flags_status(c->host_flags))) return st;
  c->mom_valid = c->store_pieces;
  if (!c->store_pieces) {
    // memory-saving mode: no piece store kept; the reverse mode clips again
    // (the stream is idle after the read-back)
    release(c, c->pool);
    release(c, c->pmom);
    c->pool_cap = 0;
  }
  return IBVT_OK;
}

}  // namespace

int solid_masses(ibvt_coupling* c, hipStream_t s) {
  const int64_t n_v = c->n_vert;
  ProfScope ps("masses", s);
  if (c->precision == IBVT_FP32_MIXED)
    k_lumped<float><<<blocks_for(n_v, 256), 256, 0, s>>>(
        n_v, c->vt_ptr.as<int64_t>(), c->vt_tet.as<int32_t>(), c->tetvol.as<double>(),
        c->mlump.as<double>(), c->minv.as<float>());
  else
    k_lumped<double><<<blocks_for(n_v, 256), 256, 0, s>>>(
        n_v, c->vt_ptr.as<int64_t>(), c->vt_tet.as<int32_t>(), c->tetvol.as<double>(),
        c->mlump.as<double>(), c->minv.as<double>());
  if (c->has_M) {
    k_mass_values<<<blocks_for(n_v * kMassLanes, 256), 256, 0, s>>>(
        n_v, c->vt_ptr.as<int64_t>(), c->vt_tet.as<int32_t>(), c->tets.as<int32_t>(),
        c->tetvol.as<double>(), c->M.rowptr.as<int64_t>(), c->M.col.as<int32_t>(),
        c->M.val.as<double>(), c->precision == IBVT_FP32_MIXED ? c->Mval32.as<float>() : nullptr,
        c->Mdiag_inv.as<double>());
  }
  return hip_check(hipGetLastError(), "mass launch");
}

int build_topology(ibvt_coupling* c, hipStream_t s) {
  const int64_t n_t = c->n_tet, n_v = c->n_vert;
  int st;
  if ((st = ensure(c, c->flags_dev, 64))) return st;
  if ((st = ensure(c, c->counters, kCntSlots * sizeof(unsigned long long)))) return st;
  if ((st = ensure(c, c->vt_ptr, size_t(n_v + 1) * sizeof(int64_t)))) return st;
  const int K = c->dim + 1;  // vertices per element
  if ((st = ensure(c, c->vt_tet, size_t(K * n_t + 1) * sizeof(int32_t)))) return st;
  if ((st = ensure(c, c->rownnz, size_t(3 * n_v + 1) * sizeof(int64_t)))) return st;
  unsigned* flags = c->flags_dev.as<unsigned>();
  if ((st = hip_check(hipMemsetAsync(flags, 0, sizeof(unsigned), s), "memset"))) return st;
  auto* deg = c->rownnz.as<unsigned long long>();  // scratch: degrees, then cursors
  if ((st = hip_check(hipMemsetAsync(deg, 0, size_t(n_v + 1) * sizeof(int64_t), s), "memset")))
    return st;
  if (K == 4) k_vt_count<4><<<blocks_for(n_t, 256), 256, 0, s>>>(n_t, n_v, c->tets.as<int32_t>(), deg, flags);
  else k_vt_count<3><<<blocks_for(n_t, 256), 256, 0, s>>>(n_t, n_v, c->tets.as<int32_t>(), deg, flags);
  if ((st = check_flags(c, s))) return st;
  if ((st = scan_i64(c, c->rownnz.as<int64_t>(), c->vt_ptr.as<int64_t>(), n_v, s))) return st;
  if ((st = hip_check(hipMemsetAsync(deg, 0, size_t(n_v + 1) * sizeof(int64_t), s), "memset")))
    return st;
  if (K == 4)
    k_vt_fill<4><<<blocks_for(n_t, 256), 256, 0, s>>>(n_t, c->tets.as<int32_t>(),
                                                      c->vt_ptr.as<int64_t>(), deg,
                                                      c->vt_tet.as<int32_t>());
  else
    k_vt_fill<3><<<blocks_for(n_t, 256), 256, 0, s>>>(n_t, c->tets.as<int32_t>(),
                                                      c->vt_ptr.as<int64_t>(), deg,
                                                      c->vt_tet.as<int32_t>());
  k_sort_segments_i32<<<blocks_for(n_v, 256), 256, 0, s>>>(n_v, c->vt_ptr.as<int64_t>(),
                                                           c->vt_tet.as<int32_t>());
  if ((st = hip_check(hipGetLastError(), "topology launch"))) return st;
  if (c->has_M) {
    auto pattern = [&](bool fill) {
      const int64_t* vp = c->vt_ptr.as<int64_t>();
      const int32_t* vt = c->vt_tet.as<int32_t>();
      const int32_t* el = c->tets.as<int32_t>();
      int64_t* cnt = fill ? nullptr : c->rownnz.as<int64_t>();
      const int64_t* rp = fill ? c->M.rowptr.as<int64_t>() : nullptr;
      int32_t* col = fill ? c->M.col.as<int32_t>() : nullptr;
      const unsigned nb = blocks_for(n_v, 256);
      if (K == 4 && !fill) k_mass_pattern<4, false><<<nb, 256, 0, s>>>(n_v, vp, vt, el, cnt, rp, col);
      if (K == 4 && fill) k_mass_pattern<4, true><<<nb, 256, 0, s>>>(n_v, vp, vt, el, cnt, rp, col);
      if (K == 3 && !fill) k_mass_pattern<3, false><<<nb, 256, 0, s>>>(n_v, vp, vt, el, cnt, rp, col);
      if (K == 3 && fill) k_mass_pattern<3, true><<<nb, 256, 0, s>>>(n_v, vp, vt, el, cnt, rp, col);
    };
    pattern(false);
    if ((st = ensure(c, c->M.rowptr, size_t(n_v + 1) * sizeof(int64_t)))) return st;
    if ((st = scan_i64(c, c->rownnz.as<int64_t>(), c->M.rowptr.as<int64_t>(), n_v, s))) return st;
    int64_t nnz = 0;
    if ((st = read_back(c, &nnz, c->M.rowptr.as<int64_t>() + n_v, sizeof(int64_t), s))) return st;
    c->M.nrows = n_v;
    c->M.nnz = nnz;
    if ((st = ensure(c, c->M.col, size_t(nnz + 1) * sizeof(int32_t)))) return st;
    if ((st = ensure(c, c->M.val, size_t(nnz + 1) * sizeof(double)))) return st;
    if ((st = ensure(c, c->Mval32, size_t(nnz + 1) * sizeof(float)))) return st;
    if ((st = ensure(c, c->Mdiag_inv, size_t(n_v + 1) * sizeof(double)))) return st;
    pattern(true);
    if ((st = hip_check(hipGetLastError(), "mass pattern launch"))) return st;
  }
  return IBVT_OK;
}

namespace {
int assemble_grid(ibvt_coupling* c, hipStream_t s);
}  // namespace

// Every assembly starts by marking the handle unusable and marks it usable
// only when every step has succeeded, so that a failed reassembly (a solid
// leaving the lattice, a capacity error) cannot leave transfers running on a
// mix of old matrices and new per-pair data.
int assemble_all(ibvt_coupling* c, hipStream_t s) {
  c->ready = false;
  c->mom_valid = false;
  c->tcorder_valid = false;
  const int st = c->dim == 2 ? assemble_all_2d(c, s)
                 : c->unstructured ? assemble_all_unstructured(c, s)
                                   : assemble_grid(c, s);
  if (st) {
    c->mom_valid = false;
    return st;
  }
  c->ready = true;
  return IBVT_OK;
}

namespace {
int assemble_grid(ibvt_coupling* c, hipStream_t s) {
  const int64_t n_t = c->n_tet, n_v = c->n_vert;
  int st;
  // the clip's pair descriptors pack the tet and cell indices
  if (n_t >= kMaxDescTets) return set_error(IBVT_E_UNSUPPORTED, "2^30 or more tets");
  for (int k = 0; k < 9; ++k)
    if (c->ld.n[k] > (1 << kCellBits))
      return set_error(IBVT_E_UNSUPPORTED, "more than 2^21 lattice cells along one axis");
  if ((st = ensure(c, c->tetvol, size_t(n_t + 1) * sizeof(double)))) return st;
  if ((st = ensure(c, c->tetrec, size_t(n_t + 1) * kTetRec * sizeof(double)))) return st;
  if ((st = ensure(c, c->tetgrad, size_t(n_t + 1) * 12 * sizeof(double)))) return st;
  if ((st = ensure(c, c->rng, size_t(3 * n_t + 1) * sizeof(CellRange)))) return st;
  if ((st = ensure(c, c->cnt, size_t(3 * n_t + 1) * sizeof(int64_t)))) return st;
  if ((st = ensure(c, c->pair_off, size_t(3 * n_t + 1) * sizeof(int64_t)))) return st;
  if ((st = ensure(c, c->mlump, size_t(n_v + 1) * sizeof(double)))) return st;
  for (int d = 0; d < 3; ++d)
    if ((st = ensure(c, c->B[d].rowptr, size_t(n_v + 1) * sizeof(int64_t)))) return st;
  if (c->precision == IBVT_FP32_MIXED) {
    if ((st = ensure(c, c->minv, size_t(n_v + 1) * sizeof(float)))) return st;
    return assemble_typed<float>(c, s);
  }
  if ((st = ensure(c, c->minv, size_t(n_v + 1) * sizeof(double)))) return st;
  return assemble_typed<double>(c, s);
}
}  // namespace

}  // namespace ibvt
