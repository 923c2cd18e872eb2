// Moments of tet ∩ octant from boundary integrals (no clipped polyhedron).
//
// A piece tet ∩ cell is bounded by parts of the tet's faces and of the
// straddled cell planes.  Put the origin on one cell plane per straddled
// axis and orient the axes so that the piece lies in the octant r >= 0.  By
// the divergence theorem with the field r f/(|α| + 3), f = r^α,
//   ∫_P r^α dV = 1/(|α| + 3) Σ_faces ∫_face (n · r) r^α dA,
// and the faces on the cell planes drop out: they contain the origin.  On a
// tet face n · r is constant; the face is projected along its dominant axis
// w (|n_w| largest), where w = k0 + k1 u + k2 v with |k1|, |k2| <= 1, so
//   ∫_face (n · r) r^α dA = k0 ∫_D w^a u^b v^c du dv,
// D being the projection of the triangle's part in the octant.  The same
// step once more: with the field (u, v) g/(b + c + 2),
//   ∫_D u^b v^c du dv = 1/(b + c + 2) Σ_edges (p × q) ∫_0^1 u^b v^c dt,
// and the edges of D on the lines u = 0 and v = 0 drop out.  What is left
// are the parts of the triangle's three edges in the octant and the segment
// where the face crosses the plane w = 0, each integrated in closed form: no
// vertex graph, no lists, no sub-tetrahedra.
//
// Signs are decided once per vertex and axis (r >= 0 is inside) and every
// crossing point is computed once per face, so the boundary closes to
// rounding; all terms are bounded by the tet's bounding box.
#pragma once

#include "geometry.hpp"

namespace ibvt {

// 1/x to an ulp or two (device: hardware reciprocal and two Newton steps).
__host__ __device__ __forceinline__ double recip(double x) {
#if defined(__HIP_DEVICE_COMPILE__)
  double r = __builtin_amdgcn_rcp(x);
  r = fma(fma(-x, r, 1.0), r, r);
  return fma(fma(-x, r, 1.0), r, r);
#else
  return 1.0 / x;
#endif
}

// N reciprocals at a time, step by step (each alone is a chain of dependent
// operations).
template <int N>
__host__ __device__ __forceinline__ void recips(const double* x, double* r) {
#if defined(__HIP_DEVICE_COMPILE__)
  double q[N];
#pragma unroll
  for (int e = 0; e < N; ++e) r[e] = __builtin_amdgcn_rcp(x[e]);
#pragma unroll
  for (int k = 0; k < 2; ++k) {
#pragma unroll
    for (int e = 0; e < N; ++e) q[e] = fma(-x[e], r[e], 1.0);
#pragma unroll
    for (int e = 0; e < N; ++e) r[e] = fma(q[e], r[e], r[e]);
  }
#else
  for (int e = 0; e < N; ++e) r[e] = 1.0 / x[e];
#endif
}

// Makes the compiler finish x here: left free, it works on all segments of a
// face at once and needs 50 registers more.
__host__ __device__ __forceinline__ void finish(double& x) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("" : "+v"(x));
#endif
}

// Two-dimensional moments of one projected face: m[b][c] sums, over the
// boundary segments p → q, (p × q) C(n, b) Σ_{i <= n} sym(p^i q^(n − i))_{b,c}
// with n = b + c <= 4, which is (n + 1) C(n, b) (p × q) ∫_0^1 u^b v^c dt.
struct FaceMoments {
  double m[5][5];
};

// One segment p → (u, v) (live: it has a part in the octant).  With the
// binomials inside, S_n = p S_{n−1} + q^n (products of polynomials in the two
// coordinates): 55 operations for the 15 sums, against 103 with three Gauss
// points.
__host__ __device__ __forceinline__ void add_segment(FaceMoments& f, bool live, double pu,
                                                     double pv, double u, double v) {
  const double cr = live ? pu * v - pv * u : 0.0;
  f.m[0][0] += cr;
  const double a1 = pu + u, a0 = pv + v;  // by the power of u
  f.m[1][0] = fma(cr, a1, f.m[1][0]);
  f.m[0][1] = fma(cr, a0, f.m[0][1]);
  const double u2 = u * u, v2 = v * v;
  const double b2 = fma(pu, a1, u2), b1 = fma(pu, a0, fma(pv, a1, (2.0 * u) * v)),
               b0 = fma(pv, a0, v2);
  f.m[2][0] = fma(cr, b2, f.m[2][0]);
  f.m[1][1] = fma(cr, b1, f.m[1][1]);
  f.m[0][2] = fma(cr, b0, f.m[0][2]);
  const double u3 = u2 * u, v3 = v2 * v;
  const double c3 = fma(pu, b2, u3), c2 = fma(pu, b1, fma(pv, b2, u2 * (3.0 * v))),
               c1 = fma(pu, b0, fma(pv, b1, (3.0 * u) * v2)), c0 = fma(pv, b0, v3);
  f.m[3][0] = fma(cr, c3, f.m[3][0]);
  f.m[2][1] = fma(cr, c2, f.m[2][1]);
  f.m[1][2] = fma(cr, c1, f.m[1][2]);
  f.m[0][3] = fma(cr, c0, f.m[0][3]);
  const double d4 = fma(pu, c3, u2 * u2), d3 = fma(pu, c2, fma(pv, c3, u3 * (4.0 * v))),
               d2 = fma(pu, c1, fma(pv, c2, u2 * (6.0 * v2))),
               d1 = fma(pu, c0, fma(pv, c1, (4.0 * u) * v3)), d0 = fma(pv, c0, v2 * v2);
  f.m[4][0] = fma(cr, d4, f.m[4][0]);
  f.m[3][1] = fma(cr, d3, f.m[3][1]);
  f.m[2][2] = fma(cr, d2, f.m[2][2]);
  f.m[1][3] = fma(cr, d1, f.m[1][3]);
  f.m[0][4] = fma(cr, d0, f.m[0][4]);
#pragma unroll
  for (int b = 0; b <= 4; ++b)
#pragma unroll
    for (int c = 0; c <= 4 - b; ++c) finish(f.m[b][c]);
}

// The part [t0, t1] of the segment a → b where the first N coordinates are
// >= 0 (returns whether there is one), and the parameters t[e] at which the
// segment meets the planes (any number of [0, 1] where it does not, so that
// what is computed from them and masked later is finite).  Selects only, a step of all the axes at a time: a branch per case costs a
// wave more than it saves, and one axis after the other is a chain of
// dependent operations.
template <int N>
__host__ __device__ __forceinline__ bool clip_interval(const double* a, const double* b, double* t,
                                                       double& t0, double& t1) {
  double den[N], r[N];
#pragma unroll
  for (int e = 0; e < N; ++e) den[e] = a[e] - b[e];
  recips<N>(den, r);
  t0 = 0.0;
  t1 = 1.0;
  bool dead = false;
#pragma unroll
  for (int e = 0; e < N; ++e) t[e] = fmin(fmax(a[e] * r[e], 0.0), 1.0);
#pragma unroll
  for (int e = 0; e < N; ++e) {
    const bool na = a[e] < 0.0, nb = b[e] < 0.0;
    t0 = fmax(t0, na ? t[e] : 0.0);
    t1 = fmin(t1, nb ? t[e] : 1.0);
    dead |= na & nb;
  }
  return !dead & (t1 > t0);
}

// Power A of w = k0 + k1 u + k2 v: m ← k0 m + k1 (m, b + 1) + k2 (m, c + 1),
// one degree less each time, and its sums into M: M[α] += m[b][c] for the
// exponents (u, v, w) = (b, c, A).  is[W] = 1 if w is axis W, else 0: three
// multiply-adds instead of three branches, which a wave would run anyway and
// for which the compiler keeps a second copy of M.
template <int A>
__host__ __device__ __forceinline__ void next_power(FaceMoments& f, const double is[3], double k0,
                                                    double k1, double k2, double M[kMom]) {
  if (A > 0) {
#pragma unroll
    for (int b = 0; b <= 4 - A; ++b)
#pragma unroll
      for (int c = 0; c <= 4 - A - b; ++c)
        f.m[b][c] = fma(k0, f.m[b][c], fma(k1, f.m[b + 1][c], k2 * f.m[b][c + 1]));
  }
#pragma unroll
  for (int b = 0; b <= 4 - A && b <= 3; ++b)
#pragma unroll
    for (int c = 0; c <= 4 - A - b && c <= 3; ++c) {
      const double x = f.m[b][c];
      M[mom_idx(b, c, A)] = fma(is[2], x, M[mom_idx(b, c, A)]);
      M[mom_idx(A, b, c)] = fma(is[0], x, M[mom_idx(A, b, c)]);
      M[mom_idx(c, A, b)] = fma(is[1], x, M[mom_idx(c, A, b)]);
    }
}

// Adds the face with vertices a, b, c (counter-clockwise seen from outside)
// to M: M[α] += ∫ (n · r) r^α dA over its part in the octant.  vert(v, e):
// coordinate e of vertex v (read again in the order of the face's axes,
// which costs less than choosing among registers).
template <typename Vert>
__host__ __device__ __forceinline__ void add_face(Vert&& vert, int va, int vb, int vc,
                                                  double M[kMom]) {
  double n[3];
  {
    const double A[3] = {vert(va, 0), vert(va, 1), vert(va, 2)};
    const double e[3] = {vert(vb, 0) - A[0], vert(vb, 1) - A[1], vert(vb, 2) - A[2]};
    const double g[3] = {vert(vc, 0) - A[0], vert(vc, 1) - A[1], vert(vc, 2) - A[2]};
    n[0] = e[1] * g[2] - e[2] * g[1];
    n[1] = e[2] * g[0] - e[0] * g[2];
    n[2] = e[0] * g[1] - e[1] * g[0];
  }
  const double an0 = fabs(n[0]), an1 = fabs(n[1]), an2 = fabs(n[2]);
  const int w = (an2 >= an0 && an2 >= an1) ? 2 : (an0 >= an1 ? 0 : 1);
  // cyclic axes: w = 2: (x, y, z), w = 0: (y, z, x), w = 1: (z, x, y)
  const int au = w == 2 ? 0 : w + 1, av = w == 1 ? 0 : (w == 0 ? 2 : 1);
  const double nu = w == 2 ? n[0] : (w == 0 ? n[1] : n[2]);
  const double nv = w == 2 ? n[1] : (w == 0 ? n[2] : n[0]);
  const double nw = w == 2 ? n[2] : (w == 0 ? n[0] : n[1]);
  FaceMoments f;
#pragma unroll
  for (int b = 0; b <= 4; ++b)
#pragma unroll
    for (int c = 0; c <= 4 - b; ++c) f.m[b][c] = 0.0;
  double xu = 0, xv = 0, yu = 0, yv = 0;  // where the boundary leaves and enters w >= 0
  auto edge = [&](int ka, int kb) {
    const double a[3] = {vert(ka, au), vert(ka, av), vert(ka, w)};
    const double b[3] = {vert(kb, au), vert(kb, av), vert(kb, w)};
    const double du = b[0] - a[0], dv = b[1] - a[1];
    double t[3], t0, t1;
    const bool live = clip_interval<3>(a, b, t, t0, t1);
    const bool in = a[2] < 0.0 & !(b[2] < 0.0), out = !(a[2] < 0.0) & b[2] < 0.0;
    const double cu = fma(t[2], du, a[0]), cv = fma(t[2], dv, a[1]);
    yu = in ? cu : yu;
    yv = in ? cv : yv;
    xu = out ? cu : xu;
    xv = out ? cv : xv;
    add_segment(f, live, fma(t0, du, a[0]), fma(t0, dv, a[1]), fma(t1, du, a[0]),
                fma(t1, dv, a[1]));
  };
  edge(va, vb);
  edge(vb, vc);
  edge(vc, va);
  {
    // the segment on w = 0 closes the boundary (both ends are the origin,
    // giving nothing, where the face does not cross that plane)
    const double x[2] = {xu, xv}, y[2] = {yu, yv};
    const double du = yu - xu, dv = yv - xv;
    double t[2], t0, t1;
    const bool live = clip_interval<2>(x, y, t, t0, t1);
    add_segment(f, live, fma(t0, du, xu), fma(t0, dv, xv), fma(t1, du, xu), fma(t1, dv, xv));
  }
  // a face without area has no axis and adds nothing
  const bool flat = nw == 0.0;
  const double in = flat ? 0.0 : recip(nw);
  const double is[3] = {!flat && w == 0 ? 1.0 : 0.0, !flat && w == 1 ? 1.0 : 0.0,
                        !flat && w == 2 ? 1.0 : 0.0};
  const double k1 = -nu * in, k2 = -nv * in;
  const double k0 = vert(va, w) - k1 * vert(va, au) - k2 * vert(va, av);
#pragma unroll
  for (int b = 0; b <= 4; ++b)
#pragma unroll
    for (int c = 0; c <= 4 - b; ++c) {
      // C(n, b) for n = b + c <= 4
      const int n = b + c, lo = b < c ? b : c;
      const double binom = lo == 0 ? 1.0 : (lo == 1 ? double(n) : 6.0);
      f.m[b][c] *= k0 * (1.0 / ((n + 1) * (n + 2) * binom));
    }
  next_power<0>(f, is, k0, k1, k2, M);
  next_power<1>(f, is, k0, k1, k2, M);
  next_power<2>(f, is, k0, k1, k2, M);
  next_power<3>(f, is, k0, k1, k2, M);
}

// ∫ (r + d e_x)^α from ∫ r^α, one axis (AX) at a time: along each chain of
// powers of that axis the shift is a triangle of multiply-adds.
template <int AX>
__host__ __device__ __forceinline__ void shift_axis(double M[kMom], double d) {
#pragma unroll
  for (int p = 0; p <= 3; ++p)
#pragma unroll
    for (int q = 0; q <= 4 - p && q <= 3; ++q) {
      constexpr int kTop = 3;
      const int top = 4 - p - q < kTop ? 4 - p - q : kTop;
#pragma unroll
      for (int j = 1; j <= top; ++j)
#pragma unroll
        for (int k = top; k >= j; --k) {
          const int hi = AX == 0 ? mom_idx(k, p, q) : (AX == 1 ? mom_idx(p, k, q) : mom_idx(p, q, k));
          const int lo = AX == 0 ? mom_idx(k - 1, p, q)
                                 : (AX == 1 ? mom_idx(p, k - 1, q) : mom_idx(p, q, k - 1));
          M[hi] += d * M[lo];
        }
    }
}

// From the octant sums M (Σ_faces of add_face) in r_e = sg_e (x_e − c_e)/h_e
// to the moments about the cell centre, s_e = sg_e (r_e + d_e), times
// `factor`.
__host__ __device__ __forceinline__ void centre_moments(double M[kMom], const double sg[3],
                                                        const double d[3], double factor) {
#pragma unroll
  for (int a = 0; a <= 3; ++a)
#pragma unroll
    for (int b = 0; b <= 4 - a && b <= 3; ++b)
#pragma unroll
      for (int c = 0; c <= 4 - a - b && c <= 3; ++c) M[mom_idx(a, b, c)] *= 1.0 / (a + b + c + 3);
  shift_axis<0>(M, d[0]);
  shift_axis<1>(M, d[1]);
  shift_axis<2>(M, d[2]);
#pragma unroll
  for (int a = 0; a <= 3; ++a) {
    const double fa = (a & 1) ? factor * sg[0] : factor;
#pragma unroll
    for (int b = 0; b <= 4 - a && b <= 3; ++b) {
      const double fb = (b & 1) ? fa * sg[1] : fa;
#pragma unroll
      for (int c = 0; c <= 4 - a - b && c <= 3; ++c)
        M[mom_idx(a, b, c)] *= (c & 1) ? fb * sg[2] : fb;
    }
  }
}

// The octants of one piece.  Along an axis with n cells in the tet's range,
// cell k is cut by its low plane if k > 0 and by its high plane if
// k < n − 1.  One plane (or none: the tet's least coordinate takes its
// place) gives the axis one term.  A cell cut by both is the difference of
// two half-lines, taken on the side where fewer of the tet's cells lie
// beyond.  A piece with m such axes has 2^m terms; bit i of `term` chooses
// on the i-th of them.  The terms are queued with three bits for k: at most
// kOctantCells cells an axis.
constexpr int kOctantCells = 6;

struct AxisOctant {
  double c;   // coordinate of the origin
  double sg;  // r = sg (x − c)/h
  bool minus; // the term is subtracted
};

__host__ __device__ __forceinline__ bool axis_two(int k, int n) { return k > 0 && k < n - 1; }

__host__ __device__ __forceinline__ AxisOctant axis_octant(int k, int n, double lo, double hi,
                                                           double mn, bool second) {
  const bool low = k > 0, high = k < n - 1;
  const bool up = low && (!high || n - k <= k + 1);  // measured upwards from the low plane
  AxisOctant a;
  a.sg = (high && !up) ? -1.0 : 1.0;
  const bool at_lo = up != (second && low && high);
  a.c = (low || high) ? (at_lo ? lo : hi) : mn;
  a.minus = second && low && high;
  return a;
}

// Which tets these sums are for.  Two things cost digits that the clip, whose
// arithmetic stays in the piece, keeps:
//  - the difference of two half-lines cancels what lies beyond the cell.
//    axis_reach is how far they reach, in widths of that cell (a narrow cell
//    between wide ones reaches far), 1 where no cell of the axis is cut
//    twice.  The volume grows by the product over the axes, a moment by up to
//    the fourth power of one of them;
//  - the moments' roundings are independent, and λ multiplies them by its
//    gradients.  hat_range is the most λ varies over the tet's box: 2 for the
//    six tets of a box, 4 to 5 when they are jittered and turned, any number
//    for a flat tet askew to the axes.
// A tet past a limit is clipped, as is one wider than kOctantCells.
//
// Error of ∫ λ_i N_j / of the shape terms over the clip's, both against 113
// bits, root mean square over the cells of 230,656 tets of 0.05 to 5 cells
// (of boxes, jittered, turned, stretched, and of random vertices; cells equal
// or with neighbours up to 1 : 100), the range at most 6:
//   product of the reaches 1: 0.17 / 0.09, 1 to 2: 0.5 / 0.7,
//   2 to 2.5: 0.7 / 1.3 (one reach above 2: 2.7 / 4.8), 3 to 4: 1.2 / 2.1
//   (above 2.5: 4.8 / 13); cubes of 4 cells 5 / 4, of 4.9 cells 9 / 6;
//   three cells of widths 1, 1/100, 1 along every axis: more than 1e4.
// By size and kind of tet, those within the limits are at 0.2 to 0.6 / 0.3 to
// 1.3.  A range of 40 and more costs a factor of tens to thousands.
// Within the limits the volume of a cell that the tet misses rounds to at
// most 5e-16 of the tet's, far below what is kept (1e-14).
constexpr double kOctantReach = 1.7;     // along each axis
constexpr double kOctantProduct = 2.5;   // of the three
constexpr double kOctantRange = 6.0;

// L: the n + 1 cell planes of the tet's range along the axis; [mn, mx]: the tet.
__host__ __device__ inline double axis_reach(const double* L, int n, double mn, double mx) {
  double r = 1.0;
  for (int k = 1; k < n - 1; ++k) {
    const AxisOctant a = axis_octant(k, n, L[k], L[k + 1], mn, false);
    r = fmax(r, (a.sg > 0.0 ? mx - a.c : a.c - mn) / (L[k + 1] - L[k]));
  }
  return r;
}

// g[i]: ∇λ_i; [mn, mx]: the tet's box.
__host__ __device__ inline double hat_range(const double g[4][3], const double mn[3],
                                            const double mx[3]) {
  double r = 0.0;
  for (int i = 0; i < 4; ++i) {
    double x = 0.0;
    for (int e = 0; e < 3; ++e) x += fabs(g[i][e]) * (mx[e] - mn[e]);
    r = fmax(r, x);
  }
  return r;
}

}  // namespace ibvt
