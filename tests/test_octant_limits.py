"""Which tets csrc/moments.hpp integrates over their boundary, compiled for the
host: within its limits the values ∫ λ_i N_j are as near the exact ones as the
clip's and a missed cell's volume is rounding far below what is kept; tets past
them (flat ones, cells much narrower than their neighbours, wide tets) go to
the clip.  The reference cuts and integrates in 113-bit arithmetic."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_1810_13046_amd", "csrc")
HOST = r"""
#include <cmath>
#include <vector>
#include "moments.hpp"
using namespace ibvt;
typedef __float128 Q;
struct Tet { Q v[4][3]; };
static std::vector<Tet> cut(const std::vector<Tet>& in, int e, Q c, int sign) {
  std::vector<Tet> out;
  for (const Tet& T : in) {
    Q s[4];
    int a[4], b[4], na = 0, nb = 0;
    for (int k = 0; k < 4; ++k) {
      s[k] = sign * (T.v[k][e] - c);
      if (s[k] >= 0) a[na++] = k;
      else b[nb++] = k;
    }
    Tet p = T, q = T;  // corner k of the triangles of a prism
    auto mid = [&](int i, int j, Q* x) {
      for (int k = 0; k < 3; ++k) x[k] = T.v[i][k] + s[i] / (s[i] - s[j]) * (T.v[j][k] - T.v[i][k]);
    };
    auto put = [&](const Q* w, const Q* x, const Q* y, const Q* z) {
      Tet t;
      for (int k = 0; k < 3; ++k) { t.v[0][k] = w[k]; t.v[1][k] = x[k]; t.v[2][k] = y[k]; t.v[3][k] = z[k]; }
      out.push_back(t);
    };
    if (nb == 0) out.push_back(T);
    if (na == 0 || nb == 0) continue;
    if (na == 1) {
      for (int j = 0; j < 3; ++j) mid(a[0], b[j], p.v[j]);
      put(T.v[a[0]], p.v[0], p.v[1], p.v[2]);
      continue;
    }
    for (int j = 0; j < 3; ++j) {
      if (na == 3) {
        mid(a[j], b[0], p.v[j]);
        for (int k = 0; k < 3; ++k) q.v[j][k] = T.v[a[j]][k];
      } else if (j == 0) {
        for (int k = 0; k < 3; ++k) { p.v[0][k] = T.v[a[0]][k]; q.v[0][k] = T.v[a[1]][k]; }
      } else {
        mid(a[0], b[j - 1], p.v[j]);
        mid(a[1], b[j - 1], q.v[j]);
      }
    }
    put(p.v[0], p.v[1], p.v[2], q.v[2]);
    put(p.v[0], p.v[1], q.v[1], q.v[2]);
    put(p.v[0], q.v[0], q.v[1], q.v[2]);
  }
  return out;
}
// ∫ λ_i N_j, i * 8 + j, in cell units, with the collapsed 4 x 4 x 4 Gauss rule
static Q exact(const double* V, const double* lo, const double* hi, Q* b) {
  static Q x4[4], w4[4];
  static bool init = false;
  if (!init) {
    for (int i = 0; i < 4; ++i) {
      Q x = std::cos(M_PI * (i + 0.75) / 4.5), dp = 0;
      for (int it = 0; it < 12; ++it) {
        Q p0 = 1, p1 = x;
        for (int k = 2; k <= 4; ++k) { const Q p2 = ((2 * k - 1) * x * p1 - (k - 1) * p0) / k; p0 = p1; p1 = p2; }
        dp = 4 * (x * p1 - p0) / (x * x - 1);
        x -= p1 / dp;
      }
      x4[i] = (x + 1) / 2;
      w4[i] = 1 / ((1 - x * x) * dp * dp);
    }
    init = true;
  }
  Q E[3][3], c[3][3], g[4][3];
  for (int k = 0; k < 3; ++k)
    for (int e = 0; e < 3; ++e) E[k][e] = Q(V[3 * k + 3 + e]) - Q(V[e]);
  for (int k = 0; k < 3; ++k)
    for (int e = 0; e < 3; ++e) {
      const Q *p = E[(k + 1) % 3], *q = E[(k + 2) % 3];
      c[k][e] = p[(e + 1) % 3] * q[(e + 2) % 3] - p[(e + 2) % 3] * q[(e + 1) % 3];
    }
  const Q det = E[0][0] * c[0][0] + E[0][1] * c[0][1] + E[0][2] * c[0][2];
  for (int e = 0; e < 3; ++e) {
    for (int k = 0; k < 3; ++k) g[k + 1][e] = c[k][e] / det;
    g[0][e] = -(g[1][e] + g[2][e] + g[3][e]);
  }
  std::vector<Tet> parts(1);
  for (int k = 0; k < 12; ++k) parts[0].v[k / 3][k % 3] = V[k];
  for (int e = 0; e < 3; ++e) parts = cut(cut(parts, e, lo[e], 1), e, hi[e], -1);
  for (int k = 0; k < 32; ++k) b[k] = 0;
  const Q cell = (Q(hi[0]) - Q(lo[0])) * (Q(hi[1]) - Q(lo[1])) * (Q(hi[2]) - Q(lo[2]));
  Q total = 0;
  for (const Tet& T : parts) {
    Q d[3][3];
    for (int k = 0; k < 9; ++k) d[k / 3][k % 3] = T.v[k / 3 + 1][k % 3] - T.v[0][k % 3];
    Q vol = (d[0][0] * (d[1][1] * d[2][2] - d[1][2] * d[2][1]) -
             d[0][1] * (d[1][0] * d[2][2] - d[1][2] * d[2][0]) +
             d[0][2] * (d[1][0] * d[2][1] - d[1][1] * d[2][0])) / (6 * cell);
    if (vol < 0) vol = -vol;
    total += vol;
    for (int n = 0; n < 64; ++n) {
      const Q A = x4[n & 3], B = x4[(n >> 2) & 3], C = x4[n >> 4];
      const Q m[4] = {(1 - A) * (1 - B) * (1 - C), A, (1 - A) * B, (1 - A) * (1 - B) * C};
      const Q w = 6 * w4[n & 3] * w4[(n >> 2) & 3] * w4[n >> 4] * (1 - A) * (1 - A) * (1 - B) * vol;
      Q lam[4] = {1, 0, 0, 0}, xi[3];
      for (int e = 0; e < 3; ++e) {
        Q x = 0;
        for (int k = 0; k < 4; ++k) x += m[k] * T.v[k][e];
        for (int i = 0; i < 4; ++i) lam[i] += g[i][e] * (x - Q(V[e]));
        xi[e] = (x - Q(lo[e])) / (Q(hi[e]) - Q(lo[e]));
      }
      for (int j = 0; j < 8; ++j) {
        Q N = w;
        for (int e = 0; e < 3; ++e) N *= (j >> e) & 1 ? xi[e] : 1 - xi[e];
        for (int i = 0; i < 4; ++i) b[8 * i + j] += N * lam[i];
      }
    }
  }
  return total;
}
static void values(const double* mom, const TetGeom& G, const double* lo, const double* hi, double* b) {
  double LA[4], LG[4][3];
  cell_lambda<double>(G, lo, hi, LA, LG);
  mom_to_b<double>(mom, LA, LG, [&](int i, int j, double v) { b[8 * i + j] = v; });
}
static void geom(const double* V, TetGeom& G) {
  for (int k = 0; k < 12; ++k) G.V[k / 3][k % 3] = V[k];
  tet_geom(G);
}
extern "C" void rule(double* out) {
  out[0] = kOctantReach;
  out[1] = kOctantProduct;
  out[2] = kOctantRange;
  out[3] = kOctantCells;
}
// largest reach, their product, and the range
extern "C" void limits(const double* V, const double* const* L, const int* n, double* out) {
  TetGeom G;
  geom(V, G);
  out[0] = out[1] = 1.0;
  for (int e = 0; e < 3; ++e) {
    const double x = axis_reach(L[e], n[e], G.mn[e], G.mx[e]);
    out[0] = fmax(out[0], x);
    out[1] *= x;
  }
  out[2] = hat_range(G.g, G.mn, G.mx);
}
// largest errors of the 32 values over the cell's share of the tet (octants,
// clip), the octants' volume, the exact one
extern "C" void piece(const double* V, const double* const* L, const int* n, const int* k,
                      double* out) {
  TetGeom G;
  geom(V, G);
  double lo[3], hi[3], mom[kMom] = {0.0}, bo[32], bc[32] = {0.0};
  int two[3], m = 1;
  for (int e = 0; e < 3; ++e) {
    lo[e] = L[e][k[e]];
    hi[e] = L[e][k[e] + 1];
    m <<= (two[e] = axis_two(k[e], n[e]) ? 1 : 0);
  }
  for (int term = 0; term < m; ++term) {
    double r[4][3], sg[3], d[3], f = 1.0;
    for (int e = 0, bit = 0; e < 3; bit += two[e], ++e) {
      const AxisOctant a = axis_octant(k[e], n[e], lo[e], hi[e], G.mn[e], two[e] && ((term >> bit) & 1));
      const double ih = recip(hi[e] - lo[e]);
      for (int v = 0; v < 4; ++v) r[v][e] = a.sg * (V[3 * v + e] - a.c) * ih;
      sg[e] = a.sg;
      d[e] = a.sg * ((a.c - lo[e]) * ih - 0.5);
      if (a.minus) f = -f;
    }
    double M[kMom] = {0.0};
    auto vert = [&](int v, int e) { return r[v][e]; };
    add_face(vert, 1, 2, 3, M);
    add_face(vert, 0, 3, 2, M);
    add_face(vert, 0, 1, 3, M);
    add_face(vert, 0, 2, 1, M);
    centre_moments(M, sg, d, M[0] > 0.0 ? f : -f);
    for (int i = 0; i < kMom; ++i) mom[i] += M[i];
  }
  values(mom, G, lo, hi, bo);
  const double share = (hi[0] - lo[0]) * (hi[1] - lo[1]) * (hi[2] - lo[2]) * 6.0 / fabs(G.det);
  out[2] = mom[0] * share;
  static double x[16], y[16], z[16];
  static uint32_t nb[16];
  const PolyView P{x, y, z, nb, 1, (1u << 16) - 1u};
  Piece<16> a;
  a.walk = true;
  a.live = poly_init_tet(P, G.V, G.det < 0.0);
  poly_clip_box<16>(P, a.live, lo, hi, G.mn, G.mx, nullptr);
  if (a.live) a.want = poly_fan_prepare<16>(P, a.live, a.seen);
  double vol6 = 0.0, mc[kMom] = {0.0};
  fan_local<16>(P, a, lo, hi, [&](const double* p0, const double* p1, const double* p2,
                                  const double* p3, double) {
    double q[4][3];
    for (int e = 0; e < 3; ++e) { q[0][e] = p0[e]; q[1][e] = p1[e]; q[2][e] = p2[e]; q[3][e] = p3[e]; }
    subtet_moments<double>(q, subtet_det<double>(q[0], q[1], q[2], q[3]), mc);
  }, vol6);
  for (int i = 0; i < kMom; ++i) mc[i] *= -1.0 / 6.0;
  if (a.live) values(mc, G, lo, hi, bc);
  Q b[32];
  out[3] = double(exact(V, lo, hi, b)) * share;
  out[0] = out[1] = 0.0;
  for (int i = 0; i < 32; ++i) {
    out[0] = fmax(out[0], fabs(double(Q(bo[i]) - b[i])) * share);
    out[1] = fmax(out[1], fabs(double(Q(bc[i]) - b[i])) * share);
  }
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    hipcc = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "bin", "hipcc")
    if not (os.path.exists(hipcc) or shutil.which(hipcc)):
        pytest.skip("needs hipcc")
    d = tmp_path_factory.mktemp("limits")
    src, so = str(d / "limits.hip"), str(d / "limits.so")
    with open(src, "w") as fh:
        fh.write(HOST)
    subprocess.run([hipcc, "-x", "hip", "--offload-host-only", "-O2", "-std=c++17", "-fPIC",
                    "-shared", "-I", CSRC, src, "-o", so], check=True, capture_output=True)
    lib = ctypes.CDLL(so)
    o = (ctypes.c_double * 4)()
    lib.rule(o)
    lib.reach, lib.product, lib.range, lib.cells = o
    return lib


def look(lib, V, lines, cells=lambda n: []):
    """(largest reach, their product, range, most cells an axis) and per cell
    (octant error, clip error, octant volume, exact volume), of the tet's
    volume."""
    first = [int(np.searchsorted(a, V[:, e].min(), "right")) - 1 for e, a in enumerate(lines)]
    n = [max(int(np.searchsorted(a, V[:, e].max(), "left")) - first[e], 1)
         for e, a in enumerate(lines)]
    arr = [np.ascontiguousarray(a[first[e]:first[e] + n[e] + 1]) for e, a in enumerate(lines)]
    V = np.ascontiguousarray(V)
    ptr = (ctypes.c_void_p * 3)(*[a.ctypes.data for a in arr])
    ns, at = (ctypes.c_int * 3)(*n), (ctypes.c_double * 3)()
    lib.limits(ctypes.c_void_p(V.ctypes.data), ptr, ns, at)
    out = []
    for k in cells(n):
        o = (ctypes.c_double * 4)()
        lib.piece(ctypes.c_void_p(V.ctypes.data), ptr, ns, (ctypes.c_int * 3)(*k), o)
        out.append(list(o))
    return (*at, max(n)), np.array(out)


def within(lib, at):
    return all(x <= y for x, y in zip(at, (lib.reach, lib.product, lib.range, lib.cells)))


def kuhn(rng, size, jitter, rotate):
    """A tet of a jittered box of `size` cells."""
    c = np.zeros((4, 3))
    for v, a in enumerate(rng.permutation(3)):
        c[v + 1:, a] = 1
    q = (c + (2 * rng.random((4, 3)) - 1) * jitter) * np.asarray(size)
    if rotate:
        q = q @ np.linalg.qr(rng.standard_normal((3, 3)))[0]
    return q - q.min(0)


@pytest.mark.parametrize("size,rotate,snap,jump", [
    ((0.3,) * 3, False, 0.0, 1), ((0.9,) * 3, False, 0.0, 1), ((0.9,) * 3, True, 0.0, 1),
    ((1.3,) * 3, False, 0.5, 1), ((1.6,) * 3, True, 0.0, 1), ((2.0, 0.4, 2.0), True, 0.0, 1),
    ((1.0, 2.8, 1.0), False, 0.5, 1), ((2.2,) * 3, False, 0.0, 1), ((1.2,) * 3, False, 0.0, 3),
    ((0.7,) * 3, True, 0.0, 30)])
def test_within_the_limits(lib, size, rotate, snap, jump):
    """As near as the clip, root mean square over the cells; and no volume where
    there is none (a tenth of the 1e-14 that is kept)."""
    rng = np.random.default_rng(int(100 * sum(size)) + jump)
    sums, seen, taken = np.zeros(2), 0, 0
    while taken < 60:
        seen += 1
        assert seen < 4000
        lines = [np.concatenate([[0.0], np.cumsum(jump ** -rng.random(40))]) for _ in range(3)]
        V = kuhn(rng, size, 0.1, rotate) + [a[15] + rng.random() for a in lines]
        V = np.where(rng.random((4, 3)) < snap, np.round(2 * V) / 2, V)
        if abs(np.linalg.det(V[1:] - V[0])) < 1e-3 * np.prod(size):
            continue
        at, out = look(lib, V, lines, lambda n: [
            [int(rng.integers(m)) for m in n] for _ in range(6)])
        if not within(lib, at):
            continue
        taken += 1
        sums += (out[:, :2] ** 2).sum(0)
        assert np.all(out[out[:, 3] == 0, 2] <= 1e-15)
    assert sums[0] <= sums[1]


@pytest.mark.parametrize("axes,jump", [(1, 10), (1, 100), (1, 1000), (3, 10), (3, 100), (3, 1000)])
def test_narrow_cells_are_past_the_limits(lib, axes, jump):
    """Tets over three cells of widths 1, 1/jump, 1: the narrow cell's
    half-lines reach over a wide one."""
    rng = np.random.default_rng(jump + axes)
    lines = [np.array([0.0, 1.0, 1.0 + (1.0 / jump if e < axes else 1.0), 3.0, 4.0]) for e in range(3)]
    for _ in range(20):
        V = kuhn(rng, (1.6,) * 3, 0.1, False) + 0.3
        assert not within(lib, look(lib, V, lines)[0])


@pytest.mark.parametrize("size", [0.7, 2.5, 5.0])
@pytest.mark.parametrize("flat", [1e-2, 1e-3, 1e-4, 1e-6])
def test_flat_tets_are_past_the_limits(lib, size, flat):
    """The fourth vertex `flat` of the size off the others' plane, askew."""
    rng = np.random.default_rng(int(size * 10))
    lines = [np.arange(40.0)] * 3
    for _ in range(20):
        R = np.linalg.qr(rng.standard_normal((3, 3)))[0]
        while np.abs(R[2]).min() < 0.3:  # the normal
            R = np.linalg.qr(rng.standard_normal((3, 3)))[0]
        V = np.array([[0, 0, 0], [1, 0, 0], [0.2, 0.9, 0], [0.5, 0.4, flat]]) * size @ R + 15.3
        assert look(lib, V, lines)[0][2] > lib.range


def test_wide_tets_are_past_the_limits(lib):
    """More than six cells along an axis, a reach of more than 1.7 along one, or
    of more than 1.4 along three."""
    rng = np.random.default_rng(0)
    lines = [np.arange(40.0)] * 3
    for _ in range(20):
        assert look(lib, kuhn(rng, (6.6, 0.5, 0.5), 0.02, False) + 15.3, lines)[0][3] > lib.cells
        assert look(lib, kuhn(rng, (3.9, 0.5, 0.5), 0.02, False) + 15.3, lines)[0][0] > lib.reach
        assert look(lib, kuhn(rng, (2.2,) * 3, 0.02, False) + 15.3, lines)[0][1] > lib.product
