"""Piece moments from boundary integrals (csrc/moments.hpp), compiled for the
host, against exact pieces: the tet is cut by the cell's planes in rationals
and every simplex integrated with a product Gauss rule in extended precision.
"""
import ctypes
import itertools
import os
import shutil
import subprocess
from fractions import Fraction

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_1810_13046_amd", "csrc")
HOST = r"""
#include "moments.hpp"
using namespace ibvt;
// moments about the cell centre, in cell units, of tet V in cell k of n per axis
extern "C" void piece(const double* V, const double* lo, const double* hi, const int* n,
                      const int* k, double* out) {
  for (int i = 0; i < kMom; ++i) out[i] = 0.0;
  int two[3], m = 1;
  for (int e = 0; e < 3; ++e) m <<= (two[e] = axis_two(k[e], n[e]) ? 1 : 0);
  for (int term = 0; term < m; ++term) {
    double r[4][3], sg[3], d[3], f = 1.0;
    for (int e = 0, bit = 0; e < 3; bit += two[e], ++e) {
      const double mn = fmin(fmin(V[e], V[3 + e]), fmin(V[6 + e], V[9 + e]));
      const AxisOctant a =
          axis_octant(k[e], n[e], lo[e], hi[e], mn, two[e] && ((term >> bit) & 1));
      const double ih = 1.0 / (hi[e] - lo[e]);
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
    for (int i = 0; i < kMom; ++i) out[i] += M[i];
  }
}
"""
EXP = [(a, b, c) for a in range(4) for b in range(min(3, 4 - a) + 1)
       for c in range(min(3, 4 - a - b) + 1)]


@pytest.fixture(scope="module")
def piece(tmp_path_factory):
    hipcc = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "bin", "hipcc")
    if not (os.path.exists(hipcc) or shutil.which(hipcc)):
        pytest.skip("needs hipcc")
    d = tmp_path_factory.mktemp("octant")
    src, so = str(d / "piece.hip"), str(d / "piece.so")
    with open(src, "w") as fh:
        fh.write(HOST)
    subprocess.run([hipcc, "-x", "hip", "--offload-host-only", "-O2", "-std=c++17", "-fPIC",
                    "-shared", "-I", CSRC, src, "-o", so], check=True, capture_output=True)
    lib = ctypes.CDLL(so)

    def call(V, lo, hi, n, k):
        out = np.zeros(32)
        arr = [np.ascontiguousarray(V, dtype=np.float64), np.asarray(lo, dtype=np.float64),
               np.asarray(hi, dtype=np.float64), np.asarray(n, dtype=np.int32),
               np.asarray(k, dtype=np.int32), out]
        lib.piece(*[ctypes.c_void_p(a.ctypes.data) for a in arr])
        return out
    return call


def cut(T, e, c, sign):
    """The simplices of tet T (rational vertices) with sign·(x_e − c) >= 0."""
    s = [sign * (v[e] - c) for v in T]
    ins, outs = [i for i in range(4) if s[i] >= 0], [i for i in range(4) if s[i] < 0]

    def mid(i, j):
        t = s[i] / (s[i] - s[j])
        return tuple(T[i][k] + t * (T[j][k] - T[i][k]) for k in range(3))

    def prism(p, q):
        return [(p[0], p[1], p[2], q[2]), (p[0], p[1], q[1], q[2]), (p[0], q[0], q[1], q[2])]
    if not outs:
        return [T]
    if not ins:
        return []
    if len(ins) == 1:
        return [(T[ins[0]],) + tuple(mid(ins[0], j) for j in outs)]
    if len(ins) == 3:
        return prism([mid(i, outs[0]) for i in ins], [T[i] for i in ins])
    (a, b), (c2, d) = ins, outs
    return prism((T[a], mid(a, c2), mid(a, d)), (T[b], mid(b, c2), mid(b, d)))


def exact(V, lo, hi):
    F = lambda x: Fraction(float(x))
    parts = [tuple(tuple(F(c) for c in v) for v in V)]
    for e in range(3):
        parts = [t for T in parts for t in cut(T, e, F(lo[e]), 1)]
        parts = [t for T in parts for t in cut(T, e, F(hi[e]), -1)]
    out = np.zeros(32, dtype=np.longdouble)
    if not parts:
        return out.astype(float)
    P = np.array([[[float((v[e] - F(lo[e])) / (F(hi[e]) - F(lo[e])) - Fraction(1, 2))
                    for e in range(3)] for v in T] for T in parts], dtype=np.longdouble)
    vol = np.abs(np.linalg.det((P[:, 1:] - P[:, :1]).astype(float))) / 6
    (x4, w4), (x3, w3) = (np.polynomial.legendre.leggauss(m) for m in (4, 3))
    for (a, wa), (b, wb), (c, wc) in itertools.product(
            *[list(zip(0.5 * (x + 1), 0.5 * w)) for x, w in ((x4, w4), (x3, w3), (x3, w3))]):
        l1, l2, l3 = a, (1 - a) * b, (1 - a) * (1 - b) * c
        p = (1 - l1 - l2 - l3) * P[:, 0] + l1 * P[:, 1] + l2 * P[:, 2] + l3 * P[:, 3]
        w = 6 * wa * wb * wc * (1 - a) ** 2 * (1 - b) * vol
        for i, (q, r, s) in enumerate(EXP):
            out[i] += (w * p[:, 0] ** q * p[:, 1] ** r * p[:, 2] ** s).sum()
    return out.astype(float)


@pytest.mark.parametrize("size,snap,offset", [
    (0.02, False, 0.3), (0.8, False, 0.0), (1.5, False, 0.7), (1.5, True, 0.3),
    (2.7, True, 0.0), (2.7, False, 0.6), (5.0, False, 0.2)])
def test_piece_moments(piece, size, snap, offset):
    """Tets of `size` cells (5: up to six cells an axis), with vertices, edges
    and faces in cell planes (snap), either orientation.  Every sum is over
    terms of at most Π(extent) · reach⁴ in cell units (reach: the cells an
    octant can extend, at most 3); a few hundred roundings each."""
    rng = np.random.default_rng(int(100 * size) + snap)
    h = 1.0 / 64
    lines = np.arange(65) * h
    cells_seen = 0
    while cells_seen < 60:
        V = (rng.random((4, 3)) * size + offset / h) * h
        if snap:
            V = np.where(rng.random((4, 3)) < 0.5, np.round(2 * V / h) / 2 * h, V)
        if abs(np.linalg.det(V[1:] - V[0])) < 1e-6 * (size * h) ** 3:
            continue
        mn, mx = V.min(0), V.max(0)
        i0 = [int(np.searchsorted(lines, mn[e], "right")) - 1 for e in range(3)]
        n = [max(int(np.searchsorted(lines, mx[e], "left")) - i0[e], 1) for e in range(3)]
        assert max(n) <= 6
        ext = np.minimum((mx - mn) / h, 3.0)
        tol = 400 * 2.3e-16 * np.prod(ext) * max(1.0, ext.max()) ** 4
        cells = list(itertools.product(*map(range, n)))
        for c in [cells[j] for j in rng.permutation(len(cells))[:8]]:
            lo = [lines[i0[e] + c[e]] for e in range(3)]
            hi = [lines[i0[e] + c[e] + 1] for e in range(3)]
            assert np.abs(piece(V, lo, hi, n, c) - exact(V, lo, hi)).max() <= tol
            cells_seen += 1
