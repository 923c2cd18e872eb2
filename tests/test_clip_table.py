"""The clip by look-up (csrc/gen_clip_table.py, clip_piece_box) against the
clip that keeps and walks the vertex graph, both compiled for the host: the
same slots, the same coordinates and the same sub-tetrahedra in the same
order, bit for bit."""
import ctypes
import importlib.util
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_1810_13046_amd", "csrc")
HOST = r"""
#include <cstring>
#include "geometry.hpp"
using namespace ibvt;
struct Box { double x[16], y[16], z[16]; uint32_t nb[16]; };
// 1: not equal; 0: equal, the fan from a record; -1: equal, by a walk
template <int NS>
int compare(const double* V, const double* lo, const double* hi, const ClipTables& tab) {
  static Box A, B;
  const PolyView P{A.x, A.y, A.z, A.nb, 1, (1u << NS) - 1u};
  const PolyView Q{B.x, B.y, B.z, B.nb, 1, (1u << NS) - 1u};
  TetGeom G;
  for (int k = 0; k < 4; ++k)
    for (int e = 0; e < 3; ++e) G.V[k][e] = V[3 * k + e];
  tet_geom(G);
  ClipCount ca, cb;
  Piece<NS> a, b;
  a.walk = true;
  a.live = poly_init_tet(P, G.V, G.det < 0.0);
  if (!poly_clip_box<NS>(P, a.live, lo, hi, G.mn, G.mx, &ca)) return 1;
  if (a.live) a.want = poly_fan_prepare<NS>(P, a.live, a.seen);
  clip_piece_box<NS>(Q, tab, G, lo, hi, b, &cb);
  if (!b.ok || a.live != b.live || a.want != b.want || ca.planes != cb.planes ||
      ca.dist != cb.dist || ca.cuts != cb.cuts)
    return 1;
  static double ra[64][13], rb[64][13];
  double va = 0.0, vb = 0.0;
  int na = 0, nb = 0;
  auto into = [](double (*r)[13], int& n) {
    return [r, &n](const double* p0, const double* p1, const double* p2, const double* p3,
                   double det) {
      const double* p[4] = {p0, p1, p2, p3};
      for (int k = 0; k < 12; ++k) r[n][k] = p[k / 3][k % 3];
      r[n++][12] = det;
    };
  };
  if (!fan_local<NS>(P, a, lo, hi, into(ra, na), va)) return 1;
  if (!fan_local<NS>(Q, b, lo, hi, into(rb, nb), vb)) return 1;
  if (na != nb || va != vb || std::memcmp(ra, rb, size_t(na) * sizeof(ra[0]))) return 1;
  return b.walk ? -1 : 0;
}
extern "C" int compare(int slots, const double* V, const double* lo, const double* hi,
                       const void* cut, const void* fan, const void* graph) {
  const ClipTables tab{static_cast<const uint4*>(cut), static_cast<const uint4*>(fan),
                       static_cast<const uint4*>(graph)};
  return slots == 10 ? compare<10>(V, lo, hi, tab)
                     : (slots == 12 ? compare<12>(V, lo, hi, tab) : compare<16>(V, lo, hi, tab));
}
"""


@pytest.fixture(scope="module")
def compare(tmp_path_factory):
    hipcc = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "bin", "hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("needs hipcc")
    spec = importlib.util.spec_from_file_location("gen_clip_table",
                                                  os.path.join(CSRC, "gen_clip_table.py"))
    gen = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(gen)
    tabs = [np.array([[r >> 32 * k & 0xFFFFFFFF for k in range(4)] for r in t], dtype=np.uint32)
                for t in gen.tables()]
    d = tmp_path_factory.mktemp("clip")
    src, so = str(d / "clip.hip"), str(d / "clip.so")
    with open(src, "w") as fh:
        fh.write(HOST)
    subprocess.run([hipcc, "-x", "hip", "--offload-host-only", "-O1", "-ffp-contract=off",
                    "-std=c++17", "-fPIC", "-shared", "-I", CSRC, src, "-o", so], check=True,
                   capture_output=True)
    lib = ctypes.CDLL(so)

    def call(slots, V, lo, hi):
        a = [np.ascontiguousarray(x, dtype=np.float64) for x in (V, lo, hi)] + tabs
        return lib.compare(slots, *[ctypes.c_void_p(x.ctypes.data) for x in a])
    return call


@pytest.mark.parametrize("size,snap", [(0.2, 0.0), (0.6, 0.0), (1.3, 0.0), (1.3, 0.5), (2.5, 0.3),
                                       (2.5, 0.8)])
def test_table_clip_equals_graph_walk(compare, size, snap):
    """Random tets, some of their coordinates in cell planes, in every cell of
    their box, with the slots the number of planes around it asks for: up to
    three planes (10 slots) are looked up but for a few, more end in a walk."""
    rng = np.random.default_rng(int(10 * size + 100 * snap))
    h, seen, walked, planes = 1.0 / 32, 0, 0, np.zeros(7, dtype=int)
    while seen < 4000:
        V = (rng.random((4, 3)) * size + 8) * h
        V = np.where(rng.random((4, 3)) < snap, np.round(2 * V / h) / 2 * h, V)
        if abs(np.linalg.det(V[1:] - V[0])) < 1e-12:
            continue
        i0 = np.floor(V.min(0) / h).astype(int)
        i1 = np.maximum(np.ceil(V.max(0) / h).astype(int) - 1, i0)
        for c in np.ndindex(*(i1 - i0 + 1)):
            c = i0 + np.array(c)
            n = (c > i0).sum() + (c < i1).sum()
            got = compare(10 if n <= 3 else (12 if n == 4 else 16), V, c * h, (c + 1) * h)
            assert got <= 0
            planes[n] += 1
            if n <= 3:
                seen += 1
                walked += got < 0
    assert walked <= seen // 100
    assert size < 2 or planes[4:].all()
