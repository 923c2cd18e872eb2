"""The clip by look-up (csrc/gen_clip_table.py, table_clip_box) against the
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
// -1: no record; 0: equal; 1: not equal
extern "C" int compare(const double* V, const double* lo, const double* hi, const void* cut,
                       const void* fan) {
  const ClipTables tab{static_cast<const uint4*>(cut), static_cast<const uint4*>(fan), nullptr};
  static Box A, B;
  const PolyView P{A.x, A.y, A.z, A.nb, 1, (1u << 10) - 1u};
  const PolyView Q{B.x, B.y, B.z, B.nb, 1, (1u << 10) - 1u};
  TetGeom G;
  for (int k = 0; k < 4; ++k)
    for (int e = 0; e < 3; ++e) G.V[k][e] = V[3 * k + e];
  tet_geom(G);
  ClipCount ca, cb;
  uint32_t live = poly_init_tet(P, G.V, G.det < 0.0);
  if (!poly_clip_box<10>(P, live, lo, hi, G.mn, G.mx, &ca)) return 1;
  TablePiece q;
  poly_put_tet(Q, G.V, G.det < 0.0);
  table_clip_box(Q, q, tab, lo, hi, G.mn, G.mx, &cb);
  if (q.odd) return -1;
  if (q.live != live || ca.planes != cb.planes || ca.dist != cb.dist || ca.cuts != cb.cuts) return 1;
  if (!live) return 0;
  static double ra[16][12], rb[16][12];
  double va = 0.0, vb = 0.0;
  int na = 0, nb = 0;
  EdgeMask<10> seen;
  if (poly_fan_prepare<10>(P, live, seen) < 0) return 1;
  if (!emit_subtets<double, 10>(P, live, seen, lo, hi,
        [&](int k, const double(&r)[kRecord]) { std::memcpy(ra[k], r, sizeof(r)); }, va, na))
    return 1;
  emit_subtets_table<double>(Q, q.live, tab.fan[q.graph], lo, hi,
        [&](int k, const double(&r)[kRecord]) { std::memcpy(rb[k], r, sizeof(r)); nb = k + 1; }, vb);
  return na == nb && va == vb && !std::memcmp(ra, rb, size_t(na) * sizeof(ra[0])) ? 0 : 1;
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
    cut, fan = [np.array([[r >> 32 * k & 0xFFFFFFFF for k in range(4)] for r in t], dtype=np.uint32)
                for t in gen.tables()[:2]]
    d = tmp_path_factory.mktemp("clip")
    src, so = str(d / "clip.hip"), str(d / "clip.so")
    with open(src, "w") as fh:
        fh.write(HOST)
    subprocess.run([hipcc, "-x", "hip", "--offload-host-only", "-O1", "-ffp-contract=off",
                    "-std=c++17", "-fPIC", "-shared", "-I", CSRC, src, "-o", so], check=True,
                   capture_output=True)
    lib = ctypes.CDLL(so)

    def call(V, lo, hi):
        a = [np.ascontiguousarray(x, dtype=np.float64) for x in (V, lo, hi)] + [cut, fan]
        return lib.compare(*[ctypes.c_void_p(x.ctypes.data) for x in a])
    return call


@pytest.mark.parametrize("size,snap", [(0.6, 0.0), (1.3, 0.0), (1.3, 0.5), (2.5, 0.3), (2.5, 0.8)])
def test_table_clip_equals_graph_walk(compare, size, snap):
    """Random tets, some of their coordinates in cell planes, in every cell of
    their box that at most three planes bound for them."""
    rng = np.random.default_rng(int(10 * size + 100 * snap))
    h, seen, missing = 1.0 / 32, 0, 0
    while seen < 4000:
        V = (rng.random((4, 3)) * size + 8) * h
        V = np.where(rng.random((4, 3)) < snap, np.round(2 * V / h) / 2 * h, V)
        if abs(np.linalg.det(V[1:] - V[0])) < 1e-12:
            continue
        i0 = np.floor(V.min(0) / h).astype(int)
        i1 = np.maximum(np.ceil(V.max(0) / h).astype(int) - 1, i0)
        for c in np.ndindex(*(i1 - i0 + 1)):
            c = i0 + np.array(c)
            if (c > i0).sum() + (c < i1).sum() > 3:
                continue
            got = compare(V, c * h, (c + 1) * h)
            assert got <= 0
            seen += 1
            missing += got < 0
    assert missing <= seen // 100
