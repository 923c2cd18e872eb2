"""Combinatorics of clipping a tetrahedron by up to three planes, as tables.

A clipped piece is a graph of vertex slots (geometry.hpp): a plane keeps the
vertices with distance >= 0, puts a new vertex on every edge cut and closes
the face between them.  Which edges are cut, which slots the new vertices
take, the graph that results and the fan of sub-tetrahedra it gives depend on
the graph before and on the set of vertices outside, not on coordinates.
From a tetrahedron three planes lead to fewer than 30,000 graphs, so all of
it is looked up: this module runs the clip of geometry.hpp on the slots alone
and writes one record per (graph, outside set).

  python gen_clip_table.py FILE     writes the C initialisers

A set whose inside or outside is not connected has no record (count 0): a
plane does not cut a convex piece that way, except by rounding where vertices
coincide, and such a piece is left to the graph walk.
"""
import sys

SLOTS = 10                      # 4 vertices and 2 more for every plane
WIDTH = (4, 6, 8)               # slots in use before plane 1, 2, 3
NO_BASE = (1 << 18) - 1


def _find(w, x):
    return 0 if w[0] == x else (1 if w[1] == x else 2)


def clip(live, nb, out):
    """(live, neighbours, cuts) after a plane with the slots `out` outside;
    cuts: (u, v, w), u outside, v inside, w the new vertex's slot."""
    nb = [list(x) if x else None for x in nb]
    inside = live & ~out
    adj = [u for u in range(SLOTS) if out >> u & 1 and any(inside >> k & 1 for k in nb[u])]
    free = [w for w in range(SLOTS) if not live >> w & 1 or (out >> w & 1 and w not in adj)]
    cuts, new = [], 0
    for u in adj:
        first = True
        for v in list(nb[u]):
            if not inside >> v & 1:
                continue
            if first:
                w, first = u, False
            else:
                w = free.pop(0)
                nb[v][_find(nb[v], u)] = w
            nb[w] = [v, v, v]
            new |= 1 << w
            cuts.append((u, v, w))
    for w in range(SLOTS):
        if new >> w & 1:
            cur, nxt = w, nb[w][0]
            while True:
                k = _find(nb[nxt], cur)
                cur, nxt = nxt, nb[nxt][(k + 1) % 3]
                if new >> cur & 1:
                    break
            nb[w][2], nb[cur][1] = cur, w
    live = inside | new
    return live, tuple(tuple(nb[v]) if live >> v & 1 else None for v in range(SLOTS)), cuts


def connected(mask, nb):
    seen = mask & -mask
    todo = [seen.bit_length() - 1] if mask else []
    while todo:
        for b in nb[todo.pop()]:
            if mask >> b & 1 and not seen >> b & 1:
                seen |= 1 << b
                todo.append(b)
    return seen == mask


def fan(live, nb):
    """(v, f1, f2) of the fan's sub-tetrahedra (with the apex, the lowest
    slot) in the order the walk of geometry.hpp gives them."""
    apex = (live & -live).bit_length() - 1
    seen, out = set(), []
    for v in [apex] + [v for v in range(SLOTS) if live >> v & 1 and v != apex]:
        for k in range(3):
            if (v, k) in seen:
                continue
            seen.add((v, k))
            prev, f1 = v, nb[v][k]
            while True:
                j = (_find(nb[f1], prev) + 1) % 3
                seen.add((f1, j))
                f2 = nb[f1][j]
                if f2 == v:
                    break
                if v != apex:
                    out.append((v, f1, f2))
                prev, f1 = f1, f2
    return out


def tables():
    """(cut records, fan records, graph records), 128 bits each."""
    tet = (0xF, ((1, 3, 2), (2, 3, 0), (0, 3, 1), (1, 2, 0)) + (None,) * 6)
    states, base, level = {tet: 0}, [0], [tet]
    cuts, rows = {}, 1 << WIDTH[0]
    for width in WIDTH:
        after = []
        last = width == WIDTH[-1]
        for live, nb in level:
            b = base[states[live, nb]]
            for out in range(1, 1 << width):
                if out & ~live or out == live:
                    continue
                if not connected(out, nb) or not connected(live & ~out, nb):
                    continue
                l2, n2, c = clip(live, nb, out)
                if (l2, n2) not in states:
                    states[l2, n2] = len(states)
                    after.append((l2, n2))
                    if last:
                        base.append(NO_BASE)
                    else:
                        base.append(rows)
                        rows += 1 << WIDTH[WIDTH.index(width) + 1]
                s = states[l2, n2]
                # a cut that reuses u's slot comes after the others of u, so
                # that u is still there for them
                c = sorted(c, key=lambda x: (x[0], x[0] == x[2]))
                assert len(c) <= 6 and s < 1 << 17 and (last or l2 >> WIDTH[-1] == 0)
                r = 0
                for i, (u, v, w) in enumerate(c):
                    r |= (u | v << 4 | w << 8) << (12 * i)
                cuts[b + out] = (r | len(c) << 72 | l2 << 75 | s << 85 | base[s] << 102)
        level = after
    fans, graphs = [], []
    for live, nb in states:
        f = fan(live, nb)
        assert len(f) <= 10
        r = len(f)
        for i, (v, f1, f2) in enumerate(f):
            r |= (v | f1 << 4 | f2 << 8) << (4 + 12 * i)
        fans.append(r)
        graphs.append(sum((w[0] | w[1] << 4 | w[2] << 8) << (12 * v)
                          for v, w in enumerate(nb) if w))
    return [cuts.get(i, 0) for i in range(rows)], fans, graphs


def write(path):
    with open(path, "w") as fh:
        for name, rec in zip(("kCutRecords", "kFanRecords", "kGraphRecords"), tables()):
            fh.write(f"__device__ uint4 {name}[{len(rec)}] = {{\n")
            for r in rec:
                fh.write("{" + ",".join(hex(r >> 32 * k & 0xFFFFFFFF) for k in range(4)) + "},\n")
            fh.write("};\n")


if __name__ == "__main__":
    write(sys.argv[1])
