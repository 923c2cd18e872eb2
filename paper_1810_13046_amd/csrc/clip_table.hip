// The clip tables (gen_clip_table.py writes the initialisers when the library
// is built) and their device addresses.
#include "geometry.hpp"
#include "internal.hpp"

namespace ibvt {

#include "clip_table.inc"

int clip_tables(ClipTables& t) {
  void *c = nullptr, *f = nullptr, *g = nullptr;
  int st;
  if ((st = hip_check(hipGetSymbolAddress(&c, HIP_SYMBOL(kCutRecords)), "clip tables")) ||
      (st = hip_check(hipGetSymbolAddress(&f, HIP_SYMBOL(kFanRecords)), "clip tables")) ||
      (st = hip_check(hipGetSymbolAddress(&g, HIP_SYMBOL(kGraphRecords)), "clip tables")))
    return st;
  t.cut = static_cast<const uint4*>(c);
  t.fan = static_cast<const uint4*>(f);
  t.graph = static_cast<const uint4*>(g);
  return IBVT_OK;
}

}  // namespace ibvt
