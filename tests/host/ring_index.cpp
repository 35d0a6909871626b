// Host-only driver, for the CPU tests: the rings of four nodes at the far ends of the largest rule that a
// plan takes (65536 x 65536 radial and polar nodes).  Prints the rings' number and each node's ring; the
// test runs it with little memory.
#include <cstdio>

#include "../../paper_1504_02897_amd/csrc/ddi_internal.h"

using namespace ddi;

int main() {
  HostTables t;
  t.M = 4;
  t.index = {65535, 65535, 0, 0, 65535, 0, 65535, 0, 0, 0, 65535, 1};
  for (int a = 0; a < 3; ++a) {
    t.N[a] = 32;
    t.nf[a] = 64;
    t.W[a] = 4;
    t.ntiles[a] = 8;
  }
  t.l0 = {1, 1, 1, 9, 9, 2, 17, 17, 3, 25, 25, 2};
  t.half_factor.assign(4, 1.0);
  t.wts.assign(4 * 3 * kWMax, 0.5);
  for (Schedule& S : t.sched) S.nz = 64;
  RingTables R;
  const std::string err = build_rings(t, 65536, R);
  if (!err.empty()) {
    std::printf("error %s\n", err.c_str());
    return 1;
  }
  std::printf("%zu", R.wz.size() / kWMax);
  int ring[4] = {-1, -1, -1, -1};
  for (const RingRef& f : R.sched[kAll].refs)
    for (int k = 0; k < f.count; ++k) ring[R.sched[kAll].ent[2 * (f.ent + k)]] = f.ring;
  for (int r : ring) std::printf(" %d", r);
  std::printf("\n");
  return 0;
}
