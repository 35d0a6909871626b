// Host-only driver of the ring schedules' blocks, for the CPU tests: builds a 3D plan's tables and rings
// and prints, per schedule, "which blocks longest full outside faults entries pairs": the number of interpolation blocks,
// the entries of the longest, how many rings have more entries over one column than a block takes, how
// many blocks reach beyond the last-axis window, and how many entries are not a (column, node) pair of
// the tile lists met once, at the right offsets, the number of entries and of (column, ring) pairs.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <set>

#include "../../paper_1504_02897_amd/csrc/ddi_internal.h"

using namespace ddi;

int main(int argc, char** argv) {
  if (argc != 10) return 2;
  ddi_params p{};
  p.dim = 3;
  for (int i = 0; i < 3; ++i) {
    p.n[i] = std::atoi(argv[1 + i]);
    p.L[i] = 8.0;
    p.stretch[i] = 1.0;
  }
  p.dip_n[2] = 1.0;
  p.n_rad = std::atoi(argv[4]);
  p.n_pol = std::atoi(argv[5]);
  p.n_azi = std::atoi(argv[6]);
  p.tol = std::atof(argv[7]);
  p.split = std::atoi(argv[8]);
  p.nyquist_mask = std::atoi(argv[9]);
  HostTables t;
  int st = 0;
  std::string err = build_tables(p, t, &st);
  RingTables R;
  if (err.empty()) err = build_rings(t, static_cast<int>(p.n_pol), R);
  if (!err.empty()) {
    std::printf("error %s\n", err.c_str());
    return 1;
  }
  for (int which = 0; which < 2; ++which) {
    const RingSchedule& S = R.sched[which];
    const Schedule& H = t.sched[which];
    int longest = 0, full = 0, outside = 0, faults = 0;
    std::set<std::pair<int, int>> tiles, mine;   // (column, node) pairs
    for (const SpreadItem& it : H.items)
      for (int i = 0; i < it.count; ++i) tiles.insert({it.tile / t.ntiles[2], H.list[it.start + i]});
    std::map<std::pair<int, int>, int> over;   // (column, ring) -> entries
    for (const RingItem& it : S.interp) {
      longest = std::max(longest, it.nent);
      if (H.nz < t.nf[2] && it.zs + 4 * it.ks > H.nz) ++outside;
      int pos = it.ent0;
      for (int r = 0; r < it.nref; ++r) {
        const RingRef& f = S.refs[it.ref0 + r];
        over[{it.col, f.ring}] += f.count;
        faults += f.ent != pos || f.zr < it.zs || f.zr + t.W[2] > it.zs + 4 * it.ks;
        for (int k = 0; k < f.count; ++k, ++pos) {
          const int q = S.ent[2 * pos], o = S.ent[2 * pos + 1];
          const int dx = (o & 255) - kOffBias, dy = ((o >> 8) & 255) - kOffBias;
          faults += (o >> 16) != r || !mine.insert({it.col, q}).second;
          faults += (t.l0[3 * q + 2] - H.z0 + t.nf[2]) % t.nf[2] != f.zr;
          faults += (t.l0[3 * q] + dx - it.col / t.ntiles[1] * 8 + t.nf[0]) % t.nf[0] != 0;
          faults += (t.l0[3 * q + 1] + dy - it.col % t.ntiles[1] * 8 + t.nf[1]) % t.nf[1] != 0;
        }
      }
      faults += pos != it.ent0 + it.nent;
    }
    faults += mine != tiles;
    for (const auto& o : over) full += o.second > kRingInterpEntries;
    std::printf("%d %zu %d %d %d %d %zu %zu\n", which, S.interp.size(), longest, full, outside, faults, mine.size(), over.size());
  }
  return 0;
}
