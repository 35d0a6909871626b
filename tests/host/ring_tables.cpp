// Host-only driver of the ring schedules, for the CPU tests: builds a 3D plan's tables and rings and
// checks, per schedule, that the interpolation blocks hold every (column, node) pair of the tile lists
// once and that a node's weights over its entries add up to its whole kernel.  Prints per schedule
// "which entries faults error" (faults 0 when every index is consistent).
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <set>
#include <vector>

#include "../../paper_1504_02897_amd/csrc/ddi_internal.h"

using namespace ddi;

int main(int argc, char** argv) {
  if (argc != 9) return 2;
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
  p.nyquist_mask = 1;
  p.tol = std::atof(argv[7]);
  p.split = std::atoi(argv[8]);
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
    long faults = 0;
    std::set<std::pair<int, int>> tiles, mine;   // (column, node) pairs
    for (const SpreadItem& it : H.items)
      for (int i = 0; i < it.count; ++i) tiles.insert({it.tile / t.ntiles[2], H.list[it.start + i]});
    std::vector<double> sum(t.M, 0.0);
    std::vector<int> written(S.ent.size() / 2, 0);
    auto weights = [&](int q, int a, int d) {
      double s = 0.0;
      for (int i = 0; i < 8; ++i)
        if (d + i >= 0 && d + i < kWMax) s += t.wts[(q * 3L + a) * kWMax + d + i];
      return s;
    };
    std::vector<int> owner(S.interp.size(), 0);
    for (size_t x = 0; x + 1 < S.interp_cut.size(); ++x)
      for (int i = S.interp_cut[x]; i < S.interp_cut[x + 1]; ++i) owner[i]++;
    for (size_t b = 0; b < S.interp.size(); ++b) {
      const RingItem& it = S.interp[b];
      if (owner[b] != 1 || it.nref < 1 || it.nref > 16 || it.zs % 4 != 0 || 4 * it.ks > kRingSpan) ++faults;
      int pos = it.ent0;
      for (int r = 0; r < it.nref; ++r) {
        const RingRef& f = S.refs[it.ref0 + r];
        double sz = 0.0;
        for (int z = 0; z < 4 * it.ks; ++z) {
          const int d = it.zs + z - f.zr;
          if (d >= 0 && d < kWMax) sz += R.wz[f.ring * static_cast<size_t>(kWMax) + d];
        }
        if (f.zr < it.zs || f.ent != pos || f.count < 1) ++faults;
        for (int k = 0; k < f.count; ++k, ++pos) {
          const int q = S.ent[2 * pos], o = S.ent[2 * pos + 1];
          const int dx = (o & 255) - kOffBias, dy = ((o >> 8) & 255) - kOffBias;
          if ((o >> 16) != r) ++faults;
          if ((t.l0[3 * q + 2] - H.z0 + t.nf[2]) % t.nf[2] != f.zr) ++faults;
          if ((t.l0[3 * q] + dx - it.col / t.ntiles[1] * 8 + t.nf[0]) % t.nf[0] != 0) ++faults;
          if ((t.l0[3 * q + 1] + dy - it.col % t.ntiles[1] * 8 + t.nf[1]) % t.nf[1] != 0) ++faults;
          if (!mine.insert({it.col, q}).second) ++faults;
          written[pos]++;
          sum[q] += weights(q, 0, dx) * weights(q, 1, dy) * sz;
        }
      }
      if (pos != it.ent0 + it.nent) ++faults;
    }
    if (mine != tiles) ++faults;
    for (int w : written) faults += w != 1;
    double worst = 0.0;
    for (int64_t q = 0; q < t.M; ++q) {
      const bool used = which == kAll || t.half_factor[q] > 0.0;
      double whole = used ? 1.0 : 0.0;
      for (int a = 0; a < 3; ++a) {
        double s = 0.0;
        for (int i = 0; i < kWMax; ++i) s += t.wts[(q * 3 + a) * kWMax + i];
        whole *= s;
      }
      worst = std::fmax(worst, std::fabs(sum[q] - whole) / std::fmax(whole, 1.0));
      const int n = S.gptr[q + 1] - S.gptr[q];
      if (n > 9 || (used ? n < 1 : n != 0)) ++faults;
      for (int i = S.gptr[q]; i < S.gptr[q + 1]; ++i) faults += S.ent[2 * S.gpos[i]] != q || (i > S.gptr[q] && S.gpos[i] <= S.gpos[i - 1]);
    }
    std::printf("%d %zu %ld %.3e\n", which, mine.size(), faults, worst);
  }
  return 0;
}
