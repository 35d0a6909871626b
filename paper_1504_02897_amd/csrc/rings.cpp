// Plan-time ring schedules of the FP64 3D interpolation (host).
//
// The nodes of one (radial, polar) pair of the spherical rule, a ring, share k_z, and with it the
// support origin and the kernel weights along the last axis.  The kernels therefore contract the
// last axis once per ring instead of once per node: the fine grid is cut into columns of 8 x 8
// positions on the first two axes, every column lists the rings with a node over it (by their
// last-axis origin), and each such ring reference lists its nodes over the column.
#include <algorithm>
#include <cstdint>

#include "ddi_internal.h"

namespace ddi {

namespace {

// Work of an item in units of one node entry: a ring reference costs the matrix products of its
// column, about four entries' worth.
int64_t work_of(const RingItem& it) { return it.nent + 4 * static_cast<int64_t>(it.nref) + 16; }

// Puts the items in Morton order of (column, block) and cuts the list into one region per XCD: an XCD works in
// one compact region, front to back, and its L2 keeps the weight rows and grid rows that neighbouring items share.
std::vector<int32_t> order_items(std::vector<RingItem>& items, int nt1) {
  std::vector<std::pair<uint64_t, int32_t>> key(items.size());
  for (size_t i = 0; i < items.size(); ++i) {
    const RingItem& it = items[i];
    key[i] = {morton3(it.col / nt1, it.col % nt1, it.zs / 8), static_cast<int32_t>(i)};
  }
  std::sort(key.begin(), key.end());
  std::vector<RingItem> out(items.size());
  int64_t total = 0;
  for (size_t i = 0; i < items.size(); ++i) {
    out[i] = items[key[i].second];
    total += work_of(out[i]);
  }
  items.swap(out);
  std::vector<int32_t> cut = xcd_cuts(items, work_of);
  // the items far above the mean (the columns around k = 0 hold whole rings) go first in a region
  const int64_t heavy = 2 * total / std::max<int64_t>(1, static_cast<int64_t>(items.size()));
  for (int x = 0; x < kXcds; ++x) {
    const auto b = items.begin() + cut[x], e = items.begin() + cut[x + 1];
    const auto m = std::stable_partition(b, e, [&](const RingItem& it) { return work_of(it) > heavy; });
    std::stable_sort(b, m, [](const RingItem& p, const RingItem& q) { return work_of(p) > work_of(q); });
  }
  return cut;
}

std::string build_one(const HostTables& t, const std::vector<int32_t>& order, const std::vector<int32_t>& rstart,
                      const std::vector<int32_t>& rnode, bool half, const Schedule& S, RingSchedule& R) {
  const int nt0 = t.ntiles[0], nt1 = t.ntiles[1], ncol = nt0 * nt1;
  const int nf2 = t.nf[2], w = t.W[2];
  auto rel = [&](int l0) { const int d = l0 - S.z0; return d < 0 ? d + nf2 : d; };
  // rings in the order of their last-axis origin relative to the window
  std::vector<int32_t> byz(order);
  auto zr_of = [&](int r) { return rel(t.l0[3 * static_cast<int64_t>(rnode[rstart[r]]) + 2]); };
  std::stable_sort(byz.begin(), byz.end(), [&](int a, int b) { return zr_of(a) < zr_of(b); });
  // tiles met by a support on axis a (at most three: w <= 16 < 2 tiles + 1)
  auto tiles = [&](int l0, int a, int* out) {
    const int first = l0 / 8, last = (l0 + t.W[a] - 1) / 8;
    int c = 0;
    for (int i = first; i <= last; ++i) out[c++] = i % t.ntiles[a];
    return c;
  };
  // A ring with more than `most` entries over a column (rules with many azimuthal nodes) gets several
  // references: kRingInterpEntries, or more where blocks of that length would outnumber kRingBlocks
  int64_t total = 0;
  for (int r : byz)
    for (int i = rstart[r]; i < rstart[r + 1]; ++i) {
      const int64_t q = rnode[i];
      if (half && !(t.half_factor[q] > 0.0)) continue;
      total += ((t.l0[3 * q] % 8 + t.W[0] + 7) / 8) * ((t.l0[3 * q + 1] % 8 + t.W[1] + 7) / 8);
    }
  const int most = static_cast<int>(std::clamp<int64_t>(total / kRingBlocks, kRingInterpEntries, kRingMaxEntries));
  // pass 0 counts, pass 1 fills: references and entries per column
  std::vector<int64_t> nref(ncol + 1, 0), nent(ncol + 1, 0);
  std::vector<int32_t> seen(ncol, -1), held(ncol, 0);   // last ring over the column, entries of its reference
  R.col_ref.assign(ncol + 1, 0);
  std::vector<int64_t> fref, fent;
  int stamp = 0;
  for (int pass = 0; pass < 2; ++pass) {
    if (pass == 1) {
      int64_t cr = 0, ce = 0;
      for (int c = 0; c <= ncol; ++c) {
        const int64_t a = nref[c], b = nent[c];
        nref[c] = cr;
        nent[c] = ce;
        cr += a;
        ce += b;
      }
      if (ce > (int64_t(1) << 30) || cr > (int64_t(1) << 30)) return "ring schedule too large";
      R.refs.assign(cr, RingRef{});
      R.ent.assign(2 * ce, 0);
      fref.assign(nref.begin(), nref.end());
      fent.assign(nent.begin(), nent.end());
    }
    for (int r : byz) {
      const int zr = zr_of(r);
      ++stamp;
      for (int i = rstart[r]; i < rstart[r + 1]; ++i) {
        const int64_t q = rnode[i];
        if (half && !(t.half_factor[q] > 0.0)) continue;
        int tx[4], ty[4];
        const int l0x = t.l0[3 * q], l0y = t.l0[3 * q + 1];
        const int nx = tiles(l0x, 0, tx), ny = tiles(l0y, 1, ty);
        for (int a = 0; a < nx; ++a)
          for (int b = 0; b < ny; ++b) {
            const int c = tx[a] * nt1 + ty[b];
            const bool fresh = seen[c] != stamp || held[c] == most;
            if (fresh) {
              seen[c] = stamp;
              held[c] = 0;
            }
            ++held[c];
            if (pass == 0) {
              nref[c] += fresh;
              nent[c]++;
              continue;
            }
            if (fresh) R.refs[fref[c]++] = RingRef{r, zr, static_cast<int32_t>(fent[c]), 0};
            R.refs[fref[c] - 1].count++;
            auto off = [&](int org, int l0, int ax) {
              int d = org - l0;
              if (d < 0) d += t.nf[ax];
              if (d > t.nf[ax] - 8) d -= t.nf[ax];     // the column starts before the support
              return d;
            };
            const int dx = off(tx[a] * 8, l0x, 0), dy = off(ty[b] * 8, l0y, 1);
            if (dx < -7 || dx >= t.W[0] || dy < -7 || dy >= t.W[1]) return "ring entry outside its weight row";
            R.ent[2 * fent[c]] = static_cast<int32_t>(q);
            R.ent[2 * fent[c] + 1] = (kOffBias + dx) | (kOffBias + dy) << 8;
            fent[c]++;
          }
      }
    }
  }
  for (int c = 0; c <= ncol; ++c) R.col_ref[c] = static_cast<int32_t>(nref[c]);
  // interpolation items: up to 16 references of a column whose last-axis supports span at most
  // kRingSpan positions, with up to kRingInterpEntries entries (or one longer reference); the block
  // starts on a multiple of four positions (64 bytes of the grid)
  R.interp.clear();
  for (int c = 0; c < ncol; ++c) {
    int i = R.col_ref[c];
    const int e = R.col_ref[c + 1];
    while (i < e) {
      RingItem it{};
      it.col = c;
      it.ref0 = i;
      it.zs = R.refs[i].zr & ~3;
      it.ent0 = R.refs[i].ent;
      int n = 0;
      while (i < e && n < 16 && R.refs[i].zr + w - it.zs <= kRingSpan &&
             (n == 0 || it.nent + R.refs[i].count <= kRingInterpEntries)) {
        for (int k = 0; k < R.refs[i].count; ++k) R.ent[2 * (R.refs[i].ent + k) + 1] |= n << 16;
        it.nent += R.refs[i].count;
        it.ks = (R.refs[i].zr + w - it.zs + 3) / 4;
        ++n;
        ++i;
      }
      it.nref = n;
      R.interp.push_back(it);
    }
  }
  R.interp_cut = order_items(R.interp, nt1);
  // per node, the positions of its entries (in column order)
  entry_positions(R.ent.data(), 2, R.ent.size() / 2, t.M, R.gptr, R.gpos);
  return "";
}

}  // namespace

std::string build_rings(const HostTables& t, int npol, RingTables& out) {
  const int64_t M = t.M;
  int nrad = 0;
  for (int64_t q = 0; q < M; ++q) nrad = std::max(nrad, t.index[3 * q] + 1);
  // nodes by ring, plan order inside a ring: two counting sorts, by polar, then by radial index (a table
  // over all pairs would need memory for rings without a node)
  std::vector<int32_t> rnode(M), other(M);
  for (int64_t q = 0; q < M; ++q) other[q] = static_cast<int32_t>(q);
  for (int a : {1, 0}) {
    const std::vector<int32_t>& from = a == 1 ? other : rnode;
    std::vector<int32_t>& to = a == 1 ? rnode : other;
    std::vector<int32_t> start((a == 1 ? npol : nrad) + 1, 0);
    for (int64_t q = 0; q < M; ++q) start[t.index[3 * q + a] + 1]++;
    for (size_t i = 1; i < start.size(); ++i) start[i] += start[i - 1];
    for (int32_t q : from) to[start[t.index[3 * static_cast<int64_t>(q) + a]]++] = q;
  }
  rnode.swap(other);
  auto id = [&](int32_t q) { return std::make_pair(t.index[3 * static_cast<int64_t>(q)], t.index[3 * static_cast<int64_t>(q) + 1]); };
  std::vector<int32_t> rstart;               // the rings that hold a node
  for (int64_t i = 0; i < M; ++i)
    if (i == 0 || id(rnode[i]) != id(rnode[i - 1])) rstart.push_back(static_cast<int32_t>(i));
  const int nring = static_cast<int>(rstart.size());
  rstart.push_back(static_cast<int32_t>(M));
  out.wz.assign(static_cast<size_t>(nring) * kWMax, 0.0);
  for (int r = 0; r < nring; ++r) {
    const int64_t q0 = rnode[rstart[r]];
    for (int i = 0; i < kWMax; ++i) out.wz[static_cast<size_t>(r) * kWMax + i] = t.wts[(q0 * 3 + 2) * kWMax + i];
    for (int i = rstart[r]; i < rstart[r + 1]; ++i)
      if (t.l0[3 * static_cast<int64_t>(rnode[i]) + 2] != t.l0[3 * q0 + 2]) return "internal: a ring with two last-axis origins";
  }
  std::vector<int32_t> order(nring);
  for (int r = 0; r < nring; ++r) order[r] = r;
  for (int which = 0; which < 2; ++which) {
    std::string err = build_one(t, order, rstart, rnode, which == kHalf, t.sched[which], out.sched[which]);
    if (!err.empty()) return err;
  }
  return "";
}

}  // namespace ddi
