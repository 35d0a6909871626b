// FP64 interpolation of the 3D NUFFT on gfx950, by rings.
//
// The nodes of one (radial, polar) pair of the spherical rule share k_z and with it their weights
// along the last axis.  Per column of 8 x 8 fine-grid positions the last axis is therefore
// contracted once per ring, as FP64 matrix products over blocks of 16 rings,
//   G[ring][(x,y)] = sum_z wz_ring[z] F[(x,y)][z],
// and only the 8 x 8 plane that remains is weighted per node (w^2 instead of w^3 products),
//   partial_e = sum_(x,y) wx_e[x] wy_e[y] G[ring(e)][(x,y)],
// with one partial per (column, node) entry, summed per node by k_ring_gather.
// v_mfma_f64_16x16x4f64 takes A[i][k] from lane i + 16 k, B[k][j] from lane j + 16 k and leaves
// D[i][j] in lane j + 16 (i % 4), item i / 4.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "ddi_internal.h"
#include "wave.h"

namespace ddi {

using Cd = Complex<double>;
typedef double dbl4r __attribute__((ext_vector_type(4)));

// x + its value in the lane whose number differs by the DPP pattern (within eight lanes)
template <int CTRL>
__device__ __forceinline__ double dpp_add(double x) {
  const uint64_t u = __builtin_bit_cast(uint64_t, x);
  const int lo = __builtin_amdgcn_mov_dpp(static_cast<int>(u), CTRL, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_mov_dpp(static_cast<int>(u >> 32), CTRL, 0xF, 0xF, true);
  const uint64_t o = static_cast<uint32_t>(lo) | static_cast<uint64_t>(static_cast<uint32_t>(hi)) << 32;
  return x + __builtin_bit_cast(double, o);
}
// sum over aligned groups of eight lanes (every lane gets it): lane ^ 1, lane ^ 2, then 7 - lane
__device__ __forceinline__ double sum8(double x) {
  x = dpp_add<0xB1>(x);                      // quad_perm [1, 0, 3, 2]
  x = dpp_add<0x4E>(x);                      // quad_perm [2, 3, 0, 1]
  return dpp_add<0x141>(x);                  // row_half_mirror
}

// x of the lane at byte index b (4 x lane)
__device__ __forceinline__ double lane_get(int b, double x) {
  const uint64_t u = __builtin_bit_cast(uint64_t, x);
  const uint32_t lo = __builtin_amdgcn_ds_bpermute(b, static_cast<int>(u));
  const uint32_t hi = __builtin_amdgcn_ds_bpermute(b, static_cast<int>(u >> 32));
  return __builtin_bit_cast(double, lo | static_cast<uint64_t>(hi) << 32);
}

// Index of column position c = 8 x + y of a ring in the interpolation's plane buffer (rows of x
// padded by one value: the eight lanes of an entry read different banks).
constexpr int kGx = 9, kGring = 8 * kGx + 1;

constexpr int kRingKs = kRingSpan / 4;

// One workgroup (four waves) per block of up to 16 references of a column.  Bound by the latency of its
// dependent loads (block, references, weight rows) against six workgroups per CU, then by the grid reads
// (consecutive blocks of a column overlap: at 128^3 2.3 times the window for w = 14, 1.4 for w = 8, most of it
// from L2).  Measured with the gather at 128^3, w = 14, 138404 nodes: 88 + 9 us, against 142 + 20 us for whole
// 8 x 8 x 8 tiles contracted per (tile, node) entry (2.5 M entries and 2.47 M matrix products; here 0.90 M and
// 0.68 M); 32^3: 7 + 4 against 10 + 6; 96^3: 36 + 6 against 61 + 10.  A fixed set of workgroups stepping through
// the blocks with the next block's loads in flight needs twice the registers and took 106 us.  Wave v contracts
// the last axis for the column positions x = 2 v, 2 v + 1 (grid values loaded four lanes per 64-byte run and
// moved to the lanes of the matrix fragment), then the four waves share the block's entries, eight lanes each
// (lane u takes the row x = u).
__global__ void __launch_bounds__(256, 6) k_ring_interp(const Cd* __restrict__ F, const double* __restrict__ rows,
                                                      int stride, const double* __restrict__ wz,
                                                      const int4* __restrict__ refs, const RingItem* __restrict__ items,
                                                      const int2* __restrict__ ent, int nf1, int nf2, int nt1, int z0,
                                                      Cd* __restrict__ part) {
  constexpr int AS = kRingSpan + 1;
  __shared__ double wa[16 * AS];
  __shared__ Cd G[16 * kGring];
  __shared__ double wyl[4][64];
  const RingItem it = items[blockIdx.x];
  if (it.nref == 0) return;                  // padding item
  const int lane = threadIdx.x & 63, v = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int k = lane >> 4, j = lane & 15;
  const int e8 = lane >> 3, u = lane & 7;
  const int lr = lane >> 2, lk = lane & 3;   // grid loads: position lr of the wave's 16
  const int from = 4 * (4 * j + k);          // byte index of the lane that loads position j, place k
  auto load_ent = [&](int e) { e += 8 * v + e8; return ent[it.ent0 + (e < it.nent ? e : it.nent - 1)]; };
  auto load_w = [&](int2 r, double& x, double& y) {
    const int dx = (r.y & 255) - kOffBias + u, dy = ((r.y >> 8) & 255) - kOffBias + u;
    const double* row = rows + static_cast<int64_t>(r.x) * stride;
    x = static_cast<unsigned>(dx) < kWMax ? row[dx] : 0.0;
    y = static_cast<unsigned>(dy) < kWMax ? row[kWMax + dy] : 0.0;
  };
  int2 rec = load_ent(0), rec1 = load_ent(32);
  // the block's grid values at the wave's 16 positions; a block never reaches past the window (both end
  // on multiples of four positions), so all of them were written by the transforms
  Cd f[kRingKs];
  {
    const Cd* row = F + (static_cast<int64_t>(it.col / nt1 * 8 + 2 * v + (lr >> 3)) * nf1 + (it.col % nt1 * 8 + (lr & 7))) * nf2;
    int zb = z0 + it.zs;
    if (zb >= nf2) zb -= nf2;
    if (zb + 4 * it.ks <= nf2) {
      row += zb + lk;
#pragma unroll
      for (int s = 0; s < kRingKs; ++s) {
        if (s >= it.ks) break;
        f[s] = row[4 * s];
      }
    } else {                                 // round the end of the axis (at most twice: 32 positions, nf2 >= 16)
#pragma unroll
      for (int s = 0; s < kRingKs; ++s) {
        if (s >= it.ks) break;
        int z = zb + 4 * s + lk;
        if (z >= nf2) z -= nf2;
        if (z >= nf2) z -= nf2;
        f[s] = row[z];
      }
    }
  }
  // the rings' weights over the block, zero outside their supports
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    const int n = (threadIdx.x >> 5) + 8 * r, z = threadIdx.x & 31;
    const int4 ref = refs[it.ref0 + (n < it.nref ? n : 0)];
    const int d = it.zs + z - ref.y;
    wa[n * AS + z] = n < it.nref && static_cast<unsigned>(d) < kWMax ? wz[static_cast<int64_t>(ref.x) * kWMax + d] : 0.0;
  }
  double wx, wy;
  load_w(rec, wx, wy);
  __syncthreads();
  dbl4r re = {0.0, 0.0, 0.0, 0.0}, im = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int s = 0; s < kRingKs; ++s) {
    if (s < it.ks) {
      const double a = wa[j * AS + 4 * s + k];
      re = __builtin_amdgcn_mfma_f64_16x16x4f64(a, lane_get(from, f[s].re), re, 0, 0, 0);
      im = __builtin_amdgcn_mfma_f64_16x16x4f64(a, lane_get(from, f[s].im), im, 0, 0, 0);
    }
  }
#pragma unroll
  for (int t = 0; t < 4; ++t) G[(4 * t + k) * kGring + (2 * v + (j >> 3)) * kGx + (j & 7)] = Cd{re[t], im[t]};
  __syncthreads();
  for (int e0 = 0; e0 < it.nent; e0 += 32) {
    const Cd* g = G + ((rec.y >> 16) & 15) * kGring + u * kGx;
    const double wxc = wx;
    wyl[v][lane] = wy;
    rec = rec1;
    if (e0 + 32 < it.nent) load_w(rec, wx, wy);          // the next round's weights
    if (e0 + 64 < it.nent) rec1 = load_ent(e0 + 64);
    lds_sync_wave();
    const double* wyr = wyl[v] + e8 * 8;
    double sr = 0.0, si = 0.0;
#pragma unroll
    for (int y = 0; y < 8; ++y) {
      const Cd p = g[y];
      sr += wyr[y] * p.re;
      si += wyr[y] * p.im;
    }
    sr = sum8(sr * wxc);
    si = sum8(si * wxc);
    const int e = e0 + 8 * v + e8;
    if (u < 2 && e < it.nent) reinterpret_cast<double*>(part + (static_cast<int64_t>(it.ent0) + e))[u] = u == 0 ? sr : si;
    lds_sync_wave();
  }
}

// Sum the partials of each node (in list order) and apply the node scale.
__global__ void __launch_bounds__(256) k_ring_gather(const Cd* __restrict__ part,
                                                      const int32_t* __restrict__ gptr,
                                                      const int32_t* __restrict__ gpos, int64_t M,
                                                      const double* __restrict__ scale, double sscalar,
                                                      Cd* __restrict__ out) {
  const int64_t q = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (q >= M) return;
  const int b = gptr[q], n = gptr[q + 1] - b;
  if (n <= 0) return;                        // node outside the scheduled set
  // a node meets at most 3 x 3 columns: all its partials in flight at once, summed in list order
  constexpr int NP = 9;
  int pos[NP];
#pragma unroll
  for (int i = 0; i < NP; ++i) pos[i] = gpos[b + (i < n ? i : 0)];
  Cd p[NP];
#pragma unroll
  for (int i = 0; i < NP; ++i) p[i] = part[pos[i]];
  double sr = 0.0, si = 0.0;
#pragma unroll
  for (int i = 0; i < NP; ++i) {
    if (i < n) {
      sr += p[i].re;
      si += p[i].im;
    }
  }
  const double s = scale ? scale[q] * sscalar : sscalar;
  out[q] = Cd{s * sr, s * si};
}

hipError_t ring_interp(DevicePlan& P, int which, Cd* out, const double* scale, double sscalar, hipStream_t s) {
  const HostTables& H = P.H;
  const DevicePlan::DevRings& D = P.drings[which];
  Cd* part = reinterpret_cast<Cd*>(P.ipartial);
  // the weight rows of axes 0 and 1: the spread's where the plan has them, which then finds them in the
  // Infinity Cache (with a copy of the two axes for this kernel alone the spread at 128^3 took 143 us
  // instead of 139 at w = 14, 99 instead of 94 at w = 8), else a copy: the node records of 400 bytes
  // straddle cache lines (16^3, 6.1 M nodes, w = 14: 1283 us against 991)
  const double* rows = reinterpret_cast<const double*>(P.pads ? P.pads : P.xyw);
  const int stride = P.pads ? 3 * kRowLen : 2 * kWMax;
  if (D.ninterp > 0) {
    hipLaunchKernelGGL(k_ring_interp, dim3(D.ninterp), dim3(256), 0, s, reinterpret_cast<const Cd*>(P.fine), rows,
                       stride, P.ring_wz, reinterpret_cast<const int4*>(D.refs), D.interp,
                       reinterpret_cast<const int2*>(D.ent), H.nf[1], H.nf[2], H.ntiles[1], H.sched[which].z0,
                       part);
    DDI_CHECK(hipGetLastError());
  }
  const int blocks = static_cast<int>((H.M + 255) / 256);
  hipLaunchKernelGGL(k_ring_gather, dim3(blocks), dim3(256), 0, s, part, D.gptr, D.gpos, H.M, scale, sscalar, out);
  return hipGetLastError();
}

}  // namespace ddi
