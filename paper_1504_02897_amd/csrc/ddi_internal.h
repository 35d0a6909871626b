// Internal declarations shared by the plan builder, the kernels and the C ABI.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <string>
#include <vector>

#include "../../include/ddi.h"

namespace ddi {

constexpr int kWMax = 16;          // largest kernel width
constexpr int kTwSlots = 20;       // twiddle tables: lengths 2^0..2^10 and 3 * 2^0..3 * 2^8
constexpr int kTileZ = 8;          // spread tile extent along the last axis (registers per lane)
#ifndef DDI_INTERP_BLOCK3
#define DDI_INTERP_BLOCK3 4
#endif
#ifndef DDI_INTERP_MIN_GROUP
#define DDI_INTERP_MIN_GROUP 6
#endif
// interpolation groups: block of cells per axis (3D) and smallest group staged in LDS
constexpr int kInterpBlock3 = DDI_INTERP_BLOCK3;
constexpr int kInterpMinGroup = DDI_INTERP_MIN_GROUP;
#ifndef DDI_SPREAD_BATCH
#define DDI_SPREAD_BATCH 64
#endif
// spread: nodes staged in LDS per batch (LDS per wave ~ batch * 26 values)
constexpr int kSpreadBatch = DDI_SPREAD_BATCH;
#ifndef DDI_SPREAD_CHUNK
#define DDI_SPREAD_CHUNK 256
#endif
#ifndef DDI_SPREAD_CHUNK_MFMA
#define DDI_SPREAD_CHUNK_MFMA 512
#endif
// spread: a tile with more nodes is split into chunks of this many (partial tiles + reduce);
// the matrix-core kernels take longer chunks (cheaper per node)
constexpr int kSpreadChunk = DDI_SPREAD_CHUNK;
#ifndef DDI_SPREAD_CHUNK_2D
#define DDI_SPREAD_CHUNK_2D 32
#endif
// shortest chunk of the 2D spread (hot tiles are split into chunks of at least this many nodes)
constexpr int kSpreadChunk2d = DDI_SPREAD_CHUNK_2D;
constexpr int kSpreadChunkMfma = DDI_SPREAD_CHUNK_MFMA;
#ifndef DDI_SPREAD_WAVES
#define DDI_SPREAD_WAVES 4096
#endif
// matrix-core chunks are shortened until the entries fill about this many items (resident waves)
constexpr int kSpreadWaves = DDI_SPREAD_WAVES;
#ifndef DDI_SPREAD_XCD_ORDER
#define DDI_SPREAD_XCD_ORDER 1
#endif
#ifndef DDI_SPREAD_UNROLL
#define DDI_SPREAD_UNROLL 4
#endif
constexpr int kRowLen = kWMax;    // weight row of the matrix-core kernels: w weights, then zeros
constexpr int kOffBias = 8;       // entry offsets are stored biased by this (non-negative bytes)
constexpr int kEntPad = 32;       // zero entries after the last one (blocks of 16 may read past an item)
#ifndef DDI_SPREAD_MFMA
#define DDI_SPREAD_MFMA 1
#endif
// spread on the matrix cores where the plan has row windows
constexpr bool kSpreadMfma = DDI_SPREAD_MFMA != 0;


// One quadrature node as seen by the spread / interpolation kernels: the first
// fine-grid index of its support on each axis (already reduced mod n_fine) and
// the separable kernel weights psi(l0 + i - tau) for i < w on each axis.
template <typename T>
struct alignas(16) NodeRec {
  int32_t l0[3];
  int32_t pad;
  T w[3][kWMax];
};

// A unit of spread work: the nodes list[start, start+count) are summed into
// the tile `tile`; slot < 0 writes the tile directly, otherwise a partial
// tile is written to partial slot `slot` and summed by a reduce item.
struct SpreadItem {
  int32_t tile;
  int32_t start;
  int32_t count;
  int32_t slot;
};

// A group of nodes (plan-order range) whose supports start in one block of ib^3
// cells; their supports lie in the region org + [0, ireg) (mod n_fine), staged in LDS.
struct InterpItem {
  int32_t start;
  int32_t count;
  int32_t org[3];
  int32_t pad[3];
};

struct ReduceItem {
  int32_t tile;
  int32_t first_slot;
  int32_t nslots;
  int32_t pad;
};

// Ring schedule of the FP64 3D interpolation (rings.cpp, rings.hip).
constexpr int kRingSpan = 32;      // last-axis positions that one interpolation block covers
// Entries of an interpolation block: its rounds of 32 run one after the other, and the blocks around k = 0
// would last far longer than the others (32^3: 12.5 us with 512, 7.1 with 128).  A ring with more nodes over
// a column is cut into several references (32^3, w = 4, a 4 x 4 x 4096 rule, with the gather: 12 us, 67 with
// whole rings), except where the entries make kRingBlocks longer blocks, which fill the chip several times
// over: there a cut only repeats the ring's contraction (16^3, 6.1 M nodes, w = 14: 1157 us, 994 whole).
constexpr int kRingInterpEntries = 128;
constexpr int kRingMaxEntries = 1024;
constexpr int kRingBlocks = 4096;
// A ring met by a column (or a part of one): its last-axis origin relative to the window, and its entries
// over the column [ent, ent + count).
struct RingRef {
  int32_t ring;
  int32_t zr;
  int32_t ent;
  int32_t count;
};
// A block of ring work: references [ref0, ref0 + nref) of column col, with the nent entries from
// ent0, over the last-axis positions [zs, zs + 4 ks) of the window.
struct RingItem {
  int32_t col;
  int32_t ref0;
  int32_t nref;
  int32_t zs;
  int32_t ent0;
  int32_t nent;
  int32_t ks;
  int32_t pad;
};
struct RingSchedule {
  std::vector<RingRef> refs;
  std::vector<int32_t> ent;        // per entry: node; (kOffBias + column origin - support origin) per axis
                                   // as bytes x | y << 8, and the reference's
                                   // place in its interpolation block << 16
  std::vector<int32_t> col_ref;    // references of column c: [col_ref[c], col_ref[c + 1])
  std::vector<RingItem> interp;
  std::vector<int32_t> interp_cut; // XCD x takes the items [cut[x], cut[x + 1])
  std::vector<int32_t> gptr, gpos; // per node, the entries whose partials make its value
};
struct HostTables;
struct RingTables {
  std::vector<double> wz;          // [rings][kWMax]: last-axis weights
  RingSchedule sched[2];
};

// Interpolation and spread work lists over one subset of the nodes.
struct Schedule {
  std::vector<InterpItem> interp_items;   // grouped nodes (LDS-staged region)
  std::vector<int32_t> interp_direct;     // nodes interpolated straight from the grid
  std::vector<int32_t> list;              // spread: node indices per tile, concatenated
  std::vector<SpreadItem> items;
  std::vector<ReduceItem> reduces;
  int32_t nslots = 0;
  // the list positions of node q are gpos[gptr[q] .. gptr[q+1]) (increasing); on request only: no
  // kernel gathers by tile entries
  std::vector<int32_t> gptr;
  std::vector<int32_t> gpos;
  // row-window form (see HostTables::row_windows): per list entry i, ent[2i] = node and
  // ent[2i+1] = kOffBias + s_a packed as bytes x | y << 8 | z << 16, where s_a in [-7, w-1]
  // is the tile origin minus the support origin on axis a; kEntPad zero entries follow
  std::vector<int32_t> ent;
  // Last-axis window: every fine position that a scheduled node's support touches lies in
  // [z0, z0 + nz) (mod n_fine[2]); z0 and nz are multiples of HostTables::zalign.  The FFT passes of
  // this schedule read and write only the window, and the spread writes only its tiles.
  int32_t z0 = 0;
  int32_t nz = 0;
  // Axis-1 window (3D): every scheduled support lies at signed fine positions [-ny/2, ny/2) on
  // axis 1 (ny even; n_fine[1] when the supports reach the whole axis).  The axis-0 passes
  // transform only those lines and the axis-1 passes write (type-2) or read (type-1) only them.
  int32_t ny = 0;
};

// The two node subsets a plan schedules.  kAll: every node (the type-2 / type-1 entry
// points, whose node values are arbitrary).  kHalf: one node of each +-k pair (the
// operator on real grids, where the pair's terms are complex conjugates).
enum { kAll = 0, kHalf = 1 };

// Host-side tables built by build_tables() (all FP64).
struct HostTables {
  int dim = 3;
  int N[3] = {1, 1, 1};        // grid sizes on the internal 3-axis layout (N[0] = 1 in 2D)
  int nf[3] = {1, 1, 1};       // oversampled FFT sizes
  int W[3] = {1, 1, 1};        // kernel width per axis (1 on the unused 2D axis)
  int tile[3] = {1, 1, 1};     // spread tile extents
  int ntiles[3] = {1, 1, 1};
  int ib[3] = {1, 1, 1};       // interpolation group block extents
  int ireg[3] = {1, 1, 1};     // region extents ib + W - 1
  double h[3] = {1, 1, 1};
  double L[3] = {0, 0, 0};
  double cell = 1.0;           // prod(h)
  int w = 0;
  double es_beta = 0.0;
  double kmax = 0.0;
  int64_t m_nominal = 0;
  int64_t M = 0;               // nodes kept
  // per node, plan (sorted) order
  std::vector<int32_t> index;  // [M][3]
  std::vector<double> k;       // [M][3]
  std::vector<double> c;       // [M]  W Uhat / (2 pi)^d (times q for a split plan), for the axes nv, mv
  std::vector<double> base;    // [M]  W / (2 pi)^d (times q): c without the symbol
  bool c_stale = false;        // the axes changed (ddi_set_dipole): c is recomputed when read
  std::vector<int32_t> l0;     // [M][3]
  std::vector<double> wts;     // [M][3][kWMax]
  std::vector<double> deconv[3];   // 1/phihat per compact index, length N[a]
  // per node: 2 for the kept member of a complete +-k pair, 1 for a node whose partner
  // was masked out, 0 for the partner that is not kept in the half set
  std::vector<double> half_factor;
  // 3D with 8 x 8 x 8 tiles and n_fine >= w + 8 on every axis: a node's weights at a tile's
  // positions are one contiguous run of its weight row (no periodic wrap inside a tile); and
  // the weight rows fit 32-bit byte offsets (2 GiB)
  bool row_windows = false;
  // granularity of the schedules' last-axis windows: a multiple of kTileZ; 8 in FP64, 16 in FP32
  // (the strided FFT passes cover a window in blocks of lines that divide it: 128-byte rows)
  int zalign = 16;
  Schedule sched[2];
  // split of Eq. 3.9 (3D): c holds the I_2 weights (times q); I_1 uses the axes and s
  bool split = false;
  double split_s = 0.0;
  double nv[3] = {0, 0, 1};
  double mv[3] = {0, 0, 1};
};

// Kernel selection shared by the plan upload and the drivers.  FP64 in 3D interpolates by rings at every
// kernel width.  Against whole 8 x 8 x 8 tiles contracted per (tile, node) entry (us, tiles / rings), type-2:
// 64^3 44.5 / 44.7, 48.5 / 46.4, 66 / 51 at w = 4, 8, 14; 128^3 237 / 222, 265 / 246, 399 / 297.  Apply: 64^3
// 88 / 87, 100 / 96, 115 / 105; 128^3 311 / 312, 306 / 308, 325 / 320, 336 / 331, 440 / 394 at w = 4, 6, 8, 9, 14: the
// tiles left all of the spread's tables in the Infinity Cache, the rings only two of three weight rows, so
// at 128^3 the spread gives back what a narrow kernel's interpolation gains (16 x 16 x 1024 rule, w = 4: 248 / 260).
// FP32 in 3D interpolates node by node: there rings gained 3 us at 128^3 (w = 8: 60 / 57) and lost 54 at 256^3
// (248 / 302).
inline bool interp_by_rings(const HostTables& H, bool fp64) { return H.dim == 3 && fp64; }
inline bool uses_weight_rows(const HostTables& H) { return H.row_windows && kSpreadMfma; }

// Builds every host table of a plan.  Returns an empty string on success or an error message.
// interp_lists = false leaves out the node-owned interpolation's groups, which the interpolation by rings
// does not use; entry_lists = false the positions of every node's entries in the spread's list, which no
// plan uploads.
std::string build_tables(const ddi_params& p, HostTables& t, int* status, bool interp_lists = true,
                         bool entry_lists = true);

// Per node, the positions of its entries (in entry order): those of node q are pos[ptr[q] .. ptr[q+1]);
// entry i belongs to node[i * stride].
void entry_positions(const int32_t* node, int stride, size_t count, int64_t M, std::vector<int32_t>& ptr,
                     std::vector<int32_t>& pos);

// Builds the ring schedules of a 3D plan from its tables (npol = polar nodes of the rule).
std::string build_rings(const HostTables& t, int npol, RingTables& out);

// Morton (Z-order) key of a block coordinate, each below 2^20.
uint64_t morton3(uint32_t x, uint32_t y, uint32_t z);

// Cuts a list in spatial order into kXcds contiguous regions of about equal work: region x takes the items
// [cut[x], cut[x + 1]).  Workgroups go to the XCDs in turn, so each XCD, with its own L2, works through one
// compact region of the grid and its L2 sees the reuse.
constexpr int kXcds = 8;
template <typename Item, typename Work>
std::vector<int32_t> xcd_cuts(const std::vector<Item>& items, Work work) {
  int64_t total = 0, acc = 0;
  for (const Item& it : items) total += work(it);
  std::vector<int32_t> cut(kXcds + 1, static_cast<int32_t>(items.size()));
  cut[0] = 0;
  int seg = 1;
  for (size_t i = 0; i < items.size() && seg < kXcds; ++i) {
    acc += work(items[i]);
    while (seg < kXcds && acc * kXcds >= total * seg) cut[seg++] = static_cast<int32_t>(i + 1);
  }
  return cut;
}

// The items of the regions interleaved, since workgroup b runs on XCD b mod kXcds; shorter regions are padded
// with `pad` items, which the kernels skip.
template <typename Item>
std::vector<Item> interleave(const std::vector<Item>& items, const std::vector<int32_t>& cut, const Item& pad) {
  int longest = 0;
  for (int x = 0; x < kXcds; ++x) longest = std::max(longest, cut[x + 1] - cut[x]);
  std::vector<Item> out(static_cast<size_t>(longest) * kXcds, pad);
  for (int x = 0; x < kXcds; ++x)
    for (int j = 0; j < cut[x + 1] - cut[x]; ++j) out[static_cast<size_t>(j) * kXcds + x] = items[cut[x] + j];
  return out;
}

// Accurate e^{-2 pi i k / n}, k in [0, n), interleaved (re, im).
std::vector<double> twiddle_table(int n);

// ---------------------------------------------------------------- device side
template <typename T>
struct Complex {
  T re, im;
};

// Remap a block index so that consecutive logical blocks run on the same XCD:
// blocks are dispatched round-robin over the 8 XCDs, each with its own L2.
__device__ inline int xcd_remap(int b, int nb) {
  constexpr int X = 8;
  const int x = b % X, local = b / X;
  const int base = nb / X, rem = nb % X;
  return x * base + (x < rem ? x : rem) + local;
}

#define DDI_CHECK(x)                 \
  do {                               \
    hipError_t e_ = (x);             \
    if (e_ != hipSuccess) return e_; \
  } while (0)

// Workspace of the GPE kernels on an N0 x N1 x N2 grid of the plan's real type T.
struct GpeWork {
  void* rho = nullptr;           // T[N]
  void* phi = nullptr;           // T[N]
  void* phit = nullptr;          // T[N]
  void* c1 = nullptr;            // Complex<T>[N]
  void* c2 = nullptr;            // Complex<T>[N] (gradient flow only)
  double* red = nullptr;         // reduction scratch: gpe_red_doubles(red_blocks) doubles
  int red_blocks = 0;
};
// Doubles of the reduction scratch: 4 slots per block for two reductions, then 8 scalars (the
// gradient flow's alpha), then the 5 energies (at offset 8 nb + 8).
inline size_t gpe_red_doubles(int nb) { return 8 * static_cast<size_t>(nb) + 16; }

// Device-resident plan state.
struct DevicePlan {
  HostTables H;
  bool mixed = false;
  int device = 0;
  // tables
  void* nodes = nullptr;         // NodeRec<T>[M]
  double* c_scaled = nullptr;    // c_q * prod(h) [M]
  double* deconv[3] = {nullptr, nullptr, nullptr};
  double* c_half = nullptr;       // half_factor * c_q * prod(h) [M]
  double* ones = nullptr;         // [max N]: unit factors for the split's padded FFT passes
  // split: I_1 runs on its own stream (default priority) into its own padded grid, overlapping
  // I_2; events fork it from and join it to the caller's stream
  void* fine_short = nullptr;     // Complex<T>[nf0*nf1*nf2]
  // ddi_set_dipole (allocated on its first call): node coordinates and the weights without the
  // symbol, scaled as c_scaled and c_half
  double* kq = nullptr;           // [M][3]
  double* base_scaled = nullptr;  // base * prod(h) [M]
  double* base_half = nullptr;    // half_factor * base * prod(h) [M]
  hipStream_t aux = nullptr;
  hipEvent_t ev_fork = nullptr, ev_long = nullptr, ev_join = nullptr;
  struct DevSchedule {
    int32_t* list = nullptr;
    SpreadItem* items = nullptr;
    ReduceItem* reduces = nullptr;
    InterpItem* interp_items = nullptr;
    int32_t* interp_direct = nullptr;
    int32_t* ent = nullptr;
  } dsched[2];
  // FP64 in 3D: ring schedules (rings.hip)
  struct DevRings {
    RingRef* refs = nullptr;
    int32_t* ent = nullptr;
    RingItem* interp = nullptr;
    int32_t* gptr = nullptr;
    int32_t* gpos = nullptr;
    int ninterp = 0;             // workgroups: the regions' items interleaved, with padding
  } drings[2];
  double* ring_wz = nullptr;     // [rings][kWMax]
  void* xyw = nullptr;           // T[M][2][kWMax]: weight rows of axes 0 and 1, without row windows
  bool interp_lds_ready = false;
  void* twiddles[kTwSlots] = {}; // per FFT length n (slot tw_slot(n) of fft.h): Complex<T>[n]
  // workspace
  void* fine = nullptr;          // Complex<T>[nf0*nf1*nf2]
  void* gnodes = nullptr;        // Complex<T>[M]
  void* partial = nullptr;       // Complex<T>[nslots][tile volume]
  void* ipartial = nullptr;      // Complex<double>[ring entries]: interpolation partial sums
  void* pads = nullptr;          // T[M + 1][3][kRowLen]: weight rows (one 128-byte line per row in
                                 // FP64), then a zero record that positions outside a window read
  int64_t workspace_bytes = 0;
  // GPE workspace (allocated on first use)
  GpeWork gpe;
};

// Kernel launchers (kernels.hip), templated on the real type.
template <typename T>
hipError_t run_type2(DevicePlan& P, int which, const T* rho, Complex<T>* out, const double* scale,
                     double cscalar, int sign, hipStream_t s, hipEvent_t* ev);
template <typename T>
hipError_t run_type1(DevicePlan& P, int which, const Complex<T>* g, T* phi, int sign, hipStream_t s,
                     hipEvent_t* ev);
template <typename T>
hipError_t run_apply(DevicePlan& P, const T* rho, T* phi, int sign, hipStream_t s, hipEvent_t* ev);
// I_1 of the split (Eq. 3.9): padded FFT, (1 - q) Uhat, inverse FFT into fine_short (front),
// then the last inverse pass added to phi (back).
template <typename T>
hipError_t split_short_front(DevicePlan& P, const T* rho, hipStream_t s);
template <typename T>
hipError_t split_short_back(DevicePlan& P, T* phi, hipStream_t s);
// Re-evaluate c_scaled and c_half for new dipole axes from kq, base_scaled and base_half.
hipError_t run_set_dipole(DevicePlan& P, const double* n, const double* m, hipStream_t s);
// The operator of the plan: run_apply, plus I_1 for a split plan (I_1 is its own transpose).
template <typename T>
hipError_t run_ddi(DevicePlan& P, const T* rho, T* phi, int sign, hipStream_t s, hipEvent_t* ev);
// Interpolation at the nodes times scale, by rings (rings.hip).
hipError_t ring_interp(DevicePlan& P, int which, Complex<double>* out, const double* scale, double sscalar, hipStream_t s);
constexpr int kStages = 9;
template <typename T>
hipError_t run_gpe_energy_grad(DevicePlan& P, const GpeWork& W, const gpe_params& gp, const Complex<T>* psi,
                               double* E_dev, Complex<T>* grad, hipStream_t s);
template <typename T>
hipError_t run_gf_step(DevicePlan& P, const gpe_params& gp, double dt, int n_inner, const Complex<T>* psi_in,
                       Complex<T>* psi_out, double* residual, hipStream_t s);
template <typename T>
hipError_t run_ts_step(DevicePlan& P, const gpe_params& gp, double dt, double delta, double q,
                       const Complex<T>* psi_in, Complex<T>* psi_out, hipStream_t s);
template <typename T>
int gpe_reduction_blocks(const DevicePlan& P);

}  // namespace ddi
