// nyx_internal.h -- device-side box descriptors and launch arguments shared
// by the host ABI layer (nyx_abi.cpp) and the two precision builds of the
// stage kernels (nyx_step.hip).  Not part of the public ABI.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/nyx_hydro.h"

namespace nyx {

constexpr int kBlock = 256;  // threads per block: 4 wavefronts of 64
// Threads per workgroup of the fused final-stage kernel (8 wavefronts): a
// tile of TX x TY cell columns of a box, TX = min(n_x, 64), TY = min(n_y,
// kFinBlock / TX), over a chunk of at most `planes` planes in z, chosen per
// plan from kFinPlanes down (fin_planes).
constexpr int kFinBlock = 512;
constexpr int kFinPlanes = 64, kFinMinPlanes = 8;
// Tiles that keep the chip's 512 resident workgroups (two per CU) evenly busy
// to the end of the launch: each extra chunk solves one layer of z-faces again
// (a face in 3.2 per cell and plane), so chunks are cut only while the launch
// has fewer tiles than this.
constexpr long long kFinTiles = 2048;
// Threads per workgroup of the flattening and tracing pass (k_edges): a tile of
// at most kEdgeBlock cell columns of the [-1, n]^3 range, whose planes with a
// halo of three cells have at most kEdgeLds cells, over a chunk of planes in
// z.  Tiles span a box of up to kEdgeWide columns in x whole (the 66 of a 64^3
// patch), so that rows are loaded and stored whole.  Chunks are cut down to
// kEdgeMinPlanes while the launch has fewer than kEdgeWant tiles (256^3, 5
// chunks of 52 planes against 33 of 8: 5050 and 4915 us a step).
constexpr int kEdgeBlock = 512;
constexpr int kEdgeLds = 1100;
constexpr int kEdgeWide = 72;
constexpr int kEdgePlanes = 64, kEdgeMinPlanes = 8;
constexpr long long kEdgeWant = 4096;
// Whether an FP32 launch over `cells` cells, whose tiles have `slots` lanes in
// all planes together, takes the pass.  It has to fill the chip several times
// over, as each workgroup marches up its planes, and a third of its lanes have
// to have a cell.  Step in us, separate kernels against the pass: 64^3 187 and
// 212, 96^3 381 and 400, 104^3 443 and 451, 108^3 477 and 477, 112^3 510 and 503,
// 160^3 1376 and 1330; 3000 boxes of 8^3 (20% of the lanes) 1394 and 1450, 900
// of 12^3 (38%) 962 and 933, 256 of 16^3 536 and 510, 64 of 64^3 5610 and 5300.
// In FP64 the pass needs 228 registers, two wavefronts a SIMD, and loses: 256
// boxes of 16^3 1204 and 1240 us, 128^3 1631 and 1652.
inline bool edges_pay(long long cells, long long slots) {
  return cells >= 5 * (1ll << 18) && 3 * cells >= slots;
}
// Stored per face: the Godunov state (rho_g, u_g normal, v_g, w_g transverse,
// p_g) in the face's rotated frame; every flux is recomputed from it.
constexpr int kGod = 5;
// Device counters are accumulated per block into kStatSlots partial blocks
// (block index modulo kStatSlots) and summed once per step.
constexpr int kStatSlots = 64;
constexpr int kStatFields = 10;

// Division by a per-box invariant divisor d with a precomputed multiplier:
// q = (umulhi(n, m) + n) >> l, exact for every n < 2^31.
struct FastDiv {
  unsigned d, m, l;
};
inline FastDiv make_fastdiv(unsigned d) {
  unsigned l = 0;
  while ((1ull << l) < d) ++l;
  unsigned long long m = ((1ull << 32) * ((1ull << l) - d)) / d + 1;
  return FastDiv{d, (unsigned)m, l};
}

// One box as the kernels see it.  All offsets are element offsets.
struct BoxDev {
  int n[3];
  int ng;
  int px, py, pz;          // padded extents n + 2 ng
  int ex, ey, ez;          // extents of the cell range [-1, n]
  long long P, E, V;       // padded, [-1,n]^3 and valid cell counts
  long long soff, goff;    // state / gravity offset of padded cell 0
  long long sstride, gstride;
  long long w_prim, w_chi, w_edge, w_f0, w_f1, w_f2;  // stage arrays (elements)
  int gidx;                // index of the box in the caller's list
  int pad_;
  double dx;
  FastDiv dv[3][2];        // per Space: row length and plane size
  FastDiv dz[3];           // per Space: number of planes
  unsigned sy[3];          // per Space: rows per plane
  unsigned sc[3];          // per Space: cell count (< 2^31)
  int ntx, nty, ntiles;    // fused final stage: tiles along x and y, and in all
  int etiles;              // flattening and tracing pass: tiles in all
  unsigned short tx, ty;   // final stage: tile shape
  unsigned char tz;        // final stage: planes per chunk (at most kFinPlanes)
  unsigned char etx, ety, etz;  // flattening and tracing pass: tile shape, planes per chunk
};
// a plan's workspace holds one per box: a larger one would refuse workspaces
// that held the plan before
static_assert(sizeof(BoxDev) <= 328, "box descriptor grown");

// Stage-array element count for a box (before alignment padding).
inline long long align_elems(long long n) { return (n + 63) / 64 * 64; }

// The fused final stage's tiling of a box: tile shape, and z chunks of equal
// length (up to rounding) of at most `planes` planes.
struct FinTiling {
  int tx, ty, ntx, nty, tz, ntz;
};
inline FinTiling fin_tiling(const nyx_box& b, int planes) {
  FinTiling t;
  t.tx = b.n[0] < 64 ? b.n[0] : 64;
  t.ty = b.n[1] < kFinBlock / t.tx ? b.n[1] : kFinBlock / t.tx;
  t.ntx = (b.n[0] + t.tx - 1) / t.tx;
  t.nty = (b.n[1] + t.ty - 1) / t.ty;
  t.ntz = (b.n[2] + planes - 1) / planes;
  t.tz = (b.n[2] + t.ntz - 1) / t.ntz;
  return t;
}
// Planes per chunk for a plan's boxes: the longest chunk that gives the launch
// kFinTiles tiles.
inline int fin_planes(int nbox, const nyx_box* boxes) {
  for (int planes = kFinPlanes; planes > kFinMinPlanes; planes /= 2) {
    long long tiles = 0;
    for (int i = 0; i < nbox; ++i) {
      const FinTiling t = fin_tiling(boxes[i], planes);
      tiles += (long long)t.ntx * t.nty * t.ntz;
    }
    if (tiles >= kFinTiles) return planes;
  }
  return kFinMinPlanes;
}

// The same for the flattening and tracing pass (cells [-1, n]).
typedef FinTiling EdgeTiling;
inline EdgeTiling edge_tiling(const nyx_box& b, int planes) {
  const int ex = b.n[0] + 2, ey = b.n[1] + 2, ez = b.n[2] + 2;
  EdgeTiling t;
  t.ntx = (ex + kEdgeWide - 1) / kEdgeWide;
  t.tx = (ex + t.ntx - 1) / t.ntx;
  int ty = kEdgeBlock / t.tx;
  const int lds = kEdgeLds / (t.tx + 6) - 6;
  ty = ty < lds ? ty : lds;
  t.nty = (ey + ty - 1) / ty;
  t.ty = (ey + t.nty - 1) / t.nty;
  t.ntz = (ez + planes - 1) / planes;
  t.tz = (ez + t.ntz - 1) / t.ntz;
  return t;
}
inline long long edge_tiles(int nbox, const nyx_box* boxes, int planes) {
  long long n = 0;
  for (int i = 0; i < nbox; ++i) {
    const EdgeTiling t = edge_tiling(boxes[i], planes);
    n += (long long)t.ntx * t.nty * t.ntz;
  }
  return n;
}
// Planes per chunk: the longest chunk that gives the launch kEdgeWant tiles.
inline int edge_planes(int nbox, const nyx_box* boxes) {
  int planes = kEdgePlanes;
  while (planes > kEdgeMinPlanes && edge_tiles(nbox, boxes, planes) < kEdgeWant) planes /= 2;
  return planes;
}

// Fill the derived fields and stage offsets of a box starting at `base`;
// returns the element offset just past its stage arrays.
inline long long box_layout(const nyx_box& b, int gidx, long long base, BoxDev* out,
                            int planes = kFinPlanes, int eplanes = kEdgePlanes) {
  BoxDev d{};
  for (int i = 0; i < 3; ++i) d.n[i] = b.n[i];
  d.ng = b.ng;
  d.px = b.n[0] + 2 * b.ng;
  d.py = b.n[1] + 2 * b.ng;
  d.pz = b.n[2] + 2 * b.ng;
  d.ex = b.n[0] + 2;
  d.ey = b.n[1] + 2;
  d.ez = b.n[2] + 2;
  d.P = (long long)d.px * d.py * d.pz;
  d.E = (long long)d.ex * d.ey * d.ez;
  d.V = (long long)b.n[0] * b.n[1] * b.n[2];
  d.soff = b.state_off;
  d.goff = b.grav_off;
  d.sstride = b.comp_stride;
  d.gstride = b.grav_stride;
  d.dx = b.dx;
  d.gidx = gidx;
  long long o = base;
  d.w_prim = o; o += align_elems(6 * d.P);
  d.w_chi = o;  o += align_elems(d.E);
  d.w_edge = o; o += align_elems(30 * d.E);
  d.w_f0 = o;   o += align_elems(3 * kGod * d.E);
  d.w_f1 = o;   o += align_elems(6 * kGod * d.E);
  d.w_f2 = o;   o += align_elems(3 * kGod * d.E);
  d.dv[0][0] = make_fastdiv((unsigned)d.px);
  d.dv[0][1] = make_fastdiv((unsigned)d.px * (unsigned)d.py);
  d.dv[1][0] = make_fastdiv((unsigned)d.ex);
  d.dv[1][1] = make_fastdiv((unsigned)d.ex * (unsigned)d.ey);
  d.dv[2][0] = make_fastdiv((unsigned)b.n[0]);
  d.dv[2][1] = make_fastdiv((unsigned)b.n[0] * (unsigned)b.n[1]);
  d.dz[0] = make_fastdiv((unsigned)d.pz);
  d.dz[1] = make_fastdiv((unsigned)d.ez);
  d.dz[2] = make_fastdiv((unsigned)b.n[2]);
  d.sy[0] = (unsigned)d.py;
  d.sy[1] = (unsigned)d.ey;
  d.sy[2] = (unsigned)b.n[1];
  d.sc[0] = (unsigned)d.P;
  d.sc[1] = (unsigned)d.E;
  d.sc[2] = (unsigned)d.V;
  const FinTiling t = fin_tiling(b, planes);
  d.tx = (unsigned short)t.tx;
  d.ty = (unsigned short)t.ty;
  d.ntx = t.ntx;
  d.nty = t.nty;
  d.tz = (unsigned char)t.tz;
  d.ntiles = t.ntx * t.nty * t.ntz;
  const EdgeTiling w = edge_tiling(b, eplanes);
  d.etx = (unsigned char)w.tx;
  d.ety = (unsigned char)w.ty;
  d.etz = (unsigned char)w.tz;
  d.etiles = w.ntx * w.nty * w.ntz;
  if (out) *out = d;
  return o;
}

// Per-box constants of a step, computed once per box by the step's prologue
// kernel (the same expressions the oracle evaluates on the host).
struct StepC {
  double dt, a_h, da, kh, hdt_a, hda_a, pexp, kap1, kap2, k;
  double xo, xn;  // expansion source of the energy equations at a_old / a_new
  // the tracing's factors in FP32 (the mixed build's; a kernel then reads them
  // as scalars instead of converting them in every lane)
  float khf, hdt_af, hda_af, pexpf;
};

// Which cell range a launch walks: padded cells, the [-1, n]^3 range, valid
// cells, the column tiles of the fused final stage and those of the flattening
// and tracing pass (counted in tiles, not in blocks of cells; no cell
// coordinates of their own).
enum Space { kSpaceP = 0, kSpaceE = 1, kSpaceV = 2, kSpaceT = 3, kSpaceF = 4 };
constexpr int kSpaces = 5;

#ifdef __HIPCC__
// Workgroups are dispatched round-robin over the 8 XCDs of the chip, each
// with its own L2.  Renumber them so that every XCD walks one contiguous
// range of the (linearised) grid: neighbouring rows and planes of a stage
// array are then read through the same L2.  A bijection for any grid size.
// With remap = false the hardware order is kept (the autotuner's other
// candidate).
__device__ __forceinline__ unsigned xcd_linear_block(bool remap = true) {
  const unsigned n = gridDim.x * gridDim.y;
  const unsigned lin = blockIdx.x + blockIdx.y * gridDim.x;
  if (!remap) return lin;
  const unsigned q = n >> 3, r = n & 7;
  const unsigned xcd = lin & 7, pos = lin >> 3;
  return xcd < r ? xcd * (q + 1) + pos : r * (q + 1) + (xcd - r) * q + pos;
}

// Raise *dst (bits of a non-negative double) to the bits of m.  The stored
// maximum only grows, so a read that already shows a value at least as large
// (even a stale one) makes the atomic unnecessary; most blocks of a box then
// skip it instead of queueing on one address.
__device__ __forceinline__ void max_bits(unsigned long long* dst, double m) {
  const unsigned long long v = (unsigned long long)__double_as_longlong(m);
  if (__hip_atomic_load(dst, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < v) atomicMax(dst, v);
}

__device__ __forceinline__ unsigned fast_div(unsigned n, const FastDiv& f) {
  return (__umulhi(n, f.m) + n) >> f.l;
}
// Element i of an array through a 32-bit byte offset.  Every per-box array
// has fewer than 2^29 elements (checked on the host), so the byte offset fits
// 32 bits.  With a base that is uniform over the workgroup the compiler can
// use the scalar-base form of the memory instructions where the offset and
// the access sit in one block; elsewhere the access costs one 64-bit add.
template <class T>
__device__ __forceinline__ T ldu(const T* base, unsigned i) {
  return *(const T*)((const char*)base + i * (unsigned)sizeof(T));
}
template <class T>
__device__ __forceinline__ void stu(T* base, unsigned i, T v) {
  *(T*)((char*)base + i * (unsigned)sizeof(T)) = v;
}

// The same for a base that is uniform over the wavefront, as every stage
// array's is.  The base is kept opaque in scalar registers: left to itself the
// compiler folds the strides of neighbouring accesses into one vector address
// and spends a 64-bit vector add on most of them; this way each access takes
// the scalar-base form.  With the index extended in the block of the accesses
// (local_idx, called once in front of them) that costs no vector instruction.
// Not a gain everywhere: kernels of many loads from one offset with registers to
// spare (flattening, the separate tracing, the staged final stage) are faster
// with plain loads (ldu).
__device__ __forceinline__ unsigned local_idx(unsigned i) {
  asm("" : "+v"(i));
  return i;
}
__device__ __forceinline__ unsigned long long wave_base(const void* p) {
  const unsigned long long a = (unsigned long long)p;
  const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)a);
  const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(a >> 32));
  return (unsigned long long)hi << 32 | lo;
}
// A descriptor that no kernel of the step writes while it runs (a box, its
// step constants), through a scalar pointer into the constant address space:
// its reads stay scalar loads, also behind branches and the stage's stores.
// The same object in every lane of the wavefront: the first lane's is read.
template <class T>
__device__ __forceinline__ const T& scalar_ref(const T& r) {
  return *(const T*)(const T __attribute__((address_space(4)))*)wave_base(&r);
}
template <class T>
__device__ __forceinline__ T ldw(const T* base, unsigned i) {
  typedef const T __attribute__((address_space(1))) * G;
  typedef const char __attribute__((address_space(1))) * C;
  return *(G)((C)wave_base(base) + i * (unsigned)sizeof(T));
}
template <class T>
__device__ __forceinline__ void stw(T* base, unsigned i, T v) {
  typedef T __attribute__((address_space(1))) * G;
  typedef char __attribute__((address_space(1))) * C;
  *(G)((C)wave_base(base) + i * (unsigned)sizeof(T)) = v;
}

// Natural (x fastest, then y, then z) flat index of the cell at position q
// of a slab walk with 2^lg rows per slab (kTuneSlabShift); q >= the cell
// count is returned unchanged (lanes past the end of the box).
__device__ __forceinline__ unsigned slab_to_natural(const BoxDev& b, int space, unsigned q,
                                                    int lg) {
  if (q >= b.sc[space]) return q;
  const FastDiv& r = b.dv[space][0];
  const FastDiv& zd = b.dz[space];
  const unsigned ex = r.d, ey = b.sy[space], ez = zd.d;
  const unsigned t = fast_div(q, r);  // (slab, z, row) index
  const unsigned x = q - t * ex;
  const unsigned nfull = ey >> lg;    // whole slabs
  const unsigned tfull = (nfull << lg) * ez;
  unsigned y, z;
  if (t < tfull) {
    const unsigned yin = t & ((1u << lg) - 1u);
    const unsigned u = t >> lg;
    const unsigned sl = fast_div(u, zd);
    z = u - sl * ez;
    y = (sl << lg) + yin;
  } else {
    const unsigned t2 = t - tfull;
    const unsigned yin = fast_div(t2, zd);
    z = t2 - yin * ez;
    y = (nfull << lg) + yin;
  }
  return x + ex * (y + ey * z);
}

// (x, y, z) of flat index idx < 2^31 in the given Space of a box
__device__ __forceinline__ void space_coords(const BoxDev& b, int space, unsigned idx, int* c) {
  const FastDiv& r = b.dv[space][0];
  const FastDiv& pl = b.dv[space][1];
  unsigned q1 = fast_div(idx, r);
  unsigned q2 = fast_div(idx, pl);
  c[0] = (int)(idx - q1 * r.d);
  c[1] = (int)(q1 - q2 * b.sy[space]);
  c[2] = (int)q2;
}
#endif

// Stage kernels of a step, in launch order (also the order of the timing
// events and of the tuning entries).
constexpr int kStages = 7;
enum Stage { kStPrim = 0, kStFlat, kStTrace, kStRiem0, kStRiem1, kStRiem2, kStUpdate };
// Launch-order candidates of a stage (fields of a tuning entry):
//  bit 0 (kTuneCellMajor)  grids with one row per direction (or direction
//                  pair) walk the rows of one cell range back to back, so the
//                  stage arrays the directions share are reread from the same
//                  L2; otherwise one direction after the other;
//  bit 1 (kTuneHwOrder)    hardware workgroup order instead of the
//                  XCD-contiguous numbering;
//  bits 2-3 (kTuneSlabShift) cell order within a box: 0 plane by plane (x,
//                  then y, then z); s = 1, 2, 3: slabs of 2^(s+2) rows, each
//                  walked plane by plane along z (a z-pencil of row tiles), so
//                  a cell's z-neighbours are read shortly after it through
//                  the same L2; rows left over below a whole slab are walked
//                  one row at a time along z.
constexpr int kTuneCellMajor = 1;
constexpr int kTuneHwOrder = 2;
constexpr int kTuneSlabShift = 2;
constexpr int kTuneCandidates = 16;
// Launch orders of a new plan and of the single-box step.  Tracing and the
// transverse stage read the same cells' arrays in every direction (primitives;
// stage-0 states), so their default walks the directions of one range of cells
// back to back: direction by direction, each array comes from HBM again.
// Measured on the tracing / the transverse stage (ms), FP32-mixed: 256^3 box
// 1.19 -> 1.06 / 1.91 -> 1.82, 64 patches of 64^3 1.24 -> 1.08 / 2.14 -> 2.03,
// 96 uneven boxes 0.42 -> 0.35 / 0.74 -> 0.63.  The other stages share little
// between directions and gained nothing.
constexpr int kTuneDefault[kStages] = {0, 0, kTuneCellMajor, 0, kTuneCellMajor, 0, 0};

// Control block of the persistent step (device, zeroed before each launch):
// per stage the heads of 8 work queues (one per eighth of the part of the
// stage's walk that is not handed out statically, drained first by the
// workgroups of one XCD); per stage boundary the arrival counts of the 8 XCD
// groups of workgroups and the count of XCD groups complete; the abort flag
// a barrier that timed out raises.
constexpr int kCtlXcdBar = kStages * 8;
constexpr int kCtlBarrier = kCtlXcdBar + kStages * 8;
constexpr int kCtlAbort = kCtlBarrier + kStages;
constexpr int kCtlWords = kCtlAbort + 1;
constexpr int kCtlDone = kCtlWords;  // StepArgs::done of a plan, behind the block

// Largest grid of the final kernel whose last workgroup writes dt_next.
constexpr int kDoneBlocks = 1024;

// Launch-wide arguments of a step.
struct StepArgs {
  // box selection: a device table + block prefix per Space (the single-box
  // entry points write a one-entry table in their prologue)
  BoxDev single;
  const BoxDev* table;     // device, nb entries (batched) or nullptr
  const int* prefix[kSpaces];  // device, nb+1 block prefixes per Space (batched)
  int nb;
  int nblocks[kSpaces];    // grid size per Space
  // physics
  const double* Uin;
  double* Uout;
  const void* grav;
  void* work;              // stage region base (real elements)
  unsigned long long* smax;  // per-box running max of |u|+c (bit pattern)
  const double* dt_dev;    // per-box dt (batched) or nullptr
  double dt_host;
  double a_old, a_new;
  double gamma, eta, small_dens, small_pres, riemann_tol, cfl;
  float small_densf, small_presf;  // the floors in FP32
  double igm1;   // 1 / (gamma - 1), for the mixed build's products
  float igm1f;   // the same in FP32 (the FP32 flux formulas)
  double mixed_stop;  // FP32-mixed stopping rule (see two_shock)
  int plain;     // gamma and the floors allow the FP64 build's short divisions
  int maxiter;
  nyx_stats* stats;
  unsigned long long* slots;  // kStatSlots x kStatFields partial counters (when stats)
  double* dt_next;
  hipEvent_t* ev;          // kStages + 1 events recorded around the stages, or nullptr
  const StepC* consts;     // per-box step constants, indexed by gidx
  // Single-box step: where the first kernel puts the box (`single`), its block
  // prefixes and its constants for the kernels after it, or nullptr.
  BoxDev* single_dst;
  int* prefix_dst;
  StepC* consts_dst;
  // Workgroups of the final kernel that have finished (device, zero between
  // launches): the last one then writes dt_next itself.  nullptr for larger
  // grids, whose dt_next takes a launch of its own.
  unsigned* done;
  // learned Riemann flux (FP32-mixed build only)
  const void* mlp;         // packed network, or nullptr
  int learned_mask;        // bit s: stage s (0, 1, 2) uses the network
  double mlp_tol;          // accepted two-shock residual
  // harvest of final-stage faces for training
  float* harvest;          // [cap][15] records, or nullptr
  unsigned long long* harvest_count;
  long long harvest_cap;
  unsigned harvest_keep;   // keep a face when its 32-bit hash < harvest_keep
  unsigned long long harvest_seed;
  int tune[kStages];       // launch-order candidate per stage (kTune* bits)
  // scheme variants (Sec. 3.2)
  int recon;               // NYX_RECON_PPM or NYX_RECON_PLM
  int grav_form;           // energy gravity term, 1 or 2
  int linear_riemann;      // 1: linearised solver instead of the two-shock one
  int expansion;           // 1: gamma != 5/3, apply the a adot (2 - 3(gamma-1)) rho e term
  // persistent step: control block (kCtlWords, zeroed before the launch)
  // and the grid barrier's time limit in wall-clock ticks
  unsigned long long* ctl;
  unsigned long long barrier_ticks;
  // 1: stages riem2 and update run fused (k_final) where the step allows it
  int fuse_final;
  // 1: stages flat and trace run as one pass (k_edges)
  int edges;
  // where stage 1 reads a ghost cell of the input state: 0 the input's own
  // ghost cell; 1 its periodic image in the same box; 2 its source cell in
  // the neighbouring box of boxes that tile a periodic domain as a
  // gg[0] x gg[1] x gg[2] grid (gfull: every box of the plan in box order)
  int gsrc;
  int gg[3];
  const BoxDev* gfull;
};


// Shape check of one box (NYX_OK or a negative nyx_status).
int validate_box(const nyx_box* b);

// One face of a flux register fed by a batched step (Sec. 4.3 reflux): the
// final flux of face f (box-local; f[d] in [0, n_d] along the normal d, a
// valid cell index across it) of box `box` is added, times scale * dt, to
// register slot `slot`.  nsub = 2 sums the 2 x 2 faces f, f + e_t1,
// f + e_t2, f + e_t1 + e_t2 (t1 < t2 the transverse axes) in that order.
struct FluxRec {
  int box, d, nsub, pad_;
  int f[3], pad2_;
  double scale;
  long long slot;
};

// The records of one level of a two-level sync plan (nyx_sync.hip), sorted
// by box, with the per-box prefix (host, nbox + 1 entries) and box shapes
// (host, 3 ints per box) for matching a batch plan.
struct SyncLevelView {
  const FluxRec* recs;
  const long long* prefix;
  const int* shapes;
  int nbox;
  long long nslots;
};

#ifdef __HIPCC__
// Step constants of a box (built without contraction in every build: they are
// the expressions the oracle evaluates).
__device__ __forceinline__ StepC step_constants(const StepArgs& A, const BoxDev& b) {
#pragma clang fp contract(off)
  StepC c;
  c.dt = A.dt_dev ? A.dt_dev[b.gidx] : A.dt_host;
  const double gm1 = A.gamma - 1.0;
  c.a_h = 0.5 * (A.a_old + A.a_new);
  c.da = A.a_new - A.a_old;
  c.kh = c.dt / (c.a_h * b.dx);
  c.hdt_a = (0.5 * c.dt) / c.a_h;
  c.hda_a = (0.5 * c.da) / c.a_h;
  c.pexp = (1.5 * gm1) * (c.da / c.a_h);
  c.kap1 = c.kh / 3.0;
  c.kap2 = c.kh / 2.0;
  c.k = c.dt / b.dx;
  // a adot (2 - 3(gamma-1)) rho e = (adot / a) cgam U_e; integrated over the
  // step at a_old (predictor) and a_new (corrector)
  const double cgam = 2.0 - 3.0 * gm1;
  c.xo = cgam * (c.da / A.a_old);
  c.xn = cgam * (c.da / A.a_new);
  c.khf = (float)c.kh;
  c.hdt_af = (float)c.hdt_a;
  c.hda_af = (float)c.hda_a;
  c.pexpf = (float)c.pexp;
  return c;
}
// dt = cfl a dx / s_max of a box (Sec. 3.5)
__device__ __forceinline__ double dt_of_max(double cfl, double a, double dx, double smax) {
  return ((cfl * a) * dx) / smax;
}
#endif

// The two precision builds of the stage kernels.
// launch_step_persistent: the seven stages of a group as one launch of
// co-resident workgroups (NYX_E_UNSUPPORTED-worthy cases return
// hipErrorNotSupported: harvesting, or a learned-stage mask other than 0 or
// 7); persistent_grid: the workgroups it launches on the current device.
namespace fp64 {
hipError_t launch_step(const StepArgs& a, hipStream_t s);
hipError_t launch_step_persistent(const StepArgs& a, hipStream_t s);
int persistent_grid(const StepArgs& a);
hipError_t launch_flux_record(const StepArgs& a, const BoxDev* table, const FluxRec* recs,
                              long long nrec, double* reg, long long nslots, hipStream_t s);
}
namespace mixed {
hipError_t launch_step(const StepArgs& a, hipStream_t s);
hipError_t launch_step_persistent(const StepArgs& a, hipStream_t s);
int persistent_grid(const StepArgs& a);
hipError_t launch_flux_record(const StepArgs& a, const BoxDev* table, const FluxRec* recs,
                              long long nrec, double* reg, long long nslots, hipStream_t s);
}
// Precision-independent kernels (in nyx_abi.cpp's companion nyx_util.hip).
hipError_t launch_zero_u64(unsigned long long* p, int n, hipStream_t s);
hipError_t launch_dtmax(const StepArgs& a, double a_state, hipStream_t s);
hipError_t launch_dt_finalize(const StepArgs& a, double a_state, double cfl, double* dt_out,
                              hipStream_t s);
hipError_t launch_min_dt(double* dt, int n, hipStream_t s);
hipError_t launch_stats_reduce(const unsigned long long* slots, nyx_stats* stats, hipStream_t s);
// Prologue of a batched step: per-box step constants of boxes [0, nbox) of
// `a.table`; clears the CFL maxima (with a.dt_next), the partial counters
// (with a.stats) and the count of finished workgroups.
hipError_t launch_prologue(const StepArgs& a, int nbox, StepC* consts, hipStream_t s);
// learned flux (nyx_mlp.hip)
hipError_t launch_mlp_init(float* P, unsigned long long seed, hipStream_t st);
hipError_t launch_mlp_loss_grad(const float* P, const float* rec, long long n, double gamma,
                                float inv_n, float* grad, float* loss, hipStream_t st);
hipError_t launch_mlp_adam(float* P, float* m, float* v, const float* g, int t, float lr, float b1,
                           float b2, float eps, hipStream_t st);
hipError_t launch_mlp_pack(const float* P, void* packed, hipStream_t st);
hipError_t launch_mlp_predict(const void* packed, const float* rec, long long n, double gamma,
                              float* out, hipStream_t st);
hipError_t launch_fill_periodic(const StepArgs& a, const BoxDev* full, double* state, int ncomp,
                                int mode, int gx, int gy, int gz, hipStream_t s);

int sync_level_view(const nyx_sync_plan* p, int level, SyncLevelView* out);

}  // namespace nyx
