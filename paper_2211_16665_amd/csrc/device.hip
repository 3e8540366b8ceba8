// Device side of the fictitious-wave-domain engine for gfx950 (MI355X).
//
// One leapfrog step (Section 2, eq. fictitiouswave) computes
//   H^{n+1/2} = H^{n-1/2} - dt/mu curl E^n                + CPML
//   E^{n+1}   = E^n + dt/eps (curl H^{n+1/2} - J'^{n+1/2}) + CPML
// fused with the injection of J' at the source (or adjoint-source) edges,
// the receiver transform, and the volume transform acc_k += E z_k (eq. dft)
// in the forward run or the on-the-fly gradient product in the adjoint run.
// These forms carry out the same arithmetic per edge:
//   one launch   k_leap, a wave per 64 nodes of a row, which recomputes the
//                H it differences (order 2, one node per thread);
//   two kernels  k_update_h then k_update_e, one thread per (i, j, k) node
//                or per 16-byte vector of x nodes; order 4: k_rows_h4 then
//                k_rows_e4, a wave per 64 nodes of a row, or their general
//                forms k_update_h4 and k_update_e4;
//   fused        k_step, one launch per step: a block owns a column tile and
//                a chunk of z planes, stages each E plane (with a one-node
//                halo) and the new H plane (with its low-side halo) in LDS,
//                recomputes the H halo of its tile and marches up in z with
//                the plane below carried in registers.
// Fields and CPML memory are double-buffered: step n reads half n % 2 and
// writes the other half, so no block of a launch reads a value that another
// block has already overwritten.  The step index lives in device memory, in
// two counters: the launches of a step read one (the last completed step)
// and block 0 of its final launch writes the other, so no launch writes a
// counter it reads; the host alternates the pair from step to step and
// equalises them when it starts stepping.  A captured HIP graph of an even
// number of steps therefore replays for any position in the run.
//
// The kernels are bound by memory traffic and latency (a 3D stencil plus an
// accumulator sweep, ~0.1-0.8 flop/byte): no matrix cores.  Field layout
// [k][j][PX] (x fastest, PX a multiple of 64).  The batched sources are a
// grid dimension (fastest), so the blocks of one tile for all sources run
// side by side and share the per-edge coefficients in cache, and no thread
// loops over sources (on this GPU a loop whose stores precede the next
// iteration's loads waits for the stores: loads and stores share one
// in-order completion counter).  The 1D grid is remapped so that the
// consecutive blocks of one XCD are spatial neighbours (their halos hit the
// same L2).
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <type_traits>
#include <vector>

#include "fwdem_internal.hpp"

namespace fwdem {

#define HIP_CHECK(x)                                                                   \
  do {                                                                                 \
    hipError_t e_ = (x);                                                               \
    if (e_ != hipSuccess) fail(FWD_ERR_HIP, std::string(#x ": ") + hipGetErrorString(e_)); \
  } while (0)

// ---------------------------------------------------------------------------
// kernel parameter blocks
// ---------------------------------------------------------------------------
// Axis tables, one array [3 axes][8 tables][LA] (few pointers keep the
// kernel arguments in scalar registers): 1/h (n), 1/hd (n+1), CPML 1/kappa,
// b, a at integer nodes (n+1) and at half nodes (n).
enum { AX_IH = 0, AX_IHD, AX_KN, AX_BN, AX_AN, AX_KH, AX_BH, AX_AH, AX_TABLES };

// Division of numerators 0 <= n < 2^31 by a runtime divisor 1 <= d < 2^31 as
// a multiply-high (round-up method of Granlund and Montgomery, 1994): with
// l = ceil(log2 d) and m = ceil(2^(32+l) / d) - 2^32 (< 2^32),
//     n / d = (mulhi(n, m) + n) >> l,
// exact because the rounding of m adds less than n / 2^(32+l) < 1 / (2d)
// to n / d.  The block decode runs on the scalar unit, where a plain
// integer division is a long instruction sequence.
struct FDiv {
  uint32_t d, m, l;
};
static inline FDiv fdiv_make(uint32_t d) {
  uint32_t l = 0;
  while ((1ull << l) < d) ++l;
  const uint64_t num = 1ull << (32 + l);
  return FDiv{d, (uint32_t)((num + d - 1) / d - (1ull << 32)), l};
}
__device__ __forceinline__ uint32_t fdiv(uint32_t n, const FDiv &f) {
  return (__umulhi(n, f.m) + n) >> f.l;
}

template <typename T>
struct StepArgs {
  int nx, ny, nz, npml, PX, NY, NZ, ns;
  int64_t F;          // elements per field
  int64_t psi_src;    // psi elements per source
  T *fields;          // [2][ns][6][F]: Ex Ey Ez Hx Hy Hz per source, two halves
  T *psi;             // [2][ns][psi_src]
  int64_t fbuf, pbuf; // elements per half of fields and of psi
  const T *ce;        // [3][F] dt/eps per edge component
  const T *axt;       // [3][AX_TABLES][LA] axis tables
  int LA;
  T dtmu;             // dt / mu0
  const int *step;    // index of the last completed step (read by the step)
  int *step_w;        // the other counter: set to this step by block 0
  // tiling: (bx x by) threads over x-y; two kernels: one plane per block,
  // each thread a vector of x nodes; fused: kz planes per block
  int nbx, nby, nbz, nblocks, xcd, kz;   // nblocks = tiles * ns (the grid)
  int lean;           // interior tiles take the lean paths (npml >= 1)
  int kb;             // samples per transform block
  int dl;             // log2 of the volume transform's decimation (forward runs; 0: every sample)
  int nts;            // 1: non-temporal stores for the field halves and the history
  FDiv dplane, dpx;   // node decode of the block transform (q -> k, j, i)
  int order;          // tile numbering: 0 x fastest, 1 z fastest
  FDiv dns, dnbx, dnby, dnbz;             // dividers of the block decode (set_grid)
  // strides, precomputed on the host: plane = NY PX; CPML slabs sX (x), sY
  // (y), sZ (z) per variable; per-source field stride 6F; the y and z slab
  // offsets inside a source's psi block
  int64_t plane, sX, sY, sZ, F6, oY, oZ;
  // volume transform / gradient
  int nf;
  const double2 *zE;  // [nt][nf] z^{n+1}
  void *vol;          // [ns][nf][3][F] accumulators (forward) or forward transform (adjoint)
  const double2 *Q;   // [nt][nf] gradient weights (adjoint)
  double *gedge;      // [ns][3][F] gradient accumulators per source (adjoint)
  T *hist;            // [ns][kb-2][3][F] samples of the current transform block
  int64_t hist_src;   // history elements per source
  const int *flushed; // last sample already in the volume transform / gradient
  // per-thread lists of injection targets and receiver nodes (see build_lists)
  const int *tile_tab;  // [nblocks]: offset of the tile's table in tl_off, or -1
  const int *tl_off;    // per listed tile: bx*by + 1 entry offsets
  const int2 *tl_ent;   // entries: x = c | kind << 2 | sub << 3 | s << 9, y = ref
  int nrow, nt;         // rows of the time-function table, steps
  const double *coef;   // injection coefficients (entry ref = first row)
  const double *Ftab;   // [nrow][nt] time functions (wavelet or basis functions)
  double2 *racc;        // [ns][nn][nf] receiver-node transforms
  int nn;               // receiver nodes
  const int *rn_c;      // [nn] component of each receiver node (3..5: H)
  double dtmu64;        // dt / mu in double (magnetic sources)
  const double2 *zH;    // [nt][nf] z^{n+1/2} (H samples)
};

// Block -> (tile, source).  Blocks b = tile * ns + s, sources fastest, so
// the sources of a tile run side by side and share its coefficients in
// cache.  With xcd on, the blocks (dealt round-robin to the 8 XCDs) are
// remapped so that XCD x gets the contiguous range [base_x, base_x + cnt_x)
// of b: spatial neighbours (and all sources of a tile) share one L2.
// Tiles are numbered x fastest, t = (bz * nby + by) * nbx + bx (order 0),
// or z fastest, t = (by * nbx + bx) * nbz + bz (order 1: the blocks of
// consecutive planes of a column tile run side by side, so the plane
// neighbours a stencil reads are still in L2).  Returns the tile index.
template <typename T>
__device__ __forceinline__ int tile_of_b(const StepArgs<T> &A, uint32_t b, int &bx, int &by,
                                         int &bz, int &s) {
  if (A.xcd) {
    const uint32_t q = (uint32_t)A.nblocks >> 3, r = (uint32_t)A.nblocks & 7u;
    const uint32_t x = b & 7u, local = b >> 3;
    b = x * q + min(x, r) + local;
  }
  const uint32_t tile = fdiv(b, A.dns);
  s = (int)(b - tile * (uint32_t)A.ns);
  if (A.order) {
    const uint32_t t = fdiv(tile, A.dnbz), u = fdiv(t, A.dnbx);
    bz = (int)(tile - t * (uint32_t)A.nbz);
    bx = (int)(t - u * (uint32_t)A.nbx);
    by = (int)u;
  } else {
    const uint32_t t = fdiv(tile, A.dnbx), u = fdiv(t, A.dnby);
    bx = (int)(tile - t * (uint32_t)A.nbx);
    by = (int)(t - u * (uint32_t)A.nby);
    bz = (int)u;
  }
  return (int)tile;
}
template <typename T>
__device__ __forceinline__ int tile_of(const StepArgs<T> &A, int &bx, int &by, int &bz, int &s) {
  return tile_of_b(A, blockIdx.x, bx, by, bz, s);
}

// Index of the step a launch computes: one uniform scalar load of the
// counter the previous step wrote.  In the launch that ends a step, the
// first thread of block 0 stores it in the other counter (no launch writes
// a counter it reads, so no block waits on another).
template <typename T>
__device__ __forceinline__ int step_of(const StepArgs<T> &A, bool last_launch) {
  const int n = A.step[0] + 1;
  if (last_launch && blockIdx.x == 0 && threadIdx.x == 0 && threadIdx.y == 0) A.step_w[0] = n;
  return n;
}

// This thread's slice [lo, hi) of its tile's entry list; empty for the
// tiles without entries (most of them).  The tile's table index is one
// uniform scalar load; callers ask for the slice after issuing their
// stencil loads, so its round trip overlaps theirs.
template <typename T>
__device__ __forceinline__ void entry_slice_at(const StepArgs<T> &A, int b, int n, int slot, int &lo,
                                               int &hi) {
  lo = hi = 0;
  if (!A.tile_tab || n >= A.nt) return;   // no injection or recording past the run
  const int tt = A.tile_tab[__builtin_amdgcn_readfirstlane(b)];
  if (tt < 0) return;
  lo = A.tl_off[tt + slot];
  hi = A.tl_off[tt + slot + 1];
}
template <typename T>
__device__ __forceinline__ void entry_slice(const StepArgs<T> &A, int b, int n, int &lo, int &hi) {
  entry_slice_at(A, b, n, threadIdx.y * blockDim.x + threadIdx.x, lo, hi);
}

// slab index of a CPML node: half nodes i+1/2 with i < npml or i >= n-npml;
// integer nodes with i < npml or i > n-npml; both map to [0, 2 npml)
__device__ __forceinline__ bool pml_half(int i, int n, int npml, int &l) {
  if (i < npml) { l = i; return true; }
  if (i >= n - npml) { l = i - n + 2 * npml; return true; }
  return false;
}
__device__ __forceinline__ bool pml_int(int i, int n, int npml, int &l) {
  if (i < npml) { l = i; return true; }
  if (i > n - npml) { l = i - n + 2 * npml - 1; return true; }
  return false;
}

// One source's fields and CPML memory slabs in one half of the double
// buffer.  Slabs: X [4][NZ][NY][W], Y [4][NZ][W][PX], Z [4][W][NY][PX] with
// W = 2 npml; memory variables 0 and 1 belong to H, 2 and 3 to E (the E
// ones are updated in place in half 0).
template <typename T>
struct Half {
  T *ex, *ey, *ez, *hx, *hy, *hz;
  T *psX, *psY, *psZ;
};

template <typename T>
__device__ __forceinline__ Half<T> half_of(const StepArgs<T> &A, int par, int s) {
  Half<T> h;
  T *f = A.fields + (par ? A.fbuf : 0) + (int64_t)s * A.F6;
  h.ex = f;
  h.ey = f + A.F;
  h.ez = f + 2 * A.F;
  h.hx = f + 3 * A.F;
  h.hy = f + 4 * A.F;
  h.hz = f + 5 * A.F;
  T *ps = A.psi + (par ? A.pbuf : 0) + (int64_t)s * A.psi_src;
  h.psX = ps;
  h.psY = ps + A.oY;
  h.psZ = ps + A.oZ;
  return h;
}

// Vector of N consecutive x values of a field: N = 1 (one element per
// thread) or N = 16 / sizeof(T) (one 16-byte access per field)
template <typename T, int N_>
struct Vec {
  static constexpr int N = N_;
  T v[N];
};

template <int N, typename T>
__device__ __forceinline__ Vec<T, N> vload(const T *p) {
  Vec<T, N> r;
  if constexpr (N == 1) {
    r.v[0] = *p;
  } else if constexpr (sizeof(T) == 4) {
    static_assert(N == 4, "16-byte vectors");
    const float4 x = *reinterpret_cast<const float4 *>(p);
    r.v[0] = x.x; r.v[1] = x.y; r.v[2] = x.z; r.v[3] = x.w;
  } else {
    static_assert(N == 2, "16-byte vectors");
    const double2 x = *reinterpret_cast<const double2 *>(p);
    r.v[0] = x.x; r.v[1] = x.y;
  }
  return r;
}

template <typename T, int N>
__device__ __forceinline__ void vstore(T *p, const Vec<T, N> &r) {
  if constexpr (N == 1) {
    *p = r.v[0];
  } else if constexpr (sizeof(T) == 4) {
    *reinterpret_cast<float4 *>(p) = make_float4(r.v[0], r.v[1], r.v[2], r.v[3]);
  } else {
    *reinterpret_cast<double2 *>(p) = make_double2(r.v[0], r.v[1]);
  }
}

// Non-temporal store of a vector: for data that the next touch reads from
// HBM anyway (a field half read one step later, a history sample read at
// the block's close).  On the large grids the streaming hint took the H
// update from 2.22 to 2.10 ms and the E update from 3.12 to 3.00 ms per
// launch (8 sources, 32 M cells); the same hint on loads made them slower,
// and on the accumulators of the block transform it gained under 1 %.
// Where the whole working set stays in the Infinity Cache (the marine grid)
// it costs 15-20 %, so the update kernels take it as a template parameter
// chosen per run (StepArgs::nts); a run-time branch between the two store
// forms is merged by the compiler into one plain store.
template <typename T, int N>
__device__ __forceinline__ void vstore_nt(T *p, const Vec<T, N> &r) {
  if constexpr (N == 1) {
    __builtin_nontemporal_store(r.v[0], p);
  } else if constexpr (sizeof(T) == 4) {
    typedef float f4v __attribute__((ext_vector_type(4)));
    const f4v x = {r.v[0], r.v[1], r.v[2], r.v[3]};
    __builtin_nontemporal_store(x, reinterpret_cast<f4v *>(p));
  } else {
    typedef double d2v __attribute__((ext_vector_type(2)));
    const d2v x = {r.v[0], r.v[1]};
    __builtin_nontemporal_store(x, reinterpret_cast<d2v *>(p));
  }
}

template <bool NT, typename T, int N>
__device__ __forceinline__ void vstore_h(T *p, const Vec<T, N> &r) {
  if constexpr (NT)
    vstore_nt(p, r);
  else
    vstore(p, r);
}

template <typename T, int N>
__device__ __forceinline__ Vec<T, N> vzero() {
  Vec<T, N> r;
#pragma unroll
  for (int e = 0; e < N; ++e) r.v[e] = T(0);
  return r;
}

template <typename T>
__device__ __forceinline__ Vec<T, 1> vec1(T x) {
  Vec<T, 1> r;
  r.v[0] = x;
  return r;
}

template <typename T>
__device__ __forceinline__ T axv(const StepArgs<T> &A, int a, int t, int i) {
  return A.axt[(a * AX_TABLES + t) * A.LA + i];
}

// ---------------------------------------------------------------------------
// Per-node arithmetic shared by both schedules.  Explicit fused multiply-adds
// fix the rounding, so both schedules give the same bits whatever the
// compiler would contract.
// ---------------------------------------------------------------------------
// CPML-stretched derivative: psi <- b psi + a d; returns d / kappa + psi
template <typename T>
__device__ __forceinline__ T stretch(T d, T &psi, T b, T a, T kinv) {
  psi = fma(b, psi, a * d);
  return fma(d, kinv, psi);
}

// H^{n+1/2} = H^{n-1/2} - dt/mu (d1 - d2), forward differences over a cell
//   H_x: d1 = dEz/dy, d2 = dEy/dz   H_y: d1 = dEx/dz, d2 = dEz/dx
//   H_z: d1 = dEy/dx, d2 = dEx/dy
template <typename T>
__device__ __forceinline__ T hx_node(const StepArgs<T> &A, int j, int k, T h, T ez, T ez_jp, T ey,
                                     T ey_kp, bool py, T &psy, bool pz, T &psz) {
  T d1 = (ez_jp - ez) * axv(A, 1, AX_IH, j);
  T d2 = (ey_kp - ey) * axv(A, 2, AX_IH, k);
  if (py) d1 = stretch(d1, psy, axv(A, 1, AX_BH, j), axv(A, 1, AX_AH, j), axv(A, 1, AX_KH, j));
  if (pz) d2 = stretch(d2, psz, axv(A, 2, AX_BH, k), axv(A, 2, AX_AH, k), axv(A, 2, AX_KH, k));
  return fma(-A.dtmu, d1 - d2, h);
}
template <typename T>
__device__ __forceinline__ T hy_node(const StepArgs<T> &A, int i, int k, T h, T ex, T ex_kp, T ez,
                                     T ez_ip, bool pz, T &psz, bool px, T &psx) {
  T d1 = (ex_kp - ex) * axv(A, 2, AX_IH, k);
  T d2 = (ez_ip - ez) * axv(A, 0, AX_IH, i);
  if (pz) d1 = stretch(d1, psz, axv(A, 2, AX_BH, k), axv(A, 2, AX_AH, k), axv(A, 2, AX_KH, k));
  if (px) d2 = stretch(d2, psx, axv(A, 0, AX_BH, i), axv(A, 0, AX_AH, i), axv(A, 0, AX_KH, i));
  return fma(-A.dtmu, d1 - d2, h);
}
template <typename T>
__device__ __forceinline__ T hz_node(const StepArgs<T> &A, int i, int j, T h, T ey, T ey_ip, T ex,
                                     T ex_jp, bool px, T &psx, bool py, T &psy) {
  T d1 = (ey_ip - ey) * axv(A, 0, AX_IH, i);
  T d2 = (ex_jp - ex) * axv(A, 1, AX_IH, j);
  if (px) d1 = stretch(d1, psx, axv(A, 0, AX_BH, i), axv(A, 0, AX_AH, i), axv(A, 0, AX_KH, i));
  if (py) d2 = stretch(d2, psy, axv(A, 1, AX_BH, j), axv(A, 1, AX_AH, j), axv(A, 1, AX_KH, j));
  return fma(-A.dtmu, d1 - d2, h);
}

// E^{n+1} = E^n + dt/eps (d1 - d2), backward differences over a dual width
//   E_x: d1 = dHz/dy, d2 = dHy/dz   E_y: d1 = dHx/dz, d2 = dHz/dx
//   E_z: d1 = dHy/dx, d2 = dHx/dy
template <typename T>
__device__ __forceinline__ T ex_node(const StepArgs<T> &A, int j, int k, T e, T c, T hz, T hz_jm,
                                     T hy, T hy_km, bool py, T &psy, bool pz, T &psz) {
  T d1 = (hz - hz_jm) * axv(A, 1, AX_IHD, j);
  T d2 = (hy - hy_km) * axv(A, 2, AX_IHD, k);
  if (py) d1 = stretch(d1, psy, axv(A, 1, AX_BN, j), axv(A, 1, AX_AN, j), axv(A, 1, AX_KN, j));
  if (pz) d2 = stretch(d2, psz, axv(A, 2, AX_BN, k), axv(A, 2, AX_AN, k), axv(A, 2, AX_KN, k));
  return fma(c, d1 - d2, e);
}
template <typename T>
__device__ __forceinline__ T ey_node(const StepArgs<T> &A, int i, int k, T e, T c, T hx, T hx_km,
                                     T hz, T hz_im, bool pz, T &psz, bool px, T &psx) {
  T d1 = (hx - hx_km) * axv(A, 2, AX_IHD, k);
  T d2 = (hz - hz_im) * axv(A, 0, AX_IHD, i);
  if (pz) d1 = stretch(d1, psz, axv(A, 2, AX_BN, k), axv(A, 2, AX_AN, k), axv(A, 2, AX_KN, k));
  if (px) d2 = stretch(d2, psx, axv(A, 0, AX_BN, i), axv(A, 0, AX_AN, i), axv(A, 0, AX_KN, i));
  return fma(c, d1 - d2, e);
}
template <typename T>
__device__ __forceinline__ T ez_node(const StepArgs<T> &A, int i, int j, T e, T c, T hy, T hy_im,
                                     T hx, T hx_jm, bool px, T &psx, bool py, T &psy) {
  T d1 = (hy - hy_im) * axv(A, 0, AX_IHD, i);
  T d2 = (hx - hx_jm) * axv(A, 1, AX_IHD, j);
  if (px) d1 = stretch(d1, psx, axv(A, 0, AX_BN, i), axv(A, 0, AX_AN, i), axv(A, 0, AX_KN, i));
  if (py) d2 = stretch(d2, psy, axv(A, 1, AX_BN, j), axv(A, 1, AX_AN, j), axv(A, 1, AX_KN, j));
  return fma(c, d1 - d2, e);
}

// One walk of a thread's entry list (entry format with inject_value below)
// for every injection of kind 0 into its own nodes: per component c and
// vector element e, slot c * VX + e, summed in entry order with the fused
// multiply-adds of inject_value, so both give the same bits.  Used by the E
// update (J') and, on its own grid, by the H update (magnetic M').
template <typename T, int VX>
__device__ __forceinline__ void inject_all(const StepArgs<T> &A, int lo, int hi, int s, int n,
                                           double (&inj)[3 * VX]) {
#pragma unroll
  for (int q = 0; q < 3 * VX; ++q) inj[q] = 0.0;
  for (int e = lo; e < hi; ++e) {
    const int2 en = A.tl_ent[e];
    if ((en.x & 4) || (en.x >> 9) != s) continue;           // kind 0 of this source
    const int slot = (en.x & 3) * VX + ((en.x >> 3) & 63);
    double cur = 0.0;
#pragma unroll
    for (int q = 0; q < 3 * VX; ++q) cur = q == slot ? inj[q] : cur;
    const double *cf = A.coef + en.y;
#pragma unroll 4
    for (int r = 0; r < A.nrow; ++r) cur = fma(cf[r], A.Ftab[(int64_t)r * A.nt + n], cur);
#pragma unroll
    for (int q = 0; q < 3 * VX; ++q) inj[q] = q == slot ? cur : inj[q];
  }
}

// Magnetic adjoint source M'^n (Faraday row of eq. fictitiouswave) added to
// H^{n-1/2} of the thread's own nodes before their update: the arithmetic
// of k_hinj, (T)(H + (dt/mu) M'), on the values in registers.  Nodes with
// no entry are left alone.
template <typename T, int VX>
__device__ __forceinline__ void inject_h(const StepArgs<T> &A, int lo, int hi, int s, int n,
                                         Vec<T, VX> &hx, Vec<T, VX> &hy, Vec<T, VX> &hz) {
  double inj[3 * VX];
  inject_all<T, VX>(A, lo, hi, s, n, inj);
#pragma unroll
  for (int e = 0; e < VX; ++e) {
    if (inj[e] != 0.0) hx.v[e] = (T)((double)hx.v[e] + A.dtmu64 * inj[e]);
    if (inj[VX + e] != 0.0) hy.v[e] = (T)((double)hy.v[e] + A.dtmu64 * inj[VX + e]);
    if (inj[2 * VX + e] != 0.0) hz.v[e] = (T)((double)hz.v[e] + A.dtmu64 * inj[2 * VX + e]);
  }
}

// Interior tile of the two-kernel schedule (uniform per block): every node of
// the block lies at least npml nodes from the low walls and npml + 1 from
// the high ones (so it is no CPML node, and every H component and E edge it
// owns is updated), on a plane of the same kind.  Such blocks take the lean
// paths below; A.lean is off when npml == 0 (walls next to the interior).
template <typename T>
__device__ __forceinline__ bool interior_tile(const StepArgs<T> &A, int bx, int by, int k, int wx) {
  const int wy = blockDim.y;
  return A.lean && k >= A.npml && k < A.nz - A.npml && bx * wx >= A.npml &&
         (bx + 1) * wx <= A.nx - A.npml && by * wy >= A.npml && (by + 1) * wy <= A.ny - A.npml;
}

// ---------------------------------------------------------------------------
// H update (two-kernel schedule): each thread owns VX consecutive x nodes
// (one 16-byte vector per field); the x neighbour beyond the vector is one
// extra element load.  All loads are issued before any store (loads and
// stores share one in-order completion counter on this GPU).
// ---------------------------------------------------------------------------
// LEAN: the block's tile is interior (see interior_tile): every lattice mask
// and bounds test is true and no node is inside a CPML layer, as compile-time
// constants; the per-node arithmetic is the same helpers' (same bits).
template <typename T, int VX, bool INJ, bool LEAN, bool NT = false>
__device__ __forceinline__ void h_vec(const StepArgs<T> &A, const Half<T> &I, const Half<T> &O,
                                      int i0, int j, int k, int lo, int hi, int s, int n) {
  using V = Vec<T, VX>;
  const int PX = A.PX, NY = A.NY, npml = A.npml, W = 2 * npml;
  const int64_t plane = A.plane;
  const int64_t sX = A.sX, sY = A.sY, sZ = A.sZ;
  const bool j_in = LEAN || j < A.ny, k_in = LEAN || k < A.nz;
  int ly = 0, lz = 0;
  const bool py = !LEAN && npml > 0 && pml_half(j, A.ny, npml, ly);
  const bool pz = !LEAN && npml > 0 && pml_half(k, A.nz, npml, lz);
  const bool pyv = py && j_in, pzv = pz && k_in;
  const int64_t q = (int64_t)k * plane + (int64_t)j * PX + i0;
  const bool nbr = LEAN || i0 + VX <= A.nx;   // the x neighbour of the last element is used
  // ---- loads ----
  const V ex0 = vload<VX>(I.ex + q), ey0 = vload<VX>(I.ey + q), ez0 = vload<VX>(I.ez + q);
  const V exk = k_in ? vload<VX>(I.ex + q + plane) : vzero<T, VX>();
  const V eyk = k_in ? vload<VX>(I.ey + q + plane) : vzero<T, VX>();
  const V ezj = j_in ? vload<VX>(I.ez + q + PX) : vzero<T, VX>();
  const V exj = j_in ? vload<VX>(I.ex + q + PX) : vzero<T, VX>();
  const T eyn = nbr ? I.ey[q + VX] : T(0), ezn = nbr ? I.ez[q + VX] : T(0);
  V hxv = vload<VX>(I.hx + q), hyv = vload<VX>(I.hy + q), hzv = vload<VX>(I.hz + q);
  const int64_t iY = ((int64_t)k * W + ly) * PX + i0;
  const int64_t iZ = ((int64_t)lz * NY + j) * PX + i0;
  V ps_hx_y = pyv && k_in ? vload<VX>(I.psY + 0 * sY + iY) : vzero<T, VX>();
  V ps_hz_y = pyv ? vload<VX>(I.psY + 1 * sY + iY) : vzero<T, VX>();
  V ps_hx_z = pzv && j_in ? vload<VX>(I.psZ + 0 * sZ + iZ) : vzero<T, VX>();
  V ps_hy_z = pzv ? vload<VX>(I.psZ + 1 * sZ + iZ) : vzero<T, VX>();
  if constexpr (INJ)
    if (lo < hi) inject_h<T, VX>(A, lo, hi, s, n, hxv, hyv, hzv);
  // ---- compute ----
#pragma unroll
  for (int e = 0; e < VX; ++e) {
    const int i = i0 + e;
    const bool i_in = LEAN || i < A.nx;
    const T ey_ip = e + 1 < VX ? ey0.v[(e + 1) % VX] : eyn;
    const T ez_ip = e + 1 < VX ? ez0.v[(e + 1) % VX] : ezn;
    int lx = 0;
    const bool px = !LEAN && npml > 0 && i_in && pml_half(i, A.nx, npml, lx);
    const int64_t iX = ((int64_t)k * NY + j) * W + lx;
    if (LEAN || (i <= A.nx && j_in && k_in))
      hxv.v[e] = hx_node(A, j, k, hxv.v[e], ez0.v[e], ezj.v[e], ey0.v[e], eyk.v[e], py,
                         ps_hx_y.v[e], pz, ps_hx_z.v[e]);
    if (i_in && k_in) {
      T ps = px ? I.psX[0 * sX + iX] : T(0);
      hyv.v[e] = hy_node(A, i, k, hyv.v[e], ex0.v[e], exk.v[e], ez0.v[e], ez_ip, pz, ps_hy_z.v[e],
                         px, ps);
      if (px) O.psX[0 * sX + iX] = ps;
    }
    if (i_in && j_in) {
      T ps = px ? I.psX[1 * sX + iX] : T(0);
      hzv.v[e] = hz_node(A, i, j, hzv.v[e], ey0.v[e], ey_ip, ex0.v[e], exj.v[e], px, ps, py,
                         ps_hz_y.v[e]);
      if (px) O.psX[1 * sX + iX] = ps;
    }
  }
  // ---- stores (slots outside a component's lattice keep their zero) ----
  vstore_h<NT>(O.hx + q, hxv);
  vstore_h<NT>(O.hy + q, hyv);
  vstore_h<NT>(O.hz + q, hzv);
  if (pyv && k_in) vstore(O.psY + 0 * sY + iY, ps_hx_y);
  if (pyv) vstore(O.psY + 1 * sY + iY, ps_hz_y);
  if (pzv && j_in) vstore(O.psZ + 0 * sZ + iZ, ps_hx_z);
  if (pzv) vstore(O.psZ + 1 * sZ + iZ, ps_hy_z);
}

// INJ: adjoint runs with magnetic receivers (the H update adds the magnetic
// sources of its nodes); otherwise the plain update.  NT: streaming stores.
template <typename T, int VX, bool INJ, bool NT>
__global__ void __launch_bounds__(256) k_update_h(StepArgs<T> A) {
  int bx, by, bz, s;
  const int b = tile_of(A, bx, by, bz, s);
  const int n = step_of(A, false);
  const int par = n & 1;                 // this step reads half par
  const int i0 = (bx * blockDim.x + threadIdx.x) * VX;
  const int j = by * blockDim.y + threadIdx.y;
  const int k = bz;
  if (i0 > A.nx || j > A.ny || k > A.nz) return;
  int lo = 0, hi = 0;
  if constexpr (INJ) entry_slice(A, b, n, lo, hi);
  if (interior_tile(A, bx, by, k, blockDim.x * VX))
    h_vec<T, VX, INJ, true, NT>(A, half_of(A, par, s), half_of(A, par ^ 1, s), i0, j,
                                __builtin_amdgcn_readfirstlane(k), lo, hi, s, n);
  else
    h_vec<T, VX, INJ, false, NT>(A, half_of(A, par, s), half_of(A, par ^ 1, s), i0, j, k, lo, hi,
                                 s, n);
}

// ---------------------------------------------------------------------------
// accumulator flavours for the volume transform acc += E z (eq. dft)
// ---------------------------------------------------------------------------
enum { ACC_NONE = 0, ACC_F64 = 1, ACC_KAHAN = 2, ACC_F32 = 3 };

template <int ACC>
__device__ __forceinline__ double2 acc_read(const void *base, int64_t idx) {
  if constexpr (ACC == ACC_F64) {
    return reinterpret_cast<const double2 *>(base)[idx];
  } else if constexpr (ACC == ACC_KAHAN) {
    const float4 v = reinterpret_cast<const float4 *>(base)[idx];
    return make_double2((double)v.x - (double)v.z, (double)v.y - (double)v.w);
  } else {
    const float2 v = reinterpret_cast<const float2 *>(base)[idx];
    return make_double2((double)v.x, (double)v.y);
  }
}

// Accumulator flavours as load / add / store, so that the block transform
// can issue all its loads before any store (loads and stores share one
// in-order completion counter: a load behind a store waits for the store).
// Compensated FP32 keeps (hi, lo) per real component, the sum being hi - lo
// (Kahan's running compensation).
template <int ACC>
struct Acc;
template <>
struct Acc<ACC_F64> {
  using S = double2;
  static __device__ __forceinline__ S zero() { return make_double2(0.0, 0.0); }
  static __device__ __forceinline__ S load(const void *b, int64_t i) {
    return reinterpret_cast<const double2 *>(b)[i];
  }
  static __device__ __forceinline__ void store(void *b, int64_t i, S v) {
    reinterpret_cast<S *>(b)[i] = v;
  }
  static __device__ __forceinline__ S add(S v, double2 x) {
    v.x += x.x;
    v.y += x.y;
    return v;
  }
  static __device__ __forceinline__ double2 value(S v) { return v; }
};
template <>
struct Acc<ACC_KAHAN> {
  using S = float4;
  static __device__ __forceinline__ S zero() { return make_float4(0.f, 0.f, 0.f, 0.f); }
  static __device__ __forceinline__ S load(const void *b, int64_t i) {
    return reinterpret_cast<const float4 *>(b)[i];
  }
  static __device__ __forceinline__ void store(void *b, int64_t i, S v) {
    reinterpret_cast<S *>(b)[i] = v;
  }
  static __device__ __forceinline__ S add(S v, double2 x) {
    const float xr = (float)x.x, xi = (float)x.y;
    float yr = xr - v.z, tr = v.x + yr;
    v.z = (tr - v.x) - yr;
    v.x = tr;
    float yi = xi - v.w, ti = v.y + yi;
    v.w = (ti - v.y) - yi;
    v.y = ti;
    return v;
  }
  static __device__ __forceinline__ double2 value(S v) {
    return make_double2((double)v.x - (double)v.z, (double)v.y - (double)v.w);
  }
};
template <>
struct Acc<ACC_F32> {
  using S = float2;
  static __device__ __forceinline__ S zero() { return make_float2(0.f, 0.f); }
  static __device__ __forceinline__ S load(const void *b, int64_t i) {
    return reinterpret_cast<const float2 *>(b)[i];
  }
  static __device__ __forceinline__ void store(void *b, int64_t i, S v) {
    reinterpret_cast<S *>(b)[i] = v;
  }
  static __device__ __forceinline__ S add(S v, double2 x) {
    v.x += (float)x.x;
    v.y += (float)x.y;
    return v;
  }
  static __device__ __forceinline__ double2 value(S v) {
    return make_double2((double)v.x, (double)v.y);
  }
};

// After the E update of the three components at q .. q+VX-1 (new values e1
// = sample m = n+1 of eq. dft): the samples of the current transform block
// wait in the history buffer until the block closes; with decimation D =
// 2^dl only samples m = jD enter, and sample j with j % KB = r (1 .. KB-1)
// goes to slot r-1 (D = 1: j = m).  The closing sample (r = 0) stays in the
// field buffer, where the block transform k_transform reads it.
// Elements outside a component's lattice (ok bit clear) keep garbage that
// k_transform never reads; steps past the run keep nothing.
template <typename T, int VX, bool NT = false>
__device__ __forceinline__ void hist_store(const StepArgs<T> &A, int s, int64_t q,
                                           const Vec<T, VX> (&e1)[3], const unsigned (&ok)[3],
                                           int n) {
  const int kb = A.kb, m = n + 1;
  if (kb <= 1 || n >= A.nt || !(ok[0] | ok[1] | ok[2])) return;
  if (m & ((1 << A.dl) - 1)) return;
  const int r = (m >> A.dl) & (kb - 1);
  if (r == 0) return;
  T *h = A.hist + (int64_t)s * A.hist_src + q + (int64_t)(r - 1) * 3 * A.F;
#pragma unroll
  for (int c = 0; c < 3; ++c)
    if (ok[c]) vstore_h<NT>(h + c * A.F, e1[c]);
}

// per-thread list walk.  Entry x = c | kind << 2 | sub << 3 | s << 9, where
// sub is the vector element (two-kernel schedule) or the plane within the
// block's chunk (fused schedule): kind 0 = injection J'^{n+1/2} into
// component c of source s, value sum_r coef[ref + r] F[r][n]; kind 1 =
// receiver node (racc[s][node = ref] += E^{n+1} z^{n+1}, every source);
// kind 1 with c = 3 = H receiver node (two-kernel schedule: the E update of
// step n holds H^{n+1/2} of its own node, its curl operand, and adds
// H^{n+1/2} z^{n+1/2} for the node's H component, rn_c[ref]).
template <typename T>
__device__ __forceinline__ double inject_value(const StepArgs<T> &A, int lo, int hi, int s, int c,
                                               int sub, int n) {
  double v = 0.0;
  for (int e = lo; e < hi; ++e) {
    const int2 en = A.tl_ent[e];
    if ((en.x & 511) == (c | (sub << 3)) && (en.x >> 9) == s) {
      const double *cf = A.coef + en.y;
      for (int r = 0; r < A.nrow; ++r) v = fma(cf[r], A.Ftab[(int64_t)r * A.nt + n], v);
    }
  }
  return v;
}

// The same walks done once per thread (two-kernel schedule): every thread
// that owns entries makes one pass before the update for all injections
// (inject_all, with the H update above) and one pass after it for all
// records (E nodes with E^{n+1} z^{n+1}, H nodes with H^{n+1/2} z^{n+1/2}).
// Each walk costs dependent memory round trips, and the threads of the
// receiver and source tiles set the tail of the launch.
template <typename T, int VX>
__device__ __forceinline__ void record_all(const StepArgs<T> &A, int lo, int hi, int s, int n,
                                           const Vec<T, VX> (&e1)[3], const unsigned (&ok)[3],
                                           const Vec<T, VX> (&h)[3]) {
  for (int e2 = lo; e2 < hi; ++e2) {
    const int2 en = A.tl_ent[e2];
    if (!(en.x & 4)) continue;                                // kind 1: receiver node
    const int c = en.x & 3, sub = (en.x >> 3) & 63;
    const int ch = c < 3 ? -1 : A.rn_c[en.y] - 3;
    // select with compile-time indices only (no addressable arrays)
    T val = T(0);
    bool on = false;
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
      for (int e = 0; e < VX; ++e) {
        if (e != sub) continue;
        if (q == c) {
          val = e1[q].v[e];
          on = (ok[q] >> e) & 1u;
        }
        if (q == ch) {
          val = h[q].v[e];
          on = true;
        }
      }
    if (!on) continue;
    const double v = (double)val;
    // the sums and the twiddles never overlap: their loads can be issued
    // together
    double2 *__restrict__ a = A.racc + ((int64_t)s * A.nn + en.y) * A.nf;
    const double2 *__restrict__ z = (c < 3 ? A.zE : A.zH) + (int64_t)n * A.nf;
#pragma unroll 4
    for (int kf = 0; kf < A.nf; ++kf) {
      double2 x = a[kf];
      x.x = fma(v, z[kf].x, x.x);
      x.y = fma(v, z[kf].y, x.y);
      a[kf] = x;
    }
  }
}

template <typename T>
__device__ __forceinline__ void record(const StepArgs<T> &A, int lo, int hi, int s, int c,
                                       int sub, int n, double e) {
  for (int e2 = lo; e2 < hi; ++e2) {
    const int2 en = A.tl_ent[e2];
    if ((en.x & 511) == (c | 4 | (sub << 3))) {
      double2 *a = A.racc + ((int64_t)s * A.nn + en.y) * A.nf;
      const double2 *z = A.zE + (int64_t)n * A.nf;
      for (int kf = 0; kf < A.nf; ++kf) {
        double2 v = a[kf];
        v.x = fma(e, z[kf].x, v.x);
        v.y = fma(e, z[kf].y, v.y);
        a[kf] = v;
      }
    }
  }
}

// ---------------------------------------------------------------------------
// E update (two-kernel schedule): E^{n+1} from E^n (half par) and H^{n+1/2}
// (half par ^ 1) on interior edges, written to half par ^ 1.  Fused:
// injection at the source (or adjoint-source) edges, the receiver
// transform, and the volume transform / gradient product.  Each thread owns
// VX consecutive x nodes; the x neighbour before the vector is one extra
// element load; all stencil loads precede the stores.
// ---------------------------------------------------------------------------
template <typename T, bool HIST, int VX, bool LEAN, bool NT = false>
__device__ __forceinline__ void e_vec(const StepArgs<T> &A, int s, int b, const Half<T> &I,
                                      const Half<T> &O, const Half<T> &P, int i0, int j, int k,
                                      int n) {
  using V = Vec<T, VX>;
  const int PX = A.PX, NY = A.NY, npml = A.npml, W = 2 * npml;
  const int64_t plane = A.plane;
  const int64_t sX = A.sX, sY = A.sY, sZ = A.sZ;
  const bool j_int = LEAN || (j >= 1 && j < A.ny), k_int = LEAN || (k >= 1 && k < A.nz);
  const bool j_in = LEAN || j < A.ny, k_in = LEAN || k < A.nz;
  int ly = 0, lz = 0;
  const bool py = !LEAN && npml > 0 && pml_int(j, A.ny, npml, ly);
  const bool pz = !LEAN && npml > 0 && pml_int(k, A.nz, npml, lz);
  const int64_t q = (int64_t)k * plane + (int64_t)j * PX + i0;
  // lattice masks per element
  unsigned okx = 0, oky = 0, okz = 0;
  if constexpr (LEAN) {
    okx = oky = okz = (1u << VX) - 1u;
  } else {
#pragma unroll
    for (int e = 0; e < VX; ++e) {
      const int i = i0 + e;
      if (i < A.nx && j_int && k_int) okx |= 1u << e;
      if (i >= 1 && i < A.nx && j_in && k_int) oky |= 1u << e;
      if (i >= 1 && i < A.nx && j_int && k_in) okz |= 1u << e;
    }
  }
  // ---- loads ----
  const V hx0 = vload<VX>(O.hx + q), hy0 = vload<VX>(O.hy + q), hz0 = vload<VX>(O.hz + q);
  const V hzj = LEAN || j >= 1 ? vload<VX>(O.hz + q - PX) : vzero<T, VX>();
  const V hxj = LEAN || j >= 1 ? vload<VX>(O.hx + q - PX) : vzero<T, VX>();
  const V hyk = LEAN || k >= 1 ? vload<VX>(O.hy + q - plane) : vzero<T, VX>();
  const V hxk = LEAN || k >= 1 ? vload<VX>(O.hx + q - plane) : vzero<T, VX>();
  const T hzp = LEAN || i0 >= 1 ? O.hz[q - 1] : T(0), hyp = LEAN || i0 >= 1 ? O.hy[q - 1] : T(0);
  const V e0x = vload<VX>(I.ex + q), e0y = vload<VX>(I.ey + q), e0z = vload<VX>(I.ez + q);
  const V cx = okx ? vload<VX>(A.ce + q) : vzero<T, VX>();
  const V cy = oky ? vload<VX>(A.ce + A.F + q) : vzero<T, VX>();
  const V cz = okz ? vload<VX>(A.ce + 2 * A.F + q) : vzero<T, VX>();
  const int64_t iY = ((int64_t)k * W + ly) * PX + i0;
  const int64_t iZ = ((int64_t)lz * NY + j) * PX + i0;
  V ps_ex_y = py && okx ? vload<VX>(P.psY + 2 * sY + iY) : vzero<T, VX>();
  V ps_ez_y = py && okz ? vload<VX>(P.psY + 3 * sY + iY) : vzero<T, VX>();
  V ps_ex_z = pz && okx ? vload<VX>(P.psZ + 2 * sZ + iZ) : vzero<T, VX>();
  V ps_ey_z = pz && oky ? vload<VX>(P.psZ + 3 * sZ + iZ) : vzero<T, VX>();
  int lo, hi;
  entry_slice(A, b, n, lo, hi);
  double inj[3 * VX];
  if (lo < hi) inject_all<T, VX>(A, lo, hi, s, n, inj);
  // ---- compute ----
  V e1x = e0x, e1y = e0y, e1z = e0z;
#pragma unroll
  for (int e = 0; e < VX; ++e) {
    const int i = i0 + e;
    const bool i_int = LEAN || (i >= 1 && i < A.nx);
    const T hz_im = e > 0 ? hz0.v[(e + VX - 1) % VX] : hzp;
    const T hy_im = e > 0 ? hy0.v[(e + VX - 1) % VX] : hyp;
    int lx = 0;
    const bool px = !LEAN && npml > 0 && i_int && pml_int(i, A.nx, npml, lx);
    const int64_t iX = ((int64_t)k * NY + j) * W + lx;
    if ((okx >> e) & 1u) {
      T v = ex_node(A, j, k, e0x.v[e], cx.v[e], hz0.v[e], hzj.v[e], hy0.v[e], hyk.v[e], py,
                    ps_ex_y.v[e], pz, ps_ex_z.v[e]);
      if (lo < hi) v -= (T)((double)cx.v[e] * inj[0 * VX + e]);
      e1x.v[e] = v;
    }
    if ((oky >> e) & 1u) {
      T dummy = T(0);
      T &psx = px ? P.psX[2 * sX + iX] : dummy;
      T v = ey_node(A, i, k, e0y.v[e], cy.v[e], hx0.v[e], hxk.v[e], hz0.v[e], hz_im, pz,
                    ps_ey_z.v[e], px, psx);
      if (lo < hi) v -= (T)((double)cy.v[e] * inj[1 * VX + e]);
      e1y.v[e] = v;
    }
    if ((okz >> e) & 1u) {
      T dummy = T(0);
      T &psx = px ? P.psX[3 * sX + iX] : dummy;
      T v = ez_node(A, i, j, e0z.v[e], cz.v[e], hy0.v[e], hy_im, hx0.v[e], hxj.v[e], px, psx, py,
                    ps_ez_y.v[e]);
      if (lo < hi) v -= (T)((double)cz.v[e] * inj[2 * VX + e]);
      e1z.v[e] = v;
    }
  }
  // ---- stores ----
  if (okx) vstore_h<NT>(O.ex + q, e1x);
  if (oky) vstore_h<NT>(O.ey + q, e1y);
  if (okz) vstore_h<NT>(O.ez + q, e1z);
  if (py && okx) vstore(P.psY + 2 * sY + iY, ps_ex_y);
  if (py && okz) vstore(P.psY + 3 * sY + iY, ps_ez_y);
  if (pz && okx) vstore(P.psZ + 2 * sZ + iZ, ps_ex_z);
  if (pz && oky) vstore(P.psZ + 3 * sZ + iZ, ps_ey_z);
  if (lo < hi) {
    const Vec<T, VX> e1[3] = {e1x, e1y, e1z}, hh[3] = {hx0, hy0, hz0};
    const unsigned ok[3] = {okx, oky, okz};
    record_all<T, VX>(A, lo, hi, s, n, e1, ok, hh);
  }
  // ---- the sample's place in the transform block ----
  if constexpr (HIST) {
    const Vec<T, VX> e1[3] = {e1x, e1y, e1z};
    const unsigned ok[3] = {okx, oky, okz};
    hist_store<T, VX, NT>(A, s, q, e1, ok, n);
  }
}

// HIST: the run takes the volume transform (forward) or the gradient
// product (adjoint): each sample is kept for the block transform.  NT:
// streaming stores.
template <typename T, bool HIST, int VX, bool NT>
__device__ __forceinline__ void e_update(const StepArgs<T> &A) {
  int bx, by, bz, s;
  const int b = tile_of(A, bx, by, bz, s);
  const int n = step_of(A, true);        // this launch completes step n
  const int i0 = (bx * blockDim.x + threadIdx.x) * VX;
  const int j = by * blockDim.y + threadIdx.y;
  const int k = bz;
  if (i0 <= A.nx && j <= A.ny && k <= A.nz) {
    const int par = n & 1;
    if (interior_tile(A, bx, by, k, blockDim.x * VX))
      e_vec<T, HIST, VX, true, NT>(A, s, b, half_of(A, par, s), half_of(A, par ^ 1, s),
                                   half_of(A, 0, s), i0, j, __builtin_amdgcn_readfirstlane(k), n);
    else
      e_vec<T, HIST, VX, false, NT>(A, s, b, half_of(A, par, s), half_of(A, par ^ 1, s),
                                    half_of(A, 0, s), i0, j, k, n);
  }
}

template <typename T, bool HIST, int VX, bool NT>
__global__ void __launch_bounds__(256) k_update_e(StepArgs<T> A) {
  e_update<T, HIST, VX, NT>(A);
}

// The streaming E update of FP32 fields, one node per thread, held to 64
// VGPRs so that 8 waves share a SIMD (the compiler's own choice, 65, allows
// 7; the scalar registers it gives up are spilled to VGPR lanes, not to
// memory).  On the large grid (8 sources) this took the launch from 3.00
// to 2.83 ms; on the marine grid, whose data stay in the Infinity Cache,
// the same form was 1 % slower, so it goes with the streaming stores.
template <bool HIST>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(8, 8)))
k_update_e_s(StepArgs<float> A) {
  e_update<float, HIST, 1, true>(A);
}

// ---------------------------------------------------------------------------
// One-launch step (schedule 0 at order 2, k_leap).  A wave owns 64 consecutive
// x nodes of one row (j, k).  Each lane computes H^{n+1/2} at its node and
// again at the neighbours that its E edges difference, (j - 1) and (k - 1),
// with the operands and operations of their owners (the same bits); H at
// i - 1 comes from the lane below, and only the first lane recomputes it.
// Then E^{n+1}, in registers: no barrier, no LDS, and H^{n+1/2} is written
// but not read back, so a step moves 48 B a node (FP32) for the 72 B of two
// launches.
//
// What bounds it: instruction issue, and behind it L2.  The two kernels took
// 250 to 320 scalar instructions a wave against 133 to 223 vector ones
// (SQ_INSTS_*; the scalar unit of a CU serves its four SIMDs in turn), most of
// them 64-bit addresses.  Hence: j and k are uniform (one row per wave), so
// rows, layers and coefficients are scalar; every row is a 32-bit offset on
// one buffer descriptor (a scalar add a row, 25 rows); the layers' branches
// cost nothing off the layers; and three quarters of a large grid take the
// form with none.  A wave issues 299 scalar, 233 vector and 66 vector memory
// instructions on average on 101x101x61 (issue bounds it there) and 229, 158
// and 56 on 200x200x100 with 8 sources, where the texture addresser is busy
// 85 % of the launch (41 % on 101x101x61): waves of 62 own nodes, whose end
// lanes carry the neighbours instead of one-lane loads, took 15 % fewer
// instructions, but their rows leave the 128-byte lines (20.9 -> 24.3 ms
// there; 12.25 -> 11.4 on 101x101x61 with 4 sources): not kept.
// Rows of the high walls are not computed: H there stays zero (it
// differences E edges on the wall), and E there is never updated.
//
// Measured a step, two kernels -> this (one MI355X): 101x101x61 FP32, the
// kernels alone, with the history sample, 30.1 -> 17.2 us; without a volume, a
// run's time over its steps: the same grid with 4 sources 77.0 -> 47.5 us,
// 200x200x100 with 8 sources 967 -> 644 us (2.9 TB/s of the 1.89 GB it cannot
// do without), 400x400x200 with 8 sources 5.71 -> 4.40 ms; FP64 128x128x96
// 90.5 -> 63.4 us, 400x400x200 1395 -> 1299 us.  Not kept: 2 nodes a lane
// (FP32; 20.5 us on the marine grid), a march in z with H of the plane below
// carried (slower below 32 M node updates a step, 3 % faster above), blocks
// of 4 rows (5 to 10 % slower than one-wave blocks), holding the layers'
// forms to fewer registers (5 waves a SIMD for 4: no gain).
// ---------------------------------------------------------------------------
// Coefficients of one axis index, read as one row: 1/h, 1/hd, then CPML
// 1/kappa, b, a at the node and at the half node.
template <typename T>
struct AxRow {
  T ih, ihd, kn, bn, an, kh, bh, ah;
};

// Raw buffer access: uniform base and 32-bit uniform row offset in scalar
// registers, the lane's offset in one vector register, so that each of the
// many rows of a stencil costs one scalar addition.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc_of(const void *p) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, 0xffffffffu, 0x00027000);
}
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
template <typename T>
__device__ __forceinline__ T bload(__amdgpu_buffer_rsrc_t r, uint32_t lane, uint32_t row) {
  if constexpr (sizeof(T) == 4)
    return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, lane, row, 0));
  else
    return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, lane, row, 0));
}
template <bool NT, typename T>
__device__ __forceinline__ void bstore(T v, __amdgpu_buffer_rsrc_t r, uint32_t lane, uint32_t row) {
  constexpr int aux = NT ? 2 : 0;        // bit 1: non-temporal
  if constexpr (sizeof(T) == 4)
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, lane, row, aux);
  else
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, lane, row, aux);
}

// The value of the lane below / above (one lane along x); the first / last
// active lane keeps `edge`.
template <int CTRL, typename T>
__device__ __forceinline__ T lane_shift(T edge, T v) {
  if constexpr (sizeof(T) == 4) {
    return __builtin_bit_cast(T, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, edge),
                                                             __builtin_bit_cast(int, v), CTRL, 0xf,
                                                             0xf, false));
  } else {
    const u32x2 e = __builtin_bit_cast(u32x2, edge), u = __builtin_bit_cast(u32x2, v);
    u32x2 r;
    r.x = __builtin_amdgcn_update_dpp((int)e.x, (int)u.x, CTRL, 0xf, 0xf, false);
    r.y = __builtin_amdgcn_update_dpp((int)e.y, (int)u.y, CTRL, 0xf, 0xf, false);
    return __builtin_bit_cast(T, r);
  }
}
template <typename T>
__device__ __forceinline__ T lane_below(T edge, T v) { return lane_shift<0x138>(edge, v); }
template <typename T>
__device__ __forceinline__ T lane_above(T edge, T v) { return lane_shift<0x130>(edge, v); }

// b, a and 1/kappa of a stretched difference
template <typename T>
struct Stretch {
  T b, a, k;
};

// fma(c, d1 - d2, f) with d1 = (a1 - a0) s1 and d2 = (b1 - b0) s2, each
// stretched inside a layer: the update of every component (c = -dt/mu for H,
// dt/eps for E).  P1, P2: the direction can be stretched at all; p1, p2: it
// is at this node.
template <bool P1, bool P2, typename T>
__device__ __forceinline__ T curl_update(T f, T c, T a1, T a0, T s1, bool p1, T &m1,
                                         const Stretch<T> &t1, T b1, T b0, T s2, bool p2, T &m2,
                                         const Stretch<T> &t2) {
  T d1 = (a1 - a0) * s1;
  T d2 = (b1 - b0) * s2;
  if constexpr (P1) {
    const T d = stretch(d1, m1, t1.b, t1.a, t1.k);
    d1 = p1 ? d : d1;
  }
  if constexpr (P2) {
    const T d = stretch(d2, m2, t2.b, t2.a, t2.k);
    d2 = p2 ? d : d2;
  }
  return fma(c, d1 - d2, f);
}

template <typename T>
struct LeapArgs {
  T *f0, *f1, *p0, *p1;              // halves of the fields and of the CPML memory (E's: half 0)
  const T *ce, *axt;
  const AxRow<T> *axr;               // [3][LA]
  T *hist;                           // slot of this step's sample (HIST)
  const int *step;
  int *step_w;
  int64_t F6, psi_src, hist_src;     // elements per source
  uint32_t PXb, PLb, Fb, LAb;        // row, plane, field and axis table strides in bytes
  uint32_t sXb, sYb, sZb, oYb, oZb;  // psi slab strides and offsets in bytes
  int nx, ny, nz, npml, LA, NY;
  T dtmu;
  int ns, order;
  uint32_t runs;                     // blocks in whole rounds of runs (0: not remapped)
  FDiv dns, d1, d2;                  // sources, tiles along the fastest and the next axis
  // first and number of the wave starts i0, rows j and planes k that hold
  // neither a layer nor a wall within the stencil's reach
  uint32_t xs, xn, ys, yn, zs, zn;
  // injections and receivers by row (see build_rows): of each row its receiver
  // table, of each row of the box below and source its source table, or -1
  // (adjoint runs: null)
  const int *row_tab, *src_tab;
  const int *row_rec;                // [tables][6][64] receiver node of the lane's component, or -1
  const int *row_src;                // [tables][3][64] first coefficient of its injection, or -1
  int rec_mask;                      // components that have receiver nodes at all (Ex .. Hz)
  int adj;                           // adjoint run: the E receiver nodes are the injections
  uint32_t ej, ejn, ek, ekn;         // first and number of the rows and planes they span
  uint32_t nbx;                      // tiles of a row
};

// The step a launch computes, from the counter in the workspace, and the
// halves that it reads and writes: a captured launch may be replayed, and a
// plan may step several workspaces in turn, so the host's count decides
// nothing here.  No field can be read before it: its load is kept before the
// block decode, and nothing that ends a lane stands between them and the
// variants, so that all arguments come in one wait and the counter's and the
// rows' tables in the next (ms: 32x32x32 FP64, 512 steps, 2.87 -> 2.82;
// 101x101x61 gradient 22.39 -> 22.13, with 4 sources 12.23 -> 12.15; with the
// halves chosen by the host, wrong in a replay, 2.76, 22.3 and 12.0).
template <typename T>
struct Place {
  int n;
  const T *fi, *pi;
  T *fo, *po;
};
template <typename T>
__device__ __forceinline__ Place<T> place_of(const LeapArgs<T> &L) {
  const int n = L.step[0] + 1;
  const bool odd = n & 1;
  return {n, odd ? L.f1 : L.f0, odd ? L.p1 : L.p0, odd ? L.f0 : L.f1, odd ? L.p0 : L.p1};
}

// Block -> (64-node tile of x, row, plane, source) and the row's index, for
// rows of waves: as tile_of, but each XCD takes runs of 128 consecutive b,
// dealt round-robin, and the blocks past the last whole round stay where they
// are.  Rows of a run still share their neighbours in one L2, and every XCD
// gets its part of the layers, whose rows cost twice as much: with one
// contiguous range per XCD the XCDs of the outermost planes finish last (when
// the runs were introduced: 101x101x61, 4 sources, 53.5 us a step against 47.5
// with runs and 47.3 unmapped; 1 source 17.5, 17.2 and 19.7; runs of 16 to 1024
// within 4 %).  The decode has no branches.  The
// scalar work before a wave's first load was 40 % of an interior wave's
// instructions, so its limits and divisors come ready from the host (ms before
// and after: 128x128x96 FP64 9.95 -> 9.65, 200x200x100 with 8 sources 20.9 ->
// 20.4, 101x101x61 with 4 sources 12.25 -> 12.0, FP32 grids of some 10^4 cells
// 2 to 12 % less).
enum { XCD_RUN_LOG2 = 7 };
template <typename T>
__device__ __forceinline__ int row_of(const LeapArgs<T> &L, int &bx, int &j, int &k, int &s) {
  constexpr uint32_t g = XCD_RUN_LOG2;
  uint32_t b = blockIdx.x;
  const uint32_t local = b >> 3;
  const uint32_t m = ((((local >> g) << 3) + (b & 7u)) << g) + (local & ((1u << g) - 1u));
  b = b < L.runs ? m : b;
  const uint32_t tile = fdiv(b, L.dns), t = fdiv(tile, L.d1), u = fdiv(t, L.d2);
  s = (int)(b - tile * L.dns.d);
  const int c0 = (int)(tile - t * L.d1.d), c1 = (int)(t - u * L.d2.d), c2 = (int)u;
  bx = L.order ? c1 : c0;
  j = L.order ? c2 : c1;
  k = L.order ? c0 : c2;
  return (int)tile;
}
// Which variant a row takes: a layer or a wall (within the nodes that the
// differences reach) in x, and in y or z
template <typename T>
__device__ __forceinline__ void row_kind(const LeapArgs<T> &L, int i0, int j, int k, bool &xl, bool &yz) {
  xl = (uint32_t)i0 - L.xs >= L.xn;
  yz = ((uint32_t)j - L.ys >= L.yn) | ((uint32_t)k - L.zs >= L.zn);
}
// The tables of a row, if any (rows outside the box of the entries do not
// ask); n: the step, past the run's last one nothing is injected or recorded
// (tested last, so that the counter and the tables are in flight together)
template <typename T>
__device__ __forceinline__ int2 row_tables(const LeapArgs<T> &L, int b, int bx, int j, int k, int s,
                                           int n, int nt) {
  int2 row = make_int2(-1, -1);
  const uint32_t jj = (uint32_t)j - L.ej, kk = (uint32_t)k - L.ek;
  if ((jj < L.ejn) & (kk < L.ekn)) {
    row.x = L.row_tab[b];
    if (L.src_tab) row.y = L.src_tab[((kk * L.ejn + jj) * L.nbx + bx) * L.ns + s];
  }
  return n < nt ? row : make_int2(-1, -1);
}

// The lane's receiver nodes and injections.  A lane has at most one of each a
// component, so they come as rows of lanes: the loads of all components, then
// those of all their coefficients or sums, are in flight together.  A list a
// lane (an offset, the entries, for each its coefficients, sums and twiddles,
// one after the other) made the waves that hold entries the longest of the
// launch.  Measured, lists -> rows, FP64 gradient of 14x12x10 cells 9.2 -> 5.5
// ms over 800 steps (4.1 without any entry), data of 32x32x32 cells 4.2 -> 2.9
// ms over 512; FP32 gradient of 101x101x61 cells 22.2 -> 21.7 ms.
struct RowEnt {
  int node[6], src[3];
};
template <typename T>
__device__ __forceinline__ RowEnt row_entries(const LeapArgs<T> &L, const StepArgs<T> &A, int2 row, int s,
                                              int tid) {
  RowEnt e;
#pragma unroll
  for (int c = 0; c < 6; ++c) {
    e.node[c] = -1;
    if (row.x >= 0 && (L.rec_mask >> c & 1)) e.node[c] = L.row_rec[(row.x * 6 + c) * 64 + tid];
  }
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    e.src[c] = -1;
    if (L.adj) e.src[c] = e.node[c] >= 0 ? (s * A.nn + e.node[c]) * A.nrow : -1;
    else if (row.y >= 0) e.src[c] = L.row_src[(row.y * 3 + c) * 64 + tid];
  }
  return e;
}

// injected currents of the lane's edges at step n (the sums of inject_all)
template <typename T>
__device__ __forceinline__ void inject_row(const StepArgs<T> &A, const RowEnt &e, int n, double (&inj)[3]) {
  inj[0] = inj[1] = inj[2] = 0.0;
  if (max(e.src[0], max(e.src[1], e.src[2])) < 0) return;
  const double *cf[3];
#pragma unroll
  for (int c = 0; c < 3; ++c) cf[c] = A.coef + max(e.src[c], 0);
#pragma unroll 2
  for (int r = 0; r < A.nrow; ++r) {
    const double f = A.Ftab[(int64_t)r * A.nt + n];
    double k[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) k[c] = cf[c][r];
#pragma unroll
    for (int c = 0; c < 3; ++c) inj[c] = e.src[c] >= 0 ? fma(k[c], f, inj[c]) : inj[c];
  }
}

// receiver transforms of the lane's nodes of the components C .. C + 2, twiddles z
template <int C, typename T>
__device__ __forceinline__ void record_row(const StepArgs<T> &A, const RowEnt &e, int s, const double2 *z,
                                           const double (&v)[3]) {
  if (max(e.node[C], max(e.node[C + 1], e.node[C + 2])) < 0) return;
  double2 *a[3];                         // absent components point at node 0
#pragma unroll
  for (int c = 0; c < 3; ++c) a[c] = A.racc + ((int64_t)s * A.nn + max(e.node[C + c], 0)) * A.nf;
#pragma unroll 2
  for (int kf = 0; kf < A.nf; ++kf) {
    const double2 w = z[kf];
    double2 x[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) x[c] = a[c][kf];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      x[c].x = fma(v[c], w.x, x[c].x);
      x[c].y = fma(v[c], w.y, x[c].y);
      if (e.node[C + c] >= 0) a[c][kf] = x[c];
    }
  }
}

// XL: nodes of the wave may lie in an x layer or at an x wall; YZ: the row
// may lie in a y or z layer or at a wall; ENT: it holds entries (row: its tables).
template <typename T, bool HIST, bool NT, bool XL, bool YZ, bool ENT>
__device__ __forceinline__ void leap_wave(const LeapArgs<T> &L, const StepArgs<T> &A, const Place<T> &P,
                                          int s, int2 row, int i0, int j, int k) {
  // coefficients of the rows j, j - 1, k, k - 1 and of i0 - 1: read before
  // the marker below, so that they are scalar loads
  const bool j_lo = !YZ || j >= 1, k_lo = !YZ || k >= 1, left = !XL || i0 > 0;
  const int jm = j_lo ? j - 1 : j, km = k_lo ? k - 1 : k;
  const AxRow<T> yj = L.axr[L.LA + j], ym = L.axr[L.LA + jm], zk = L.axr[2 * L.LA + k],
                 zm = L.axr[2 * L.LA + km], xl = L.axr[left ? i0 - 1 : 0];
  const int n = P.n;
  // each variant starts with its own marker: loads common to the variants
  // are not hoisted above the branches (that kept the registers of all of
  // them alive at once)
  asm volatile("; %0" ::"n"(XL * 4 + YZ * 2 + ENT));
  const int tid = threadIdx.x, i = i0 + tid;
  if (XL && i >= L.nx) return;            // (a row's last tile is of these variants)
  const int npml = L.npml, W = 2 * npml;
  const uint32_t sz = sizeof(T);
  const bool i_lo = !XL || i >= 1;
  RowEnt ent;
  if constexpr (ENT) ent = row_entries(L, A, row, s, tid);
  // rows below a wall are replaced by the node's own: their values reach no
  // stored result
  const uint32_t dj = L.PXb, ej = j_lo ? 0u - L.PXb : 0u;
  const uint32_t dk = L.PLb, ek = k_lo ? 0u - L.PLb : 0u;
  const uint32_t x0 = (uint32_t)i0 * sz, o = (uint32_t)tid * sz;
  const uint32_t q0 = (uint32_t)k * L.PLb + (uint32_t)j * L.PXb + x0;
  const int64_t so = (int64_t)s * L.F6;
  const __amdgpu_buffer_rsrc_t rI = rsrc_of(P.fi + so), rC = rsrc_of(L.ce), rX = rsrc_of(L.axt);
  const uint32_t x = q0, y = q0 + L.Fb, z = y + L.Fb, u = z + L.Fb, v = u + L.Fb, w = v + L.Fb;
  // ---- loads: E^n at the node and the neighbours, H^{n-1/2}, dt/eps ----
  const T ex0 = bload<T>(rI, o, x), ey0 = bload<T>(rI, o, y), ez0 = bload<T>(rI, o, z);
  const T hx0 = bload<T>(rI, o, u), hy0 = bload<T>(rI, o, v), hz0 = bload<T>(rI, o, w);
  const T ex_jp = bload<T>(rI, o, x + dj), ez_jp = bload<T>(rI, o, z + dj);
  const T ex_kp = bload<T>(rI, o, x + dk), ey_kp = bload<T>(rI, o, y + dk);
  const T ex_jm = bload<T>(rI, o, x + ej), ey_jm = bload<T>(rI, o, y + ej);
  const T ez_jm = bload<T>(rI, o, z + ej), ey_jm_kp = bload<T>(rI, o, y + ej + dk);
  const T hx_jm = bload<T>(rI, o, u + ej), hz_jm = bload<T>(rI, o, w + ej);
  const T ex_km = bload<T>(rI, o, x + ek), ey_km = bload<T>(rI, o, y + ek);
  const T ez_km = bload<T>(rI, o, z + ek), ez_jp_km = bload<T>(rI, o, z + ek + dj);
  const T hx_km = bload<T>(rI, o, u + ek), hy_km = bload<T>(rI, o, v + ek);
  // the nodes beyond the wave's ends, one lane each: E at i + 1 for the last
  // lane, E and H at i - 1 for the first
  const bool right = !XL || i0 + 64 <= L.nx;
  T ey_r = T(0), ez_r = T(0), ey_jm_r = T(0), ez_km_r = T(0);
  if (right && tid == 63) {
    ey_r = bload<T>(rI, o + sz, y);
    ez_r = bload<T>(rI, o + sz, z);
    ey_jm_r = bload<T>(rI, o + sz, y + ej);
    ez_km_r = bload<T>(rI, o + sz, z + ek);
  }
  T ex_l = T(0), ey_l = T(0), ez_l = T(0), ex_l_kp = T(0), ex_l_jp = T(0), hy_l = T(0), hz_l = T(0);
  if (left && tid == 0) {
    ex_l = bload<T>(rI, o, x - sz);
    ey_l = bload<T>(rI, o, y - sz);
    ez_l = bload<T>(rI, o, z - sz);
    ex_l_kp = bload<T>(rI, o, x + dk - sz);
    ex_l_jp = bload<T>(rI, o, x + dj - sz);
    hy_l = bload<T>(rI, o, v - sz);
    hz_l = bload<T>(rI, o, w - sz);
  }
  const T cx = bload<T>(rC, o, x), cy = bload<T>(rC, o, y), cz = bload<T>(rC, o, z);
  const T ih = bload<T>(rX, o, x0 + AX_IH * L.LAb), ihd = bload<T>(rX, o, x0 + AX_IHD * L.LAb);
  // ---- layers: slab indices and memory ----
  bool px = false, pxn = false, pxl = false;
  bool py = false, pym = false, pyn = false, pz = false, pzm = false, pzn = false;
  int lyh = 0, lym = 0, lyn = 0, lzh = 0, lzm = 0, lzn = 0, lxl = 0;
  uint32_t cxh = 0, cxn = 0;
  if constexpr (YZ) {
    py = pml_half(j, L.ny, npml, lyh);
    pym = j_lo && pml_half(jm, L.ny, npml, lym);
    pyn = j_lo && pml_int(j, L.ny, npml, lyn);
    pz = pml_half(k, L.nz, npml, lzh);
    pzm = k_lo && pml_half(km, L.nz, npml, lzm);
    pzn = k_lo && pml_int(k, L.nz, npml, lzn);
  }
  if constexpr (XL) {
    // as pml_half and pml_int, without branches
    px = ((i < npml) | (i >= L.nx - npml));
    pxn = i_lo & ((i < npml) | (i > L.nx - npml));
    cxh = (uint32_t)(i < npml ? i : i - L.nx + W) * sz;
    cxn = (uint32_t)(i < npml ? i : i - L.nx + W - 1) * sz;
    pxl = left && pml_half(i0 - 1, L.nx, npml, lxl);
  }
  T hx_y = T(0), hx_z = T(0), hy_z = T(0), hy_x = T(0), hz_x = T(0), hz_y = T(0);   // H at the node
  T hxj_y = T(0), hxj_z = T(0), hzj_x = T(0), hzj_y = T(0);                         // at j - 1
  T hxk_y = T(0), hxk_z = T(0), hyk_z = T(0), hyk_x = T(0);                         // at k - 1
  T hyl_z = T(0), hyl_x = T(0), hzl_x = T(0), hzl_y = T(0);                         // at i0 - 1
  T ex_y = T(0), ex_z = T(0), ey_z = T(0), ey_x = T(0), ez_x = T(0), ez_y = T(0);   // E (half 0)
  Stretch<T> xh{}, xn{};
  const int64_t sp = (int64_t)s * L.psi_src;
  const uint32_t Wb = (uint32_t)W * sz;
  const uint32_t r0 = (uint32_t)(k * L.NY + j) * Wb;
  const uint32_t oY = L.oYb + x0, oZ = L.oZb + x0;
  const uint32_t rYh = oY + (uint32_t)(k * W + lyh) * L.PXb;
  const uint32_t rYn = oY + 2 * L.sYb + (uint32_t)(k * W + lyn) * L.PXb;
  const uint32_t rZh = oZ + (uint32_t)(lzh * L.NY + j) * L.PXb;
  const uint32_t rZn = oZ + 2 * L.sZb + (uint32_t)(lzn * L.NY + j) * L.PXb;
  if constexpr (XL || YZ) {
    const __amdgpu_buffer_rsrc_t rP = rsrc_of(P.pi + sp), rE = rsrc_of(L.p0 + sp);
    if constexpr (YZ) {
      if (py) {
        hx_y = bload<T>(rP, o, rYh);
        hz_y = bload<T>(rP, o, rYh + L.sYb);
        hxk_y = bload<T>(rP, o, oY + (uint32_t)(km * W + lyh) * L.PXb);
        if (left && tid == 0) hzl_y = bload<T>(rP, o, rYh + L.sYb - sz);
      }
      if (pym) {
        const uint32_t r = oY + (uint32_t)(k * W + lym) * L.PXb;
        hxj_y = bload<T>(rP, o, r);
        hzj_y = bload<T>(rP, o, r + L.sYb);
      }
      if (pz) {
        hx_z = bload<T>(rP, o, rZh);
        hy_z = bload<T>(rP, o, rZh + L.sZb);
        hxj_z = bload<T>(rP, o, oZ + (uint32_t)(lzh * L.NY + jm) * L.PXb);
        if (left && tid == 0) hyl_z = bload<T>(rP, o, rZh + L.sZb - sz);
      }
      if (pzm) {
        const uint32_t r = oZ + (uint32_t)(lzm * L.NY + j) * L.PXb;
        hxk_z = bload<T>(rP, o, r);
        hyk_z = bload<T>(rP, o, r + L.sZb);
      }
      if (pyn) {
        ex_y = bload<T>(rE, o, rYn);
        ez_y = bload<T>(rE, o, rYn + L.sYb);
      }
      if (pzn) {
        ex_z = bload<T>(rE, o, rZn);
        ey_z = bload<T>(rE, o, rZn + L.sZb);
      }
    }
    if constexpr (XL) {
      if (px) {
        hy_x = bload<T>(rP, cxh, r0);
        hz_x = bload<T>(rP, cxh, r0 + L.sXb);
        hyk_x = bload<T>(rP, cxh, (uint32_t)(km * L.NY + j) * Wb);
        hzj_x = bload<T>(rP, cxh, (uint32_t)(k * L.NY + jm) * Wb + L.sXb);
        xh = {bload<T>(rX, o, x0 + AX_BH * L.LAb), bload<T>(rX, o, x0 + AX_AH * L.LAb),
              bload<T>(rX, o, x0 + AX_KH * L.LAb)};
      }
      if (pxl && tid == 0) {
        hyl_x = bload<T>(rP, (uint32_t)lxl * sz, r0);
        hzl_x = bload<T>(rP, (uint32_t)lxl * sz, r0 + L.sXb);
      }
      if (pxn) {
        ey_x = bload<T>(rE, cxn, r0 + 2 * L.sXb);
        ez_x = bload<T>(rE, cxn, r0 + 3 * L.sXb);
        xn = {bload<T>(rX, o, x0 + AX_BN * L.LAb), bload<T>(rX, o, x0 + AX_AN * L.LAb),
              bload<T>(rX, o, x0 + AX_KN * L.LAb)};
      }
    }
  }
  double inj[3];
  // FP64: the injections' loads beside the stencil's.  FP32: after the update,
  // where they need no registers beside the stencil's (141 otherwise, three
  // waves a SIMD for four: 13.0 ms against 12.0 with 4 sources on 101x101x61).
  if constexpr (ENT && sizeof(T) == 8) inject_row(A, ent, n, inj);
  // ---- H^{n+1/2} at the node and, recomputed, at j - 1, k - 1 and i - 1 ----
  const T mc = -L.dtmu;
  const T hj = yj.ih, hjm = ym.ih, hk = zk.ih, hkm = zm.ih;
  const Stretch<T> yh{yj.bh, yj.ah, yj.kh}, yhm{ym.bh, ym.ah, ym.kh},
      yn{yj.bn, yj.an, yj.kn}, zh{zk.bh, zk.ah, zk.kh}, zhm{zm.bh, zm.ah, zm.kh},
      zn{zk.bn, zk.an, zk.kn}, xhl{xl.bh, xl.ah, xl.kh};
  const T ey_ip = lane_above(ey_r, ey0), ez_ip = lane_above(ez_r, ez0);
  const T ey_ip_jm = lane_above(ey_jm_r, ey_jm), ez_ip_km = lane_above(ez_km_r, ez_km);
  const T Hx = curl_update<YZ, YZ>(hx0, mc, ez_jp, ez0, hj, py, hx_y, yh, ey_kp, ey0, hk, pz, hx_z, zh);
  const T Hy = curl_update<YZ, XL>(hy0, mc, ex_kp, ex0, hk, pz, hy_z, zh, ez_ip, ez0, ih, px, hy_x, xh);
  const T Hz = curl_update<XL, YZ>(hz0, mc, ey_ip, ey0, ih, px, hz_x, xh, ex_jp, ex0, hj, py, hz_y, yh);
  const T Hxj = curl_update<YZ, YZ>(hx_jm, mc, ez0, ez_jm, hjm, pym, hxj_y, yhm, ey_jm_kp, ey_jm, hk, pz,
                                    hxj_z, zh);
  const T Hzj = curl_update<XL, YZ>(hz_jm, mc, ey_ip_jm, ey_jm, ih, px, hzj_x, xh, ex0, ex_jm, hjm, pym,
                                    hzj_y, yhm);
  const T Hxk = curl_update<YZ, YZ>(hx_km, mc, ez_jp_km, ez_km, hj, py, hxk_y, yh, ey0, ey_km, hkm, pzm,
                                    hxk_z, zhm);
  const T Hyk = curl_update<YZ, XL>(hy_km, mc, ex0, ex_km, hkm, pzm, hyk_z, zhm, ez_ip_km, ez_km, ih, px,
                                    hyk_x, xh);
  // H at i - 1: the lane below holds it; the first lane recomputes it
  const T Hy_l = curl_update<YZ, XL>(hy_l, mc, ex_l_kp, ex_l, hk, pz, hyl_z, zh, ez0, ez_l, xl.ih, pxl,
                                     hyl_x, xhl);
  const T Hz_l = curl_update<XL, YZ>(hz_l, mc, ey0, ey_l, xl.ih, pxl, hzl_x, xhl, ex_l_jp, ex_l, hj, py,
                                     hzl_y, yh);
  const T Hyi = lane_below(Hy_l, Hy), Hzi = lane_below(Hz_l, Hz);
  // ---- E^{n+1} ----
  T e1x = curl_update<YZ, YZ>(ex0, cx, Hz, Hzj, yj.ihd, pyn, ex_y, yn, Hy, Hyk, zk.ihd, pzn, ex_z, zn);
  T e1y = curl_update<YZ, XL>(ey0, cy, Hx, Hxk, zk.ihd, pzn, ey_z, zn, Hz, Hzi, ihd, pxn, ey_x, xn);
  T e1z = curl_update<XL, YZ>(ez0, cz, Hy, Hyi, ihd, pxn, ez_x, xn, Hx, Hxj, yj.ihd, pyn, ez_y, yn);
  if constexpr (ENT) {
    if constexpr (sizeof(T) == 4) inject_row(A, ent, n, inj);
    e1x -= (T)((double)cx * inj[0]);
    e1y -= (T)((double)cy * inj[1]);
    e1z -= (T)((double)cz * inj[2]);
  }
  // edges on the low x wall keep their value (zero)
  if constexpr (XL) {
    e1y = i_lo ? e1y : ey0;
    e1z = i_lo ? e1z : ez0;
  }
  if constexpr (ENT) {                   // before the stores: the sums' loads would wait for them
    const double e1[3] = {(double)e1x, (double)e1y, (double)e1z}, h1[3] = {(double)Hx, (double)Hy, (double)Hz};
    record_row<0>(A, ent, s, A.zE + (int64_t)n * A.nf, e1);
    if (L.rec_mask >> 3) record_row<3>(A, ent, s, A.zH + (int64_t)n * A.nf, h1);
  }
  // ---- stores ----
  const bool row_x = j_lo && k_lo, row_y = k_lo, row_z = j_lo;
  const __amdgpu_buffer_rsrc_t rO = rsrc_of(P.fo + so);
  bstore<NT>(Hx, rO, o, u);
  bstore<NT>(Hy, rO, o, v);
  bstore<NT>(Hz, rO, o, w);
  if (row_x) bstore<NT>(e1x, rO, o, x);
  if (row_y) bstore<NT>(e1y, rO, o, y);
  if (row_z) bstore<NT>(e1z, rO, o, z);
  if (HIST && n < A.nt) {
    const __amdgpu_buffer_rsrc_t rH = rsrc_of(L.hist + (int64_t)s * L.hist_src);
    if (row_x) bstore<NT>(e1x, rH, o, x);
    if (row_y) bstore<NT>(e1y, rH, o, y);
    if (row_z) bstore<NT>(e1z, rH, o, z);
  }
  if constexpr (XL || YZ) {
    const __amdgpu_buffer_rsrc_t rQ = rsrc_of(P.po + sp), rE = rsrc_of(L.p0 + sp);
    if constexpr (YZ) {
      // memory outside a component's lattice reaches no result
      if (py) {
        bstore<false>(hx_y, rQ, o, rYh);
        bstore<false>(hz_y, rQ, o, rYh + L.sYb);
      }
      if (pz) {
        bstore<false>(hx_z, rQ, o, rZh);
        bstore<false>(hy_z, rQ, o, rZh + L.sZb);
      }
      if (pyn) {
        if (row_x) bstore<false>(ex_y, rE, o, rYn);
        if (row_z) bstore<false>(ez_y, rE, o, rYn + L.sYb);
      }
      if (pzn) {
        if (row_x) bstore<false>(ex_z, rE, o, rZn);
        if (row_y) bstore<false>(ey_z, rE, o, rZn + L.sZb);
      }
    }
    if constexpr (XL) {
      if (px) {
        bstore<false>(hy_x, rQ, cxh, r0);
        bstore<false>(hz_x, rQ, cxh, r0 + L.sXb);
      }
      if (pxn) {
        if (row_y) bstore<false>(ey_x, rE, cxn, r0 + 2 * L.sXb);
        if (row_z) bstore<false>(ez_x, rE, cxn, r0 + 3 * L.sXb);
      }
    }
  }
}

template <typename T, bool HIST, bool NT>
__global__ void __launch_bounds__(64) k_leap(LeapArgs<T> L, StepArgs<T> A) {
  const Place<T> P = place_of(L);
  __builtin_amdgcn_sched_barrier(0);      // see place_of
  int bx, j, k, s;
  const int b = row_of(L, bx, j, k, s);
  const int i0 = bx * 64;
  bool xl, yz;
  row_kind(L, i0, j, k, xl, yz);
  const int2 row = row_tables(L, b, bx, j, k, s, P.n, A.nt);
  if (max(row.x, row.y) >= 0)
    leap_wave<T, HIST, NT, true, true, true>(L, A, P, s, row, i0, j, k);
  else if (xl) {
    if (yz) leap_wave<T, HIST, NT, true, true, false>(L, A, P, s, row, i0, j, k);
    else leap_wave<T, HIST, NT, true, false, false>(L, A, P, s, row, i0, j, k);
  } else {
    if (yz) leap_wave<T, HIST, NT, false, true, false>(L, A, P, s, row, i0, j, k);
    else leap_wave<T, HIST, NT, false, false, false>(L, A, P, s, row, i0, j, k);
  }
  // last: a store before them would turn the uniform loads into vector ones
  if (blockIdx.x == 0 && threadIdx.x == 0) L.step_w[0] = P.n;
}

// ---------------------------------------------------------------------------
// Fourth-order differences (Section 2: the paper's engine is high order on
// the stretched grid).  The pair (9/8, -1/24) over the four nearest samples
// along the axis, in the index coordinate; AX_IH / AX_IHD then hold the
// inverse metric lengths (the same pair applied to the coordinates).
// Samples beyond a wall are images: tangential E (zero on the wall) odd, H
// even.  One element per thread; the raw differences go through the same
// per-node CPML and update arithmetic as order 2 (a difference (D - 0)
// scaled by the table is D scaled by it exactly).
// ---------------------------------------------------------------------------
template <typename T>
__device__ __forceinline__ T e_img(const T *f, int64_t base, int64_t st, int m, int n) {
  if (m < 0) return -f[base - (int64_t)m * st];
  if (m > n) return -f[base + (int64_t)(2 * n - m) * st];
  return f[base + (int64_t)m * st];
}
template <typename T>
__device__ __forceinline__ T h_img(const T *f, int64_t base, int64_t st, int m, int n) {
  m = m < 0 ? -1 - m : (m > n - 1 ? 2 * n - 1 - m : m);
  return f[base + (int64_t)m * st];
}
// E -> H at half node r (0 .. n-1) of E on the nodes 0 .. n
template <typename T>
__device__ __forceinline__ T d4_eh(const T *f, int64_t base, int64_t st, int r, int n) {
  const T a = e_img(f, base, st, r - 1, n), b = f[base + (int64_t)r * st];
  const T c = f[base + (int64_t)(r + 1) * st], d = e_img(f, base, st, r + 2, n);
  return fma(T(-1.0 / 24.0), d - a, T(9.0 / 8.0) * (c - b));
}
// H -> E at node i (1 .. n-1) of H on the half nodes 0 .. n-1
template <typename T>
__device__ __forceinline__ T d4_he(const T *f, int64_t base, int64_t st, int i, int n) {
  const T a = h_img(f, base, st, i - 2, n), b = f[base + (int64_t)(i - 1) * st];
  const T c = f[base + (int64_t)i * st], d = h_img(f, base, st, i + 1, n);
  return fma(T(-1.0 / 24.0), d - a, T(9.0 / 8.0) * (c - b));
}

template <typename T, bool INJ>
__global__ void __launch_bounds__(256) k_update_h4(StepArgs<T> A) {
  int bx, by, bz, s;
  const int b = tile_of(A, bx, by, bz, s);
  const int n = step_of(A, false);
  const int par = n & 1;                 // this step reads half par
  const int i = bx * blockDim.x + threadIdx.x;
  const int j = by * blockDim.y + threadIdx.y;
  const int k = bz;
  if (i > A.nx || j > A.ny || k > A.nz) return;
  const Half<T> I = half_of(A, par, s), O = half_of(A, par ^ 1, s);
  const int PX = A.PX, NY = A.NY, npml = A.npml, W = 2 * npml;
  const int64_t plane = A.plane;
  const int64_t sX = A.sX, sY = A.sY, sZ = A.sZ;
  const bool i_in = i < A.nx, j_in = j < A.ny, k_in = k < A.nz;
  int lx = 0, ly = 0, lz = 0;
  const bool py = npml > 0 && pml_half(j, A.ny, npml, ly);
  const bool pz = npml > 0 && pml_half(k, A.nz, npml, lz);
  const bool px = npml > 0 && i_in && pml_half(i, A.nx, npml, lx);
  const int64_t q = (int64_t)k * plane + (int64_t)j * PX + i;
  const int64_t iX = ((int64_t)k * NY + j) * W + lx;
  const int64_t iY = ((int64_t)k * W + ly) * PX + i;
  const int64_t iZ = ((int64_t)lz * NY + j) * PX + i;
  const T zero = T(0);
  // magnetic adjoint sources of this node (adjoint runs), else the stored H
  int lo = 0, hi = 0;
  if constexpr (INJ) entry_slice(A, b, n, lo, hi);
  Vec<T, 1> hxo = vec1(zero), hyo = vec1(zero), hzo = vec1(zero);
  if (INJ && lo < hi) {
    hxo = vec1(I.hx[q]);
    hyo = vec1(I.hy[q]);
    hzo = vec1(I.hz[q]);
    inject_h<T, 1>(A, lo, hi, s, n, hxo, hyo, hzo);
  }
  if (j_in && k_in) {                    // H_x = H_x - dt/mu (dEz/dy - dEy/dz)
    const T D1 = d4_eh(I.ez, (int64_t)k * plane + i, (int64_t)PX, j, A.ny);
    const T D2 = d4_eh(I.ey, (int64_t)j * PX + i, plane, k, A.nz);
    T psy = py ? I.psY[0 * sY + iY] : zero, psz = pz ? I.psZ[0 * sZ + iZ] : zero;
    O.hx[q] = hx_node(A, j, k, lo < hi ? hxo.v[0] : I.hx[q], zero, D1, zero, D2, py, psy, pz, psz);
    if (py) O.psY[0 * sY + iY] = psy;
    if (pz) O.psZ[0 * sZ + iZ] = psz;
  }
  if (i_in && k_in) {                    // H_y: dEx/dz - dEz/dx
    const T D1 = d4_eh(I.ex, (int64_t)j * PX + i, plane, k, A.nz);
    const T D2 = d4_eh(I.ez, (int64_t)k * plane + (int64_t)j * PX, (int64_t)1, i, A.nx);
    T psz = pz ? I.psZ[1 * sZ + iZ] : zero, psx = px ? I.psX[0 * sX + iX] : zero;
    O.hy[q] = hy_node(A, i, k, lo < hi ? hyo.v[0] : I.hy[q], zero, D1, zero, D2, pz, psz, px, psx);
    if (pz) O.psZ[1 * sZ + iZ] = psz;
    if (px) O.psX[0 * sX + iX] = psx;
  }
  if (i_in && j_in) {                    // H_z: dEy/dx - dEx/dy
    const T D1 = d4_eh(I.ey, (int64_t)k * plane + (int64_t)j * PX, (int64_t)1, i, A.nx);
    const T D2 = d4_eh(I.ex, (int64_t)k * plane + i, (int64_t)PX, j, A.ny);
    T psx = px ? I.psX[1 * sX + iX] : zero, psy = py ? I.psY[1 * sY + iY] : zero;
    O.hz[q] = hz_node(A, i, j, lo < hi ? hzo.v[0] : I.hz[q], zero, D1, zero, D2, px, psx, py, psy);
    if (px) O.psX[1 * sX + iX] = psx;
    if (py) O.psY[1 * sY + iY] = psy;
  }
}

template <typename T, bool HIST>
__global__ void __launch_bounds__(256) k_update_e4(StepArgs<T> A) {
  int bx, by, bz, s;
  const int b = tile_of(A, bx, by, bz, s);
  const int n = step_of(A, true);        // this launch completes step n
  const int i = bx * blockDim.x + threadIdx.x;
  const int j = by * blockDim.y + threadIdx.y;
  const int k = bz;
  if (i > A.nx || j > A.ny || k > A.nz) return;
  int lo, hi;
  entry_slice(A, b, n, lo, hi);
  const int par = n & 1;
  const Half<T> I = half_of(A, par, s), O = half_of(A, par ^ 1, s), P = half_of(A, 0, s);
  const int PX = A.PX, NY = A.NY, npml = A.npml, W = 2 * npml;
  const int64_t plane = A.plane;
  const int64_t sX = A.sX, sY = A.sY, sZ = A.sZ;
  const bool i_int = i >= 1 && i < A.nx, j_int = j >= 1 && j < A.ny, k_int = k >= 1 && k < A.nz;
  const bool okx = i < A.nx && j_int && k_int;
  const bool oky = i_int && j < A.ny && k_int;
  const bool okz = i_int && j_int && k < A.nz;
  int lx = 0, ly = 0, lz = 0;
  const bool py = npml > 0 && pml_int(j, A.ny, npml, ly);
  const bool pz = npml > 0 && pml_int(k, A.nz, npml, lz);
  const bool px = npml > 0 && i_int && pml_int(i, A.nx, npml, lx);
  const int64_t q = (int64_t)k * plane + (int64_t)j * PX + i;
  const int64_t iX = ((int64_t)k * NY + j) * W + lx;
  const int64_t iY = ((int64_t)k * W + ly) * PX + i;
  const int64_t iZ = ((int64_t)lz * NY + j) * PX + i;
  const T zero = T(0);
  const Vec<T, 1> e0x = vec1(I.ex[q]), e0y = vec1(I.ey[q]), e0z = vec1(I.ez[q]);
  Vec<T, 1> e1x = e0x, e1y = e0y, e1z = e0z;
  double inj[3];
  if (lo < hi) inject_all<T, 1>(A, lo, hi, s, n, inj);
  if (okx) {                             // E_x: dHz/dy - dHy/dz
    const T D1 = d4_he(O.hz, (int64_t)k * plane + i, (int64_t)PX, j, A.ny);
    const T D2 = d4_he(O.hy, (int64_t)j * PX + i, plane, k, A.nz);
    T psy = py ? P.psY[2 * sY + iY] : zero, psz = pz ? P.psZ[2 * sZ + iZ] : zero;
    const T c = A.ce[q];
    T v = ex_node(A, j, k, e0x.v[0], c, D1, zero, D2, zero, py, psy, pz, psz);
    if (lo < hi) v -= (T)((double)c * inj[0]);
    e1x.v[0] = v;
    if (py) P.psY[2 * sY + iY] = psy;
    if (pz) P.psZ[2 * sZ + iZ] = psz;
  }
  if (oky) {                             // E_y: dHx/dz - dHz/dx
    const T D1 = d4_he(O.hx, (int64_t)j * PX + i, plane, k, A.nz);
    const T D2 = d4_he(O.hz, (int64_t)k * plane + (int64_t)j * PX, (int64_t)1, i, A.nx);
    T psz = pz ? P.psZ[3 * sZ + iZ] : zero, psx = px ? P.psX[2 * sX + iX] : zero;
    const T c = A.ce[A.F + q];
    T v = ey_node(A, i, k, e0y.v[0], c, D1, zero, D2, zero, pz, psz, px, psx);
    if (lo < hi) v -= (T)((double)c * inj[1]);
    e1y.v[0] = v;
    if (pz) P.psZ[3 * sZ + iZ] = psz;
    if (px) P.psX[2 * sX + iX] = psx;
  }
  if (okz) {                             // E_z: dHy/dx - dHx/dy
    const T D1 = d4_he(O.hy, (int64_t)k * plane + (int64_t)j * PX, (int64_t)1, i, A.nx);
    const T D2 = d4_he(O.hx, (int64_t)k * plane + i, (int64_t)PX, j, A.ny);
    T psx = px ? P.psX[3 * sX + iX] : zero, psy = py ? P.psY[3 * sY + iY] : zero;
    const T c = A.ce[2 * A.F + q];
    T v = ez_node(A, i, j, e0z.v[0], c, D1, zero, D2, zero, px, psx, py, psy);
    if (lo < hi) v -= (T)((double)c * inj[2]);
    e1z.v[0] = v;
    if (px) P.psX[3 * sX + iX] = psx;
    if (py) P.psY[3 * sY + iY] = psy;
  }
  if (okx) O.ex[q] = e1x.v[0];
  if (oky) O.ey[q] = e1y.v[0];
  if (okz) O.ez[q] = e1z.v[0];
  if (lo < hi) {
    const Vec<T, 1> e1[3] = {e1x, e1y, e1z};
    const Vec<T, 1> hh[3] = {vec1(O.hx[q]), vec1(O.hy[q]), vec1(O.hz[q])};
    const unsigned ok[3] = {okx ? 1u : 0u, oky ? 1u : 0u, okz ? 1u : 0u};
    record_all<T, 1>(A, lo, hi, s, n, e1, ok, hh);
  }
  if constexpr (HIST) {
    const Vec<T, 1> e1[3] = {e1x, e1y, e1z};
    const unsigned ok[3] = {okx ? 1u : 0u, oky ? 1u : 0u, okz ? 1u : 0u};
    hist_store<T, 1>(A, s, q, e1, ok, n);
  }
}

// The same two updates as rows of waves (schedule 0 with 32-bit byte offsets
// and no magnetic node on a high wall, as k_leap): one wave a block, 64 nodes
// of one row, so that j and k, their coefficients, layer tests, images and
// the byte offsets of the 21 rows that the differences read are scalar, each
// load one scalar addition and one instruction.  The general kernels above
// spend most of their time issuing per-lane index arithmetic and branches.
// XL: nodes of the wave may lie in an x layer or within two nodes of an x
// wall; YZ: the row may lie so in y or z; ENT: it may hold entries.
// Rows of the high walls are not computed: H there stays zero.
// Measured (one MI355X, 101x101x61 FP32, the kernels alone), general -> rows: H
// update 13.1 -> 9.4 us, E update 18.4 -> 12.6 us (11.1 without the history
// sample; its 37 MB take 5 us at the rate of a large copy).
template <typename T>
__device__ __forceinline__ T d4(T a, T b, T c, T d) {
  return fma(T(-1.0 / 24.0), d - a, T(9.0 / 8.0) * (c - b));
}

template <typename T, bool XL, bool YZ, bool ENT>
__device__ __forceinline__ void h4_wave(const LeapArgs<T> &L, const StepArgs<T> &A, const Place<T> &P,
                                        int s, int b, int i0, int j, int k) {
  const AxRow<T> yj = L.axr[L.LA + j], zk = L.axr[2 * L.LA + k];   // scalar loads: before the marker
  asm volatile("; h4 %0" ::"n"(XL * 4 + YZ * 2 + ENT));            // see leap_wave
  const int tid = threadIdx.x, i = i0 + tid;
  if (XL && i >= L.nx) return;            // (a row's last tile is of these variants)
  const int npml = L.npml, W = 2 * npml;
  const uint32_t sz = sizeof(T);
  const uint32_t x0 = (uint32_t)i0 * sz, o = (uint32_t)tid * sz, Fb = L.Fb;
  // rows j - 1, j + 2 and k - 1, k + 2: beyond a wall the image, negated
  int ja = j - 1, jd = j + 2, ka = k - 1, kd = k + 2;
  T gja = T(1), gjd = T(1), gka = T(1), gkd = T(1);
  if constexpr (YZ) {
    if (ja < 0) { ja = 1; gja = T(-1); }
    if (jd > L.ny) { jd = L.ny - 1; gjd = T(-1); }
    if (ka < 0) { ka = 1; gka = T(-1); }
    if (kd > L.nz) { kd = L.nz - 1; gkd = T(-1); }
  }
  const uint32_t r = (uint32_t)k * L.PLb + (uint32_t)j * L.PXb;      // row, x = 0
  const uint32_t q = r + x0;
  const uint32_t qja = (uint32_t)k * L.PLb + (uint32_t)ja * L.PXb + x0, qjc = q + L.PXb,
                 qjd = (uint32_t)k * L.PLb + (uint32_t)jd * L.PXb + x0;
  const uint32_t qka = (uint32_t)ka * L.PLb + (uint32_t)j * L.PXb + x0, qkc = q + L.PLb,
                 qkd = (uint32_t)kd * L.PLb + (uint32_t)j * L.PXb + x0;
  const __amdgpu_buffer_rsrc_t rI = rsrc_of(P.fi + (int64_t)s * L.F6), rX = rsrc_of(L.axt);
  const T ex = bload<T>(rI, o, q), ey = bload<T>(rI, o, q + Fb), ez = bload<T>(rI, o, q + 2 * Fb);
  T ex_ja = bload<T>(rI, o, qja), ez_ja = bload<T>(rI, o, qja + 2 * Fb);
  const T ex_jc = bload<T>(rI, o, qjc), ez_jc = bload<T>(rI, o, qjc + 2 * Fb);
  T ex_jd = bload<T>(rI, o, qjd), ez_jd = bload<T>(rI, o, qjd + 2 * Fb);
  T ex_ka = bload<T>(rI, o, qka), ey_ka = bload<T>(rI, o, qka + Fb);
  const T ex_kc = bload<T>(rI, o, qkc), ey_kc = bload<T>(rI, o, qkc + Fb);
  T ex_kd = bload<T>(rI, o, qkd), ey_kd = bload<T>(rI, o, qkd + Fb);
  T ey_ia, ez_ia, ey_id, ez_id;
  const T ey_ic = bload<T>(rI, o, q + Fb + sz), ez_ic = bload<T>(rI, o, q + 2 * Fb + sz);
  bool la = false, ld = false;
  if constexpr (XL) {
    la = i == 0;
    ld = i == L.nx - 1;
    const uint32_t oa = (uint32_t)(la ? 1 : i - 1) * sz, od = (uint32_t)(ld ? i : i + 2) * sz;
    ey_ia = bload<T>(rI, oa, r + Fb);
    ez_ia = bload<T>(rI, oa, r + 2 * Fb);
    ey_id = bload<T>(rI, od, r + Fb);
    ez_id = bload<T>(rI, od, r + 2 * Fb);
  } else {
    ey_ia = bload<T>(rI, o, q + Fb - sz);
    ez_ia = bload<T>(rI, o, q + 2 * Fb - sz);
    ey_id = bload<T>(rI, o, q + Fb + 2 * sz);
    ez_id = bload<T>(rI, o, q + 2 * Fb + 2 * sz);
  }
  T hx = bload<T>(rI, o, q + 3 * Fb), hy = bload<T>(rI, o, q + 4 * Fb), hz = bload<T>(rI, o, q + 5 * Fb);
  const T ih = bload<T>(rX, o, x0 + AX_IH * L.LAb);
  // ---- layers: slab indices and memory ----
  bool px = false, py = false, pz = false;
  int lyh = 0, lzh = 0;
  uint32_t cxh = 0;
  if constexpr (YZ) {
    py = pml_half(j, L.ny, npml, lyh);
    pz = pml_half(k, L.nz, npml, lzh);
  }
  if constexpr (XL) {
    px = (i < npml) | (i >= L.nx - npml);
    cxh = (uint32_t)(i < npml ? i : i - L.nx + W) * sz;
  }
  T hx_y = T(0), hx_z = T(0), hy_z = T(0), hy_x = T(0), hz_x = T(0), hz_y = T(0);
  Stretch<T> xh{};
  const int64_t sp = (int64_t)s * L.psi_src;
  const uint32_t r0 = (uint32_t)(k * L.NY + j) * (uint32_t)W * sz;
  const uint32_t rYh = L.oYb + x0 + (uint32_t)(k * W + lyh) * L.PXb;
  const uint32_t rZh = L.oZb + x0 + (uint32_t)(lzh * L.NY + j) * L.PXb;
  if constexpr (XL || YZ) {
    const __amdgpu_buffer_rsrc_t rP = rsrc_of(P.pi + sp);
    if (YZ && py) {
      hx_y = bload<T>(rP, o, rYh);
      hz_y = bload<T>(rP, o, rYh + L.sYb);
    }
    if (YZ && pz) {
      hx_z = bload<T>(rP, o, rZh);
      hy_z = bload<T>(rP, o, rZh + L.sZb);
    }
    if (XL && px) {
      hy_x = bload<T>(rP, cxh, r0);
      hz_x = bload<T>(rP, cxh, r0 + L.sXb);
      xh = {bload<T>(rX, o, x0 + AX_BH * L.LAb), bload<T>(rX, o, x0 + AX_AH * L.LAb),
            bload<T>(rX, o, x0 + AX_KH * L.LAb)};
    }
  }
  if constexpr (ENT) {
    const int n = P.n;
    int lo, hi;
    entry_slice_at(A, b, n, tid, lo, hi);
    if (lo < hi) {
      Vec<T, 1> vx = vec1(hx), vy = vec1(hy), vz = vec1(hz);
      inject_h<T, 1>(A, lo, hi, s, n, vx, vy, vz);
      hx = vx.v[0];
      hy = vy.v[0];
      hz = vz.v[0];
    }
  }
  if constexpr (YZ) {
    ex_ja *= gja; ez_ja *= gja; ex_jd *= gjd; ez_jd *= gjd;
    ex_ka *= gka; ey_ka *= gka; ex_kd *= gkd; ey_kd *= gkd;
  }
  if constexpr (XL) {
    ey_ia = la ? -ey_ia : ey_ia;
    ez_ia = la ? -ez_ia : ez_ia;
    ey_id = ld ? -ey_id : ey_id;
    ez_id = ld ? -ez_id : ez_id;
  }
  const T mc = -L.dtmu, zero = T(0);
  const Stretch<T> yh{yj.bh, yj.ah, yj.kh}, zh{zk.bh, zk.ah, zk.kh};
  const T Hx = curl_update<YZ, YZ>(hx, mc, d4(ez_ja, ez, ez_jc, ez_jd), zero, yj.ih, py, hx_y, yh,
                                   d4(ey_ka, ey, ey_kc, ey_kd), zero, zk.ih, pz, hx_z, zh);
  const T Hy = curl_update<YZ, XL>(hy, mc, d4(ex_ka, ex, ex_kc, ex_kd), zero, zk.ih, pz, hy_z, zh,
                                   d4(ez_ia, ez, ez_ic, ez_id), zero, ih, px, hy_x, xh);
  const T Hz = curl_update<XL, YZ>(hz, mc, d4(ey_ia, ey, ey_ic, ey_id), zero, ih, px, hz_x, xh,
                                   d4(ex_ja, ex, ex_jc, ex_jd), zero, yj.ih, py, hz_y, yh);
  const __amdgpu_buffer_rsrc_t rO = rsrc_of(P.fo + (int64_t)s * L.F6);
  bstore<false>(Hx, rO, o, q + 3 * Fb);
  bstore<false>(Hy, rO, o, q + 4 * Fb);
  bstore<false>(Hz, rO, o, q + 5 * Fb);
  if constexpr (XL || YZ) {
    const __amdgpu_buffer_rsrc_t rQ = rsrc_of(P.po + sp);
    if (YZ && py) {
      bstore<false>(hx_y, rQ, o, rYh);
      bstore<false>(hz_y, rQ, o, rYh + L.sYb);
    }
    if (YZ && pz) {
      bstore<false>(hx_z, rQ, o, rZh);
      bstore<false>(hy_z, rQ, o, rZh + L.sZb);
    }
    if (XL && px) {
      bstore<false>(hy_x, rQ, cxh, r0);
      bstore<false>(hz_x, rQ, cxh, r0 + L.sXb);
    }
  }
}

template <typename T, bool HIST, bool XL, bool YZ, bool ENT>
__device__ __forceinline__ void e4_wave(const LeapArgs<T> &L, const StepArgs<T> &A, const Place<T> &P,
                                        int s, int2 row, int i0, int j, int k) {
  const AxRow<T> yj = L.axr[L.LA + j], zk = L.axr[2 * L.LA + k];
  const int n = P.n;
  asm volatile("; e4 %0" ::"n"(XL * 4 + YZ * 2 + ENT));
  const int tid = threadIdx.x, i = i0 + tid;
  if (XL && i >= L.nx) return;            // (a row's last tile is of these variants)
  RowEnt ent;
  if constexpr (ENT) ent = row_entries(L, A, row, s, tid);
  const int npml = L.npml, W = 2 * npml;
  const uint32_t sz = sizeof(T);
  const uint32_t x0 = (uint32_t)i0 * sz, o = (uint32_t)tid * sz, Fb = L.Fb;
  // rows j - 2, j - 1, j + 1 and k - 2, k - 1, k + 1: beyond a wall the image
  // (index -1 is 0, index n is n - 1); differences of the rows on a low wall
  // reach no stored result
  int ja = j - 2, jb = j - 1, jd = j + 1, ka = k - 2, kb = k - 1, kd = k + 1;
  if constexpr (YZ) {
    ja = max(ja, 0);
    jb = max(jb, 0);
    jd = min(jd, L.ny - 1);
    ka = max(ka, 0);
    kb = max(kb, 0);
    kd = min(kd, L.nz - 1);
  }
  const uint32_t rk = (uint32_t)k * L.PLb, rj = (uint32_t)j * L.PXb;
  const uint32_t r = rk + rj, q = r + x0;
  const uint32_t qja = rk + (uint32_t)ja * L.PXb + x0, qjb = rk + (uint32_t)jb * L.PXb + x0,
                 qjd = rk + (uint32_t)jd * L.PXb + x0;
  const uint32_t qka = (uint32_t)ka * L.PLb + rj + x0, qkb = (uint32_t)kb * L.PLb + rj + x0,
                 qkd = (uint32_t)kd * L.PLb + rj + x0;
  const int64_t so = (int64_t)s * L.F6;
  const __amdgpu_buffer_rsrc_t rI = rsrc_of(P.fi + so), rO = rsrc_of(P.fo + so), rC = rsrc_of(L.ce),
                               rX = rsrc_of(L.axt);
  const uint32_t fx = 3 * Fb, fy = 4 * Fb, fz = 5 * Fb;
  const T hx = bload<T>(rO, o, q + fx), hy = bload<T>(rO, o, q + fy), hz = bload<T>(rO, o, q + fz);
  const T hx_ja = bload<T>(rO, o, qja + fx), hz_ja = bload<T>(rO, o, qja + fz);
  const T hx_jb = bload<T>(rO, o, qjb + fx), hz_jb = bload<T>(rO, o, qjb + fz);
  const T hx_jd = bload<T>(rO, o, qjd + fx), hz_jd = bload<T>(rO, o, qjd + fz);
  const T hx_ka = bload<T>(rO, o, qka + fx), hy_ka = bload<T>(rO, o, qka + fy);
  const T hx_kb = bload<T>(rO, o, qkb + fx), hy_kb = bload<T>(rO, o, qkb + fy);
  const T hx_kd = bload<T>(rO, o, qkd + fx), hy_kd = bload<T>(rO, o, qkd + fy);
  T hy_ia, hz_ia, hy_ib, hz_ib, hy_id, hz_id;
  if constexpr (XL) {
    const uint32_t oa = (uint32_t)max(i - 2, 0) * sz, ob = (uint32_t)max(i - 1, 0) * sz,
                   od = (uint32_t)min(i + 1, L.nx - 1) * sz;
    hy_ia = bload<T>(rO, oa, r + fy);
    hz_ia = bload<T>(rO, oa, r + fz);
    hy_ib = bload<T>(rO, ob, r + fy);
    hz_ib = bload<T>(rO, ob, r + fz);
    hy_id = bload<T>(rO, od, r + fy);
    hz_id = bload<T>(rO, od, r + fz);
  } else {
    hy_ia = bload<T>(rO, o, q + fy - 2 * sz);
    hz_ia = bload<T>(rO, o, q + fz - 2 * sz);
    hy_ib = bload<T>(rO, o, q + fy - sz);
    hz_ib = bload<T>(rO, o, q + fz - sz);
    hy_id = bload<T>(rO, o, q + fy + sz);
    hz_id = bload<T>(rO, o, q + fz + sz);
  }
  const T ex = bload<T>(rI, o, q), ey = bload<T>(rI, o, q + Fb), ez = bload<T>(rI, o, q + 2 * Fb);
  const T cx = bload<T>(rC, o, q), cy = bload<T>(rC, o, q + Fb), cz = bload<T>(rC, o, q + 2 * Fb);
  const T ihd = bload<T>(rX, o, x0 + AX_IHD * L.LAb);
  // ---- layers ----
  const bool j_lo = !YZ || j >= 1, k_lo = !YZ || k >= 1, i_lo = !XL || i >= 1;
  bool pxn = false, pyn = false, pzn = false;
  int lyn = 0, lzn = 0;
  uint32_t cxn = 0;
  if constexpr (YZ) {
    pyn = j_lo && pml_int(j, L.ny, npml, lyn);
    pzn = k_lo && pml_int(k, L.nz, npml, lzn);
  }
  if constexpr (XL) {
    pxn = i_lo & ((i < npml) | (i > L.nx - npml));
    cxn = (uint32_t)(i < npml ? i : i - L.nx + W - 1) * sz;
  }
  T ex_y = T(0), ex_z = T(0), ey_z = T(0), ey_x = T(0), ez_x = T(0), ez_y = T(0);
  Stretch<T> xn{};
  const __amdgpu_buffer_rsrc_t rE = rsrc_of(L.p0 + (int64_t)s * L.psi_src);
  const uint32_t r0 = (uint32_t)(k * L.NY + j) * (uint32_t)W * sz + 2 * L.sXb;
  const uint32_t rYn = L.oYb + x0 + 2 * L.sYb + (uint32_t)(k * W + lyn) * L.PXb;
  const uint32_t rZn = L.oZb + x0 + 2 * L.sZb + (uint32_t)(lzn * L.NY + j) * L.PXb;
  if (YZ && pyn) {
    ex_y = bload<T>(rE, o, rYn);
    ez_y = bload<T>(rE, o, rYn + L.sYb);
  }
  if (YZ && pzn) {
    ex_z = bload<T>(rE, o, rZn);
    ey_z = bload<T>(rE, o, rZn + L.sZb);
  }
  if (XL && pxn) {
    ey_x = bload<T>(rE, cxn, r0);
    ez_x = bload<T>(rE, cxn, r0 + L.sXb);
    xn = {bload<T>(rX, o, x0 + AX_BN * L.LAb), bload<T>(rX, o, x0 + AX_AN * L.LAb),
          bload<T>(rX, o, x0 + AX_KN * L.LAb)};
  }
  double inj[3];
  if constexpr (ENT) inject_row(A, ent, n, inj);
  const T zero = T(0);
  const Stretch<T> yn{yj.bn, yj.an, yj.kn}, zn{zk.bn, zk.an, zk.kn};
  T e1x = curl_update<YZ, YZ>(ex, cx, d4(hz_ja, hz_jb, hz, hz_jd), zero, yj.ihd, pyn, ex_y, yn,
                              d4(hy_ka, hy_kb, hy, hy_kd), zero, zk.ihd, pzn, ex_z, zn);
  T e1y = curl_update<YZ, XL>(ey, cy, d4(hx_ka, hx_kb, hx, hx_kd), zero, zk.ihd, pzn, ey_z, zn,
                              d4(hz_ia, hz_ib, hz, hz_id), zero, ihd, pxn, ey_x, xn);
  T e1z = curl_update<XL, YZ>(ez, cz, d4(hy_ia, hy_ib, hy, hy_id), zero, ihd, pxn, ez_x, xn,
                              d4(hx_ja, hx_jb, hx, hx_jd), zero, yj.ihd, pyn, ez_y, yn);
  if constexpr (ENT) {
    e1x -= (T)((double)cx * inj[0]);
    e1y -= (T)((double)cy * inj[1]);
    e1z -= (T)((double)cz * inj[2]);
  }
  if constexpr (XL) {                    // edges on the low x wall keep their value (zero)
    e1y = i_lo ? e1y : ey;
    e1z = i_lo ? e1z : ez;
  }
  if constexpr (ENT) {                   // before the stores: the sums' loads would wait for them
    const double e1[3] = {(double)e1x, (double)e1y, (double)e1z}, h1[3] = {(double)hx, (double)hy, (double)hz};
    record_row<0>(A, ent, s, A.zE + (int64_t)n * A.nf, e1);
    if (L.rec_mask >> 3) record_row<3>(A, ent, s, A.zH + (int64_t)n * A.nf, h1);
  }
  const bool row_x = j_lo && k_lo, row_y = k_lo, row_z = j_lo;
  if (row_x) bstore<false>(e1x, rO, o, q);
  if (row_y) bstore<false>(e1y, rO, o, q + Fb);
  if (row_z) bstore<false>(e1z, rO, o, q + 2 * Fb);
  if (HIST && n < A.nt) {
    const __amdgpu_buffer_rsrc_t rH = rsrc_of(L.hist + (int64_t)s * L.hist_src);
    if (row_x) bstore<false>(e1x, rH, o, q);
    if (row_y) bstore<false>(e1y, rH, o, q + Fb);
    if (row_z) bstore<false>(e1z, rH, o, q + 2 * Fb);
  }
  if (YZ && pyn) {
    if (row_x) bstore<false>(ex_y, rE, o, rYn);
    if (row_z) bstore<false>(ez_y, rE, o, rYn + L.sYb);
  }
  if (YZ && pzn) {
    if (row_x) bstore<false>(ex_z, rE, o, rZn);
    if (row_y) bstore<false>(ey_z, rE, o, rZn + L.sZb);
  }
  if (XL && pxn) {
    if (row_y) bstore<false>(ey_x, rE, cxn, r0);
    if (row_z) bstore<false>(ez_x, rE, cxn, r0 + L.sXb);
  }
}

template <typename T, bool INJ>
__global__ void __launch_bounds__(64) k_rows_h4(LeapArgs<T> L, StepArgs<T> A) {
  const Place<T> P = place_of(L);
  __builtin_amdgcn_sched_barrier(0);      // see place_of
  int bx, j, k, s;
  const int b = row_of(L, bx, j, k, s);
  const int i0 = bx * 64;
  bool xl, yz;
  row_kind(L, i0, j, k, xl, yz);
  if (INJ && A.tile_tab[b] >= 0)
    h4_wave<T, true, true, true>(L, A, P, s, b, i0, j, k);
  else if (xl) {
    if (yz) h4_wave<T, true, true, false>(L, A, P, s, b, i0, j, k);
    else h4_wave<T, true, false, false>(L, A, P, s, b, i0, j, k);
  } else {
    if (yz) h4_wave<T, false, true, false>(L, A, P, s, b, i0, j, k);
    else h4_wave<T, false, false, false>(L, A, P, s, b, i0, j, k);
  }
}

template <typename T, bool HIST>
__global__ void __launch_bounds__(64) k_rows_e4(LeapArgs<T> L, StepArgs<T> A) {
  const Place<T> P = place_of(L);
  __builtin_amdgcn_sched_barrier(0);      // see place_of
  int bx, j, k, s;
  const int b = row_of(L, bx, j, k, s);
  const int i0 = bx * 64;
  bool xl, yz;
  row_kind(L, i0, j, k, xl, yz);
  const int2 row = row_tables(L, b, bx, j, k, s, P.n, A.nt);
  if (max(row.x, row.y) >= 0)
    e4_wave<T, HIST, true, true, true>(L, A, P, s, row, i0, j, k);
  else if (xl) {
    if (yz) e4_wave<T, HIST, true, true, false>(L, A, P, s, row, i0, j, k);
    else e4_wave<T, HIST, true, false, false>(L, A, P, s, row, i0, j, k);
  } else {
    if (yz) e4_wave<T, HIST, false, true, false>(L, A, P, s, row, i0, j, k);
    else e4_wave<T, HIST, false, false, false>(L, A, P, s, row, i0, j, k);
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) L.step_w[0] = P.n;
}

// ---------------------------------------------------------------------------
// Fused step (one launch per leapfrog step).  A block of bx x by threads
// owns the columns (i, j) = (x0 + tx, y0 + ty) of a tile and the planes
// k in [z0, z1) of a chunk.  For each plane:
//   1. E^n of plane k goes to LDS on the tile plus a one-node halo: the
//      high-side column and row feed the forward differences of H on the
//      tile, the low-side column and row those of H at x0 - 1 and y0 - 1;
//   2. H^{n+1/2} of plane k is computed on the tile and recomputed on the
//      low-side halo column and row (the operands and operations of the
//      owning block, so the same bits), and staged in LDS for the backward
//      differences of the E update;
//   3. E^{n+1} of plane k, with the z differences taken against H of the
//      plane below (carried in registers) and E of the plane above (loaded
//      ahead, carried into the next plane).
// A chunk with z0 > 0 first recomputes H at plane z0 - 1 of its tile.
// Threads on the tile edges load the halo; threads outside the grid take
// part in the barriers with zeros.  Two barriers per plane: after the E
// staging (H reads E) and after the H staging (E reads H); the next plane's
// E staging follows the second barrier, its H staging the next first one.
// ---------------------------------------------------------------------------
template <typename T>
__device__ __forceinline__ T ld(const StepArgs<T> &A, const T *f, int i, int j, int k) {
  return (i >= 0 && i <= A.nx && j >= 0 && j <= A.ny && k >= 0 && k <= A.nz)
             ? f[((int64_t)k * A.NY + j) * A.PX + i]
             : T(0);
}

template <typename T, bool HIST>
__global__ void __launch_bounds__(256) k_step(StepArgs<T> A) {
  extern __shared__ double lds_raw[];
  const int BX = blockDim.x, BY = blockDim.y;
  const int WE = BX + 2, WH = BX + 1;
  const int SE = WE * (BY + 2), SH = WH * (BY + 1);
  T *sEx = reinterpret_cast<T *>(lds_raw), *sEy = sEx + SE, *sEz = sEy + SE;
  T *sHx = sEz + SE, *sHy = sHx + SH, *sHz = sHy + SH;
  int tbx, tby, tbz, s;
  const int b = tile_of(A, tbx, tby, tbz, s);
  const int tx = threadIdx.x, ty = threadIdx.y;
  const int x0 = tbx * BX, y0 = tby * BY;
  const int i = x0 + tx, j = y0 + ty;
  const int z0 = tbz * A.kz, z1 = min(z0 + A.kz, A.nz);
  const int n = step_of(A, true), par = n & 1;   // this launch completes step n
  int lo, hi;
  entry_slice(A, b, n, lo, hi);
  const int npml = A.npml, W = 2 * npml, PX = A.PX, NY = A.NY;
  const int64_t sX = A.sX, sY = A.sY, sZ = A.sZ;
  // column geometry of the own node and of the low-side halo nodes
  const bool act = i <= A.nx && j <= A.ny;
  const bool i_in = i < A.nx, j_in = j < A.ny;
  const bool i_int = i >= 1 && i < A.nx, j_int = j >= 1 && j < A.ny;
  int lxh = 0, lyh = 0, lxn = 0, lyn = 0;
  const bool pxh = npml > 0 && i_in && pml_half(i, A.nx, npml, lxh);
  const bool pyh = npml > 0 && j_in && pml_half(j, A.ny, npml, lyh);
  const bool pxn = npml > 0 && i_int && pml_int(i, A.nx, npml, lxn);
  const bool pyn = npml > 0 && j_int && pml_int(j, A.ny, npml, lyn);
  const int ia = x0 - 1, jb = y0 - 1;                     // halo column / row
  const bool haloA = tx == 0 && ia >= 0 && j <= A.ny;      // node (ia, j): H_y, H_z
  const bool haloB = ty == 0 && jb >= 0 && i <= A.nx;      // node (i, jb): H_z, H_x
  int lxa = 0, lyb = 0;
  const bool pxa = npml > 0 && haloA && pml_half(ia, A.nx, npml, lxa);
  const bool pyb = npml > 0 && haloB && pml_half(jb, A.ny, npml, lyb);
  const int own = (ty + 1) * WE + tx + 1, ownH = (ty + 1) * WH + tx + 1;

  {
    const Half<T> I = half_of(A, par, s), O = half_of(A, par ^ 1, s), P = half_of(A, 0, s);
    const int kbeg = z0 > 0 ? z0 - 1 : 0;
    T ex = ld(A, I.ex, i, j, kbeg), ey = ld(A, I.ey, i, j, kbeg), ez = ld(A, I.ez, i, j, kbeg);
    T exa = tx == 0 ? ld(A, I.ex, ia, j, kbeg) : T(0);   // E_x at (ia, j, k)
    T eyb = ty == 0 ? ld(A, I.ey, i, jb, kbeg) : T(0);   // E_y at (i, jb, k)
    T hxm = T(0), hym = T(0);                             // H^{n+1/2} at (i, j, k-1)
    for (int k = kbeg; k < z1; ++k) {
      const bool pre = k < z0;
      const int sub = k - z0;
      const int64_t q = ((int64_t)k * NY + j) * PX + i;   // dereferenced only when act
      int lzh = 0, lzn = 0;
      const bool pzh = npml > 0 && pml_half(k, A.nz, npml, lzh);
      const bool pzn = npml > 0 && k >= 1 && pml_int(k, A.nz, npml, lzn);
      // ---- loads: E^n of plane k+1 (own), H^{n-1/2} of plane k, E halo ----
      const T ex1 = ld(A, I.ex, i, j, k + 1), ey1 = ld(A, I.ey, i, j, k + 1);
      const T ez1 = ld(A, I.ez, i, j, k + 1);
      const T hx = ld(A, I.hx, i, j, k), hy = ld(A, I.hy, i, j, k);
      const T hz = pre ? T(0) : ld(A, I.hz, i, j, k);
      T gEyR = 0, gEzR = 0, gExT = 0, gEzT = 0, gEyA = 0, gEzA = 0, gExAT = 0;
      T gExB = 0, gEzB = 0, gEyBR = 0, exa1 = 0, eyb1 = 0;
      if (tx == BX - 1) {                                  // high-side column x0 + BX
        gEyR = ld(A, I.ey, x0 + BX, j, k);
        gEzR = ld(A, I.ez, x0 + BX, j, k);
      }
      if (ty == BY - 1) {                                  // high-side row y0 + BY
        gExT = ld(A, I.ex, i, y0 + BY, k);
        gEzT = ld(A, I.ez, i, y0 + BY, k);
      }
      if (tx == 0) {                                       // low-side column ia
        gEyA = ld(A, I.ey, ia, j, k);
        gEzA = ld(A, I.ez, ia, j, k);
        exa1 = ld(A, I.ex, ia, j, k + 1);
        if (ty == BY - 1) gExAT = ld(A, I.ex, ia, y0 + BY, k);
      }
      if (ty == 0) {                                       // low-side row jb
        gExB = ld(A, I.ex, i, jb, k);
        gEzB = ld(A, I.ez, i, jb, k);
        eyb1 = ld(A, I.ey, i, jb, k + 1);
        if (tx == BX - 1) gEyBR = ld(A, I.ey, x0 + BX, jb, k);
      }
      // CPML memory of H at the own node (read half par)
      const int64_t iYh = ((int64_t)k * W + lyh) * PX + i, iZh = ((int64_t)lzh * NY + j) * PX + i;
      const int64_t iXh = ((int64_t)k * NY + j) * W + lxh;
      T ps_hx_y = act && pyh ? I.psY[0 * sY + iYh] : T(0);
      T ps_hz_y = act && pyh && !pre ? I.psY[1 * sY + iYh] : T(0);
      T ps_hx_z = act && pzh && j_in ? I.psZ[0 * sZ + iZh] : T(0);
      T ps_hy_z = act && pzh ? I.psZ[1 * sZ + iZh] : T(0);
      T ps_hy_x = act && pxh ? I.psX[0 * sX + iXh] : T(0);
      T ps_hz_x = act && pxh && j_in && !pre ? I.psX[1 * sX + iXh] : T(0);
      // halo H^{n-1/2} and its CPML memory
      T hyA = 0, hzA = 0, pa_hy_z = 0, pa_hy_x = 0, pa_hz_x = 0, pa_hz_y = 0;
      if (!pre && haloA) {
        hyA = ld(A, I.hy, ia, j, k);
        if (pzh) pa_hy_z = I.psZ[1 * sZ + ((int64_t)lzh * NY + j) * PX + ia];
        if (pxa) pa_hy_x = I.psX[0 * sX + ((int64_t)k * NY + j) * W + lxa];
        if (j_in) {
          hzA = ld(A, I.hz, ia, j, k);
          if (pxa) pa_hz_x = I.psX[1 * sX + ((int64_t)k * NY + j) * W + lxa];
          if (pyh) pa_hz_y = I.psY[1 * sY + ((int64_t)k * W + lyh) * PX + ia];
        }
      }
      T hxB = 0, hzB = 0, pb_hx_y = 0, pb_hx_z = 0, pb_hz_x = 0, pb_hz_y = 0;
      if (!pre && haloB) {
        hxB = ld(A, I.hx, i, jb, k);
        if (pyb) pb_hx_y = I.psY[0 * sY + ((int64_t)k * W + lyb) * PX + i];
        if (pzh) pb_hx_z = I.psZ[0 * sZ + ((int64_t)lzh * NY + jb) * PX + i];
        if (i_in) {
          hzB = ld(A, I.hz, i, jb, k);
          if (pxh) pb_hz_x = I.psX[1 * sX + ((int64_t)k * NY + jb) * W + lxh];
          if (pyb) pb_hz_y = I.psY[1 * sY + ((int64_t)k * W + lyb) * PX + i];
        }
      }
      // ---- stage E^n of plane k ----
      sEx[own] = ex;
      sEy[own] = ey;
      sEz[own] = ez;
      if (tx == BX - 1) {
        sEy[(ty + 1) * WE + BX + 1] = gEyR;
        sEz[(ty + 1) * WE + BX + 1] = gEzR;
      }
      if (ty == BY - 1) {
        sEx[(BY + 1) * WE + tx + 1] = gExT;
        sEz[(BY + 1) * WE + tx + 1] = gEzT;
      }
      if (tx == 0) {
        sEx[(ty + 1) * WE] = exa;
        sEy[(ty + 1) * WE] = gEyA;
        sEz[(ty + 1) * WE] = gEzA;
        if (ty == BY - 1) sEx[(BY + 1) * WE] = gExAT;
      }
      if (ty == 0) {
        sEx[tx + 1] = gExB;
        sEy[tx + 1] = eyb;
        sEz[tx + 1] = gEzB;
        if (tx == BX - 1) sEy[BX + 1] = gEyBR;
      }
      __syncthreads();
      // ---- H^{n+1/2} of plane k ----
      T hxn = hx, hyn = hy, hzn = hz;
      if (act) {
        if (j_in)
          hxn = hx_node(A, j, k, hx, ez, sEz[own + WE], ey, ey1, pyh, ps_hx_y, pzh, ps_hx_z);
        if (i_in)
          hyn = hy_node(A, i, k, hy, ex, ex1, ez, sEz[own + 1], pzh, ps_hy_z, pxh, ps_hy_x);
        if (i_in && j_in && !pre)
          hzn = hz_node(A, i, j, hz, ey, sEy[own + 1], ex, sEx[own + WE], pxh, ps_hz_x, pyh,
                        ps_hz_y);
      }
      if (!pre) {
        T hyAn = 0, hzAn = 0, hxBn = 0, hzBn = 0;
        if (haloA) {
          const int a0 = (ty + 1) * WE;
          hyAn = hy_node(A, ia, k, hyA, exa, exa1, sEz[a0], sEz[a0 + 1], pzh, pa_hy_z, pxa, pa_hy_x);
          if (j_in)
            hzAn = hz_node(A, ia, j, hzA, sEy[a0], sEy[a0 + 1], exa, sEx[a0 + WE], pxa, pa_hz_x, pyh,
                           pa_hz_y);
        }
        if (haloB) {
          if (i_in)
            hzBn = hz_node(A, i, jb, hzB, sEy[tx + 1], sEy[tx + 2], sEx[tx + 1], sEx[WE + tx + 1],
                           pxh, pb_hz_x, pyb, pb_hz_y);
          hxBn = hx_node(A, jb, k, hxB, sEz[tx + 1], sEz[WE + tx + 1], eyb, eyb1, pyb, pb_hx_y,
                         pzh, pb_hx_z);
        }
        sHx[ownH] = hxn;
        sHy[ownH] = hyn;
        sHz[ownH] = hzn;
        if (tx == 0) {
          sHy[(ty + 1) * WH] = hyAn;
          sHz[(ty + 1) * WH] = hzAn;
        }
        if (ty == 0) {
          sHx[tx + 1] = hxBn;
          sHz[tx + 1] = hzBn;
        }
        if (act) {
          O.hx[q] = hxn;
          O.hy[q] = hyn;
          O.hz[q] = hzn;
          if (pyh) {
            O.psY[0 * sY + iYh] = ps_hx_y;
            O.psY[1 * sY + iYh] = ps_hz_y;
          }
          if (pzh) {
            if (j_in) O.psZ[0 * sZ + iZh] = ps_hx_z;
            O.psZ[1 * sZ + iZh] = ps_hy_z;
          }
          if (pxh) {
            O.psX[0 * sX + iXh] = ps_hy_x;
            if (j_in) O.psX[1 * sX + iXh] = ps_hz_x;
          }
        }
      }
      __syncthreads();
      // ---- E^{n+1} of plane k ----
      if (!pre && act) {
        const bool k_int = k >= 1;
        const bool okx = i_in && j_int && k_int;
        const bool oky = i_int && j_in && k_int;
        const bool okz = i_int && j_int;
        const T cx = okx ? A.ce[q] : T(0), cy = oky ? A.ce[A.F + q] : T(0);
        const T cz = okz ? A.ce[2 * A.F + q] : T(0);
        const int64_t iYn = ((int64_t)k * W + lyn) * PX + i, iZn = ((int64_t)lzn * NY + j) * PX + i;
        const int64_t iXn = ((int64_t)k * NY + j) * W + lxn;
        T dummy = T(0);
        T exn = ex, eyn = ey, ezn = ez;
        if (okx) {
          T &psy = pyn ? P.psY[2 * sY + iYn] : dummy;
          T &psz = pzn ? P.psZ[2 * sZ + iZn] : dummy;
          exn = ex_node(A, j, k, ex, cx, hzn, sHz[ownH - WH], hyn, hym, pyn, psy, pzn, psz);
          if (lo < hi) exn -= (T)((double)cx * inject_value(A, lo, hi, s, 0, sub, n));
          O.ex[q] = exn;
        }
        if (oky) {
          T &psz = pzn ? P.psZ[3 * sZ + iZn] : dummy;
          T &psx = pxn ? P.psX[2 * sX + iXn] : dummy;
          eyn = ey_node(A, i, k, ey, cy, hxn, hxm, hzn, sHz[ownH - 1], pzn, psz, pxn, psx);
          if (lo < hi) eyn -= (T)((double)cy * inject_value(A, lo, hi, s, 1, sub, n));
          O.ey[q] = eyn;
        }
        if (okz) {
          T &psx = pxn ? P.psX[3 * sX + iXn] : dummy;
          T &psy = pyn ? P.psY[3 * sY + iYn] : dummy;
          ezn = ez_node(A, i, j, ez, cz, hyn, sHy[ownH - 1], hxn, sHx[ownH - WH], pxn, psx, pyn,
                        psy);
          if (lo < hi) ezn -= (T)((double)cz * inject_value(A, lo, hi, s, 2, sub, n));
          O.ez[q] = ezn;
        }
        if (lo < hi) {
          if (okx) record(A, lo, hi, s, 0, sub, n, (double)exn);
          if (oky) record(A, lo, hi, s, 1, sub, n, (double)eyn);
          if (okz) record(A, lo, hi, s, 2, sub, n, (double)ezn);
        }
        if constexpr (HIST) {
          const Vec<T, 1> e1[3] = {vec1(exn), vec1(eyn), vec1(ezn)};
          const unsigned ok[3] = {okx ? 1u : 0u, oky ? 1u : 0u, okz ? 1u : 0u};
          hist_store<T, 1>(A, s, q, e1, ok, n);
        }
      }
      // ---- carry to the next plane ----
      hxm = hxn;
      hym = hyn;
      ex = ex1;
      ey = ey1;
      ez = ez1;
      exa = exa1;
      eyb = eyb1;
    }
  }
}

// Block transform (eq. dft, KB samples per read-modify-write of the
// accumulators).  Launched after the E update whose sample m_last closes a
// block (FLUSH false: m_last % KB == 0, the KB samples m_last-KB+1 ..
// m_last), or to add an incomplete last block (FLUSH true: the m_last % KB
// newest samples; the caller then moves *flushed to m_last).  Samples at or
// before *flushed were added by an earlier flush and samples past the run
// are zero.  The block's samples are in history slots 0 .. cnt-2 and, the
// newest, in the field half m_last % 2.
//   forward  acc_k += sum_t E^{first+t} z_k^{first+t}, the sum over the
//            block formed in FP64 first, then added in the accumulator's
//            precision
//   adjoint  gedge += sum_k Re(S_k V_k), S_k = sum_t u^t Q_k^t: the
//            gradient product of eq. gradsigmaij over the block, V the
//            forward transform (Q on the host)
// One thread per node of the padded layout (grid x), source (grid y) and
// E component (grid z); threads off the component's lattice return.  A
// thread holds only its KB samples; the block's twiddles (all frequencies)
// are staged once in LDS and read as broadcasts.
// The block's twiddles (all frequencies) in LDS: s_tw[kf * KB + t] for the
// samples first, first + D, ..., first + (cnt-1) D (zero beyond cnt), each
// times the weight D of a decimated sample (a power of two: exact); the
// caller synchronises.
template <typename T, bool ADJ, int KB>
__device__ __forceinline__ void stage_twiddles(const StepArgs<T> &A, double2 *s_tw, int first,
                                               int cnt, int dl, int tid, int nthr) {
  const double2 *tw = ADJ ? A.Q : A.zE;
  const int nf = A.nf;
  const double wgt = (double)(1 << dl);
  for (int e = tid; e < nf * KB; e += nthr) {
    const int kf = e / KB, t = e - kf * KB;
    double2 v = make_double2(0.0, 0.0);
    if (t < cnt) {
      v = tw[(int64_t)(first - 1 + (t << dl)) * nf + kf];
      v.x *= wgt;
      v.y *= wgt;
    }
    s_tw[e] = v;
  }
}

// The block transform of node q (padded layout), component c of source s:
// the cnt samples first, first + D, ... (D = 2^A.dl), twiddles staged in
// s_tw.  A closing block reads its newest sample from the field half
// m_last % 2 (m_last: the step just completed); a flush reads every sample
// from the history.
template <typename T, int ACC, bool ADJ, int KB, bool FLUSH>
__device__ __forceinline__ void transform_node(const StepArgs<T> &A, int64_t q, int s, int c,
                                               int first, int cnt, int m_last,
                                               const double2 *s_tw) {
  const int nf = A.nf, nt = A.nt, dl = A.dl;
  const uint32_t qq = (uint32_t)q;
  const uint32_t k = fdiv(qq, A.dplane), rem = qq - k * (uint32_t)A.plane;
  const uint32_t j = fdiv(rem, A.dpx), i = rem - j * (uint32_t)A.PX;
  const bool iin = i < (uint32_t)A.nx, jin = j < (uint32_t)A.ny, kin = k < (uint32_t)A.nz;
  const bool ii = i >= 1 && iin, ji = j >= 1 && jin, ki = k >= 1 && kin;
  const bool on = c == 0 ? iin && ji && ki : (c == 1 ? ii && jin && ki : ii && ji && kin);
  const int fl = A.flushed[0];
  const int64_t F = A.F, F3 = 3 * A.F;
  const int64_t base = ((int64_t)s * nf * 3 + c) * F + q;    // + kf * 3 F
  using Ac = Acc<ACC>;
  // The run's first block with nothing flushed before it: the forward
  // accumulators are written, not updated (a run does not clear the volume
  // buffer first), and nodes off the component's lattice receive zeros.
  // Adding to zero gives the same bits, so this is the cleared buffer's
  // result without the clearing pass or the first block's loads.
  const bool fresh = !ADJ && first == (1 << dl) && fl == 0;
  if (!on) {
    if (fresh)
      for (int kf = 0; kf < nf; ++kf) Ac::store(A.vol, base + (int64_t)kf * F3, Ac::zero());
    return;
  }
  const T *h = A.hist + (int64_t)s * A.hist_src + (int64_t)c * F + q;
  const T *f = A.fields + ((m_last & 1) ? A.fbuf : 0) + (int64_t)s * A.F6 + (int64_t)c * F + q;
  // the samples in the field type; those outside (fl, nt] are zeroed with a
  // select (the condition is the same for every thread)
  T val[KB];
#pragma unroll
  for (int t = 0; t < KB; ++t) {
    T v = T(0);
    if (t < cnt - 1 || (FLUSH && t < cnt)) v = h[(int64_t)t * F3];
    else if (t == cnt - 1) v = f[0];
    const int idx = first + (t << dl);
    val[t] = idx <= fl || idx > nt ? T(0) : v;
  }
  if constexpr (!ADJ) {
    // two frequencies at a time: both accumulators are loaded before either
    // store (loads and stores share one in-order completion counter)
    auto block_sum = [&](int kf) {
      const double2 *z = s_tw + kf * KB;
      double2 sum = make_double2(0.0, 0.0);
#pragma unroll
      for (int t = 0; t < KB; ++t) {
        if (FLUSH && t >= cnt) break;
        const double2 zt = z[t];
        sum.x = fma((double)val[t], zt.x, sum.x);
        sum.y = fma((double)val[t], zt.y, sum.y);
      }
      return sum;
    };
    int kf = 0;
    for (; kf + 1 < nf; kf += 2) {
      const typename Ac::S a0 = fresh ? Ac::zero() : Ac::load(A.vol, base + (int64_t)kf * F3);
      const typename Ac::S a1 =
          fresh ? Ac::zero() : Ac::load(A.vol, base + (int64_t)(kf + 1) * F3);
      const double2 s0 = block_sum(kf), s1 = block_sum(kf + 1);
      Ac::store(A.vol, base + (int64_t)kf * F3, Ac::add(a0, s0));
      Ac::store(A.vol, base + (int64_t)(kf + 1) * F3, Ac::add(a1, s1));
    }
    if (kf < nf) {
      const typename Ac::S a = fresh ? Ac::zero() : Ac::load(A.vol, base + (int64_t)kf * F3);
      Ac::store(A.vol, base + (int64_t)kf * F3, Ac::add(a, block_sum(kf)));
    }
  } else {
    // per frequency Re(S V), S formed from the samples and Q while the
    // forward transform V is loading; two frequencies at a time, both
    // V loads issued before either sum (the same order of additions into
    // re as one frequency at a time)
    double re = 0.0;
    auto block_s = [&](int kf, double &sx, double &sy) {
      const double2 *Qt = s_tw + kf * KB;
      sx = 0.0;
      sy = 0.0;
#pragma unroll
      for (int t = 0; t < KB; ++t) {
        if (FLUSH && t >= cnt) break;
        const double2 qt = Qt[t];
        sx = fma((double)val[t], qt.x, sx);
        sy = fma((double)val[t], qt.y, sy);
      }
    };
    int kf = 0;
    for (; kf + 1 < nf; kf += 2) {
      const double2 v0 = Ac::value(Ac::load(A.vol, base + (int64_t)kf * F3));
      const double2 v1 = Ac::value(Ac::load(A.vol, base + (int64_t)(kf + 1) * F3));
      double sx0, sy0, sx1, sy1;
      block_s(kf, sx0, sy0);
      block_s(kf + 1, sx1, sy1);
      re = fma(sx0, v0.x, fma(-sy0, v0.y, re));
      re = fma(sx1, v1.x, fma(-sy1, v1.y, re));
    }
    if (kf < nf) {
      const double2 v = Ac::value(Ac::load(A.vol, base + (int64_t)kf * F3));
      double sx, sy;
      block_s(kf, sx, sy);
      re = fma(sx, v.x, fma(-sy, v.y, re));
    }
    double *g = A.gedge + ((int64_t)s * 3 + c) * F + q;
    *g = *g + re;
  }
}

template <typename T, int ACC, bool ADJ, int KB, bool FLUSH>
__global__ void __launch_bounds__(256) k_transform(StepArgs<T> A) {
  extern __shared__ double2 s_tw[];          // [nf][KB] twiddles of the block
  const int m_last = A.step[0] + 1;          // the step just completed
  const int j_last = m_last >> A.dl;         // the newest (decimated) sample
  const int r_end = j_last & (KB - 1);
  const int cnt = FLUSH ? r_end : KB;
  // uniform: the whole grid returns
  if (FLUSH ? cnt == 0 : r_end != 0 || (m_last & ((1 << A.dl) - 1)) != 0) return;
  const int first = (j_last - cnt + 1) << A.dl;
  stage_twiddles<T, ADJ, KB>(A, s_tw, first, cnt, A.dl, threadIdx.x, blockDim.x);
  __syncthreads();
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= A.F) return;
  transform_node<T, ACC, ADJ, KB, FLUSH>(A, q, blockIdx.y, blockIdx.z, first, cnt, m_last, s_tw);
}

// ---------------------------------------------------------------------------
// Persistent schedule (FWD_OPT_SCHEDULE = 2): one cooperative launch runs
// nsteps leapfrog steps.  Every block loops over the tiles of a phase -- the
// H update, the E update, and the block transform after a step that closes
// a transform block -- with a grid-wide barrier between phases.  The tiles,
// their entry lists and the per-node arithmetic are those of the two-kernel
// schedule, so the results are the same bit for bit.
//
// The barrier: the first thread of each block reads the generation, then
// arrives on the counter (device-scope atomics; a release fence first, so
// the block's stores, complete at workgroup scope after __syncthreads, reach
// the other XCDs); the last block to arrive resets the counter and moves the
// generation on (release); the others poll the generation with acquire loads
// and pass when it moves.  The launch is cooperative (the runtime refuses a
// grid whose blocks cannot all be resident at once) and sized from the
// occupancy of the instantiation launched.  A wait longer than `limit`
// wall-clock ticks, or the abort flag set by another block, ends the wait:
// the block sets the flag and returns, so every block exits and the host
// reports the abandoned run.
// ---------------------------------------------------------------------------
struct Bar {
  unsigned *count, *gen;
  int *abort;
  uint64_t limit;     // wall-clock ticks a block may wait at one barrier
  int naps;           // s_sleep(1) pauses (64 cycles each) between two polls
};

__device__ __forceinline__ bool grid_sync(const Bar &B) {
  __shared__ int s_ok;
  __syncthreads();
  if (threadIdx.x == 0 && threadIdx.y == 0) {
    int ok = 1;
    const unsigned g = __hip_atomic_load(B.gen, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    const unsigned a = __hip_atomic_fetch_add(B.count, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
    if (a == gridDim.x - 1) {
      __hip_atomic_store(B.count, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(B.gen, g + 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
    } else {
      const uint64_t t0 = wall_clock64();
      while (__hip_atomic_load(B.gen, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT) == g) {
        if (__hip_atomic_load(B.abort, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0 ||
            wall_clock64() - t0 > B.limit) {
          __hip_atomic_store(B.abort, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          ok = 0;
          break;
        }
        for (int z = 0; z < B.naps; ++z) __builtin_amdgcn_s_sleep(1);
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    s_ok = ok;
  }
  __syncthreads();
  return s_ok != 0;
}

// A: E-update arguments (tiles of the E update, its entry lists); Ah: the
// H update's (its tiling and, with INJ, its table of magnetic sources).  The
// host equalised the step counters; block 0 leaves both at the last step.
template <typename T, bool HIST, int ACC, bool ADJ, int KB, bool INJ>
__global__ void __launch_bounds__(256) k_persist(StepArgs<T> A, StepArgs<T> Ah, int nsteps, Bar B) {
  extern __shared__ double2 s_tw[];          // twiddles of a closing block
  const int tid = threadIdx.y * blockDim.x + threadIdx.x, nthr = blockDim.x * blockDim.y;
  const int n0 = A.step[0] + 1;
  const uint32_t nq = (uint32_t)((A.F + nthr - 1) / nthr);   // transform tiles per source, component
  for (int t = 0; t < nsteps; ++t) {
    const int n = n0 + t, par = n & 1;
    for (uint32_t vb = blockIdx.x; vb < (uint32_t)Ah.nblocks; vb += gridDim.x) {
      int bx, by, bz, s;
      const int b = tile_of_b(Ah, vb, bx, by, bz, s);
      const int i0 = bx * blockDim.x + threadIdx.x, j = by * blockDim.y + threadIdx.y, k = bz;
      if (i0 > A.nx || j > A.ny || k > A.nz) continue;
      int lo = 0, hi = 0;
      if constexpr (INJ) entry_slice(Ah, b, n, lo, hi);
      if (interior_tile(Ah, bx, by, k, blockDim.x))
        h_vec<T, 1, INJ, true>(Ah, half_of(Ah, par, s), half_of(Ah, par ^ 1, s), i0, j,
                               __builtin_amdgcn_readfirstlane(k), lo, hi, s, n);
      else
        h_vec<T, 1, INJ, false>(Ah, half_of(Ah, par, s), half_of(Ah, par ^ 1, s), i0, j, k, lo, hi,
                                s, n);
    }
    if (!grid_sync(B)) return;
    for (uint32_t vb = blockIdx.x; vb < (uint32_t)A.nblocks; vb += gridDim.x) {
      int bx, by, bz, s;
      const int b = tile_of_b(A, vb, bx, by, bz, s);
      const int i0 = bx * blockDim.x + threadIdx.x, j = by * blockDim.y + threadIdx.y, k = bz;
      if (i0 > A.nx || j > A.ny || k > A.nz) continue;
      if (interior_tile(A, bx, by, k, blockDim.x))
        e_vec<T, HIST, 1, true>(A, s, b, half_of(A, par, s), half_of(A, par ^ 1, s),
                                half_of(A, 0, s), i0, j, __builtin_amdgcn_readfirstlane(k), n);
      else
        e_vec<T, HIST, 1, false>(A, s, b, half_of(A, par, s), half_of(A, par ^ 1, s),
                                 half_of(A, 0, s), i0, j, k, n);
    }
    if (!grid_sync(B)) return;
    if (HIST && (n + 1) % KB == 0) {
      const int m = n + 1;
      stage_twiddles<T, ADJ, KB>(A, s_tw, m - KB + 1, KB, 0, tid, nthr);
      __syncthreads();
      const uint32_t total = nq * (uint32_t)A.ns * 3u;
      for (uint32_t vb = blockIdx.x; vb < total; vb += gridDim.x) {
        const uint32_t qc = vb % nq, rest = vb / nq;
        const int s = (int)(rest % (uint32_t)A.ns), c = (int)(rest / (uint32_t)A.ns);
        const int64_t q = (int64_t)qc * nthr + tid;
        if (q < A.F) transform_node<T, ACC, ADJ, KB, false>(A, q, s, c, m - KB + 1, KB, m, s_tw);
      }
      if (!grid_sync(B)) return;
    }
  }
  if (blockIdx.x == 0 && tid == 0) {          // counters r = 0 and 1 of the workspace
    const_cast<int *>(A.step)[0] = n0 + nsteps - 1;
    A.step_w[0] = n0 + nsteps - 1;
  }
}

__global__ void k_set_flushed(int *flushed, const int *step) {
  if (threadIdx.x == 0 && blockIdx.x == 0) flushed[0] = step[0] + 1;
}

// both step counters to the last completed step (the larger of the two)
__global__ void k_equalize(int *cnt) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    const int v = max(cnt[0], cnt[1]);
    cnt[0] = v;
    cnt[1] = v;
  }
}

// ---------------------------------------------------------------------------
// Time-domain adjoint (the Appendix formulation applied to the stepped
// system).  Reverse step n is the transpose of forward step n, undone in
// reverse order: first its E update, then its H update.  The adjoint state
// holds a multiplier per field value and per CPML memory variable (same
// layout as one half of the forward state).  For one stretched derivative
// d = D kinv + psi', psi' = b psi + a D (inside a layer; else d = D), the
// transpose maps the multiplier ad of d and apsi' of psi' to
//     aD = ad kinv + a (ad + apsi'),   apsi = b (ad + apsi').
//   k_td_e     per H node: the deferred update of its own H multipliers,
//              then aH += D_h^T aD over the E edges that difference it
//              (ad = +-ce aE on those edges);
//   k_td_h     per E edge: the update of its own E multipliers and the
//              gradient product aE (E^{n+1} - E^n) / (sigma_e dV_e), then
//              aE += D_e^T aD over the H nodes that difference it
//              (ad = -+dt/mu aH);
//   k_td_sens  the sensitivity of the misfit to E^m at the receiver nodes.
// Every kernel reads its neighbours' multipliers and writes only its own;
// each node's own update is deferred to the next kernel, so no neighbour
// reads a value that has already moved on.
// ---------------------------------------------------------------------------

// aD / hd of derivative d (1 or 2) of the E update of component c at edge
// (i, j, k); 0 where the edge is not updated.  Derivatives: E_x d1 = d/dy,
// d2 = d/dz; E_y d1 = d/dz, d2 = d/dx; E_z d1 = d/dx, d2 = d/dy.
template <typename T>
__device__ __forceinline__ T td_ad_e(const StepArgs<T> &A, const Half<T> &Ad, int c, int d, int i,
                                     int j, int k) {
  bool ok;
  if (c == 0) ok = i >= 0 && i < A.nx && j >= 1 && j < A.ny && k >= 1 && k < A.nz;
  else if (c == 1) ok = i >= 1 && i < A.nx && j >= 0 && j < A.ny && k >= 1 && k < A.nz;
  else ok = i >= 1 && i < A.nx && j >= 1 && j < A.ny && k >= 0 && k < A.nz;
  if (!ok) return T(0);
  const int W = 2 * A.npml;
  const int64_t sX = A.sX, sY = A.sY, sZ = A.sZ;
  const int64_t q = ((int64_t)k * A.NY + j) * A.PX + i;
  const T ae = (c == 0 ? Ad.ex : c == 1 ? Ad.ey : Ad.ez)[q];
  const T add = (d == 1 ? T(1) : T(-1)) * A.ce[c * A.F + q] * ae;
  // axis of the derivative (0 x, 1 y, 2 z) and its node index
  const int ax = c == 0 ? (d == 1 ? 1 : 2) : c == 1 ? (d == 1 ? 2 : 0) : (d == 1 ? 0 : 1);
  const int idx = ax == 0 ? i : ax == 1 ? j : k;
  const int nax = ax == 0 ? A.nx : ax == 1 ? A.ny : A.nz;
  int l = 0;
  T aD = add;
  if (A.npml > 0 && pml_int(idx, nax, A.npml, l)) {
    const T *ps;
    if (ax == 1) ps = Ad.psY + (c == 0 ? 2 : 3) * sY + ((int64_t)k * W + l) * A.PX + i;
    else if (ax == 2) ps = Ad.psZ + (c == 0 ? 2 : 3) * sZ + ((int64_t)l * A.NY + j) * A.PX + i;
    else ps = Ad.psX + (c == 1 ? 2 : 3) * sX + ((int64_t)k * A.NY + j) * W + l;
    aD = add * axv(A, ax, AX_KN, idx) + axv(A, ax, AX_AN, idx) * (add + *ps);
  }
  return aD * axv(A, ax, AX_IHD, idx);
}

// aD / h of derivative d of the H update of component c at node (i, j, k);
// 0 where the node does not exist.  H_x d1 = d/dy, d2 = d/dz; H_y d1 = d/dz,
// d2 = d/dx; H_z d1 = d/dx, d2 = d/dy.
template <typename T>
__device__ __forceinline__ T td_ad_h(const StepArgs<T> &A, const Half<T> &Ad, int c, int d, int i,
                                     int j, int k) {
  bool ok;
  if (c == 0) ok = i >= 0 && i <= A.nx && j >= 0 && j < A.ny && k >= 0 && k < A.nz;
  else if (c == 1) ok = i >= 0 && i < A.nx && j >= 0 && j <= A.ny && k >= 0 && k < A.nz;
  else ok = i >= 0 && i < A.nx && j >= 0 && j < A.ny && k >= 0 && k <= A.nz;
  if (!ok) return T(0);
  const int W = 2 * A.npml;
  const int64_t sX = A.sX, sY = A.sY, sZ = A.sZ;
  const int64_t q = ((int64_t)k * A.NY + j) * A.PX + i;
  const T ah = (c == 0 ? Ad.hx : c == 1 ? Ad.hy : Ad.hz)[q];
  const T add = (d == 1 ? -A.dtmu : A.dtmu) * ah;
  const int ax = c == 0 ? (d == 1 ? 1 : 2) : c == 1 ? (d == 1 ? 2 : 0) : (d == 1 ? 0 : 1);
  const int idx = ax == 0 ? i : ax == 1 ? j : k;
  const int nax = ax == 0 ? A.nx : ax == 1 ? A.ny : A.nz;
  int l = 0;
  T aD = add;
  if (A.npml > 0 && pml_half(idx, nax, A.npml, l)) {
    const T *ps;
    if (ax == 1) ps = Ad.psY + (c == 0 ? 0 : 1) * sY + ((int64_t)k * W + l) * A.PX + i;
    else if (ax == 2) ps = Ad.psZ + (c == 0 ? 0 : 1) * sZ + ((int64_t)l * A.NY + j) * A.PX + i;
    else ps = Ad.psX + (c == 1 ? 0 : 1) * sX + ((int64_t)k * A.NY + j) * W + l;
    aD = add * axv(A, ax, AX_KH, idx) + axv(A, ax, AX_AH, idx) * (add + *ps);
  }
  return aD * axv(A, ax, AX_IH, idx);
}

// Transposed gathers of the fourth-order differences.  An H node at half
// index r along the axis is used by the H -> E differences at nodes r (9/8),
// r+1 (-9/8), r-1 (-1/24 of H[r] = H[(r-1)+1] enters with +c2) and r+2; the
// even images add the node-1 term to r = 0 and the node-(n-1) term to
// r = n-1.  An E node at index m is used by the E -> H differences at half
// nodes m-1, m, m-2 and m+1; the odd images add the half-node-0 term to
// m = 1 and the half-node-(n-1) term to m = n-1.  at(x) is the multiplier
// of the difference at index x (zero where none is updated).
template <typename T, typename F>
__device__ __forceinline__ T gather_h4(F at, int r, int n) {
  const T c1 = T(9.0 / 8.0), c2 = T(-1.0 / 24.0);
  T v = c1 * (at(r) - at(r + 1)) + c2 * (at(r - 1) - at(r + 2));
  if (r == 0) v -= c2 * at(1);
  if (r == n - 1) v += c2 * at(n - 1);
  return v;
}
template <typename T, typename F>
__device__ __forceinline__ T gather_e4(F at, int m, int n) {
  const T c1 = T(9.0 / 8.0), c2 = T(-1.0 / 24.0);
  T v = c1 * (at(m - 1) - at(m)) + c2 * (at(m - 2) - at(m + 1));
  if (m == 1) v += c2 * at(0);
  if (m == n - 1) v -= c2 * at(n - 1);
  return v;
}

template <typename T, int ORD>
__global__ void __launch_bounds__(256) k_td_e(StepArgs<T> A) {
  int bx, by, bz, s;
  tile_of(A, bx, by, bz, s);
  const int i = bx * blockDim.x + threadIdx.x, j = by * blockDim.y + threadIdx.y, k = bz;
  if (i > A.nx || j > A.ny || k > A.nz) return;
  const Half<T> Ad = half_of(A, 0, s);
  const int npml = A.npml, W = 2 * npml;
  const int64_t sX = A.sX, sY = A.sY, sZ = A.sZ;
  const int64_t q = ((int64_t)k * A.NY + j) * A.PX + i;
  const bool hx = j < A.ny && k < A.nz, hy = i < A.nx && k < A.nz, hz = i < A.nx && j < A.ny;
  int lx = 0, ly = 0, lz = 0;
  const bool px = npml > 0 && i < A.nx && pml_half(i, A.nx, npml, lx);
  const bool py = npml > 0 && j < A.ny && pml_half(j, A.ny, npml, ly);
  const bool pz = npml > 0 && k < A.nz && pml_half(k, A.nz, npml, lz);
  const int64_t iX = ((int64_t)k * A.NY + j) * W + lx, iY = ((int64_t)k * W + ly) * A.PX + i,
                iZ = ((int64_t)lz * A.NY + j) * A.PX + i;
  const T dtmu = A.dtmu;
  // deferred update of the own H multipliers (transpose of the previous
  // reverse step's H update: apsi = b (ad + apsi'))
  if (hx) {
    const T a = Ad.hx[q];
    if (py) { T &p = Ad.psY[0 * sY + iY]; p = axv(A, 1, AX_BH, j) * (-dtmu * a + p); }
    if (pz) { T &p = Ad.psZ[0 * sZ + iZ]; p = axv(A, 2, AX_BH, k) * (dtmu * a + p); }
  }
  if (hy) {
    const T a = Ad.hy[q];
    if (pz) { T &p = Ad.psZ[1 * sZ + iZ]; p = axv(A, 2, AX_BH, k) * (-dtmu * a + p); }
    if (px) { T &p = Ad.psX[0 * sX + iX]; p = axv(A, 0, AX_BH, i) * (dtmu * a + p); }
  }
  if (hz) {
    const T a = Ad.hz[q];
    if (px) { T &p = Ad.psX[1 * sX + iX]; p = axv(A, 0, AX_BH, i) * (-dtmu * a + p); }
    if (py) { T &p = Ad.psY[1 * sY + iY]; p = axv(A, 1, AX_BH, j) * (dtmu * a + p); }
  }
  // aH += D_h^T aD: H_z is differenced by E_x d1 at j, j+1 and E_y d2 at
  // i, i+1; H_y by E_x d2 at k, k+1 and E_z d1 at i, i+1; H_x by E_y d1 at
  // k, k+1 and E_z d2 at j, j+1
  if constexpr (ORD == 2) {
    if (hz)
      Ad.hz[q] += td_ad_e(A, Ad, 0, 1, i, j, k) - td_ad_e(A, Ad, 0, 1, i, j + 1, k) +
                  td_ad_e(A, Ad, 1, 2, i, j, k) - td_ad_e(A, Ad, 1, 2, i + 1, j, k);
    if (hy)
      Ad.hy[q] += td_ad_e(A, Ad, 0, 2, i, j, k) - td_ad_e(A, Ad, 0, 2, i, j, k + 1) +
                  td_ad_e(A, Ad, 2, 1, i, j, k) - td_ad_e(A, Ad, 2, 1, i + 1, j, k);
    if (hx)
      Ad.hx[q] += td_ad_e(A, Ad, 1, 1, i, j, k) - td_ad_e(A, Ad, 1, 1, i, j, k + 1) +
                  td_ad_e(A, Ad, 2, 2, i, j, k) - td_ad_e(A, Ad, 2, 2, i, j + 1, k);
  } else {
    auto ax = [&](int c, int d) { return [&A, &Ad, c, d, i, j, k](int m) -> T {
      // the derivative's axis: E_x d1 y, d2 z; E_y d1 z, d2 x; E_z d1 x, d2 y
      const int a = c == 0 ? (d == 1 ? 1 : 2) : c == 1 ? (d == 1 ? 2 : 0) : (d == 1 ? 0 : 1);
      return td_ad_e(A, Ad, c, d, a == 0 ? m : i, a == 1 ? m : j, a == 2 ? m : k);
    }; };
    if (hz) Ad.hz[q] += gather_h4<T>(ax(0, 1), j, A.ny) + gather_h4<T>(ax(1, 2), i, A.nx);
    if (hy) Ad.hy[q] += gather_h4<T>(ax(0, 2), k, A.nz) + gather_h4<T>(ax(2, 1), i, A.nx);
    if (hx) Ad.hx[q] += gather_h4<T>(ax(1, 1), k, A.nz) + gather_h4<T>(ax(2, 2), j, A.ny);
  }
}

// Enew, Eold: E^{n+1} and E^n, [ns][3][F]; tdw: 1/(sigma_e dV_e) [3][F]
template <typename T, int ORD>
__global__ void __launch_bounds__(256) k_td_h(StepArgs<T> A, const T *Enew, const T *Eold,
                                              const double *tdw) {
  int bx, by, bz, s;
  tile_of(A, bx, by, bz, s);
  const int i = bx * blockDim.x + threadIdx.x, j = by * blockDim.y + threadIdx.y, k = bz;
  if (i > A.nx || j > A.ny || k > A.nz) return;
  const Half<T> Ad = half_of(A, 0, s);
  const int npml = A.npml, W = 2 * npml;
  const int64_t F = A.F;
  const int64_t sX = A.sX, sY = A.sY, sZ = A.sZ;
  const int64_t q = ((int64_t)k * A.NY + j) * A.PX + i;
  const bool i_int = i >= 1 && i < A.nx, j_int = j >= 1 && j < A.ny, k_int = k >= 1 && k < A.nz;
  const bool okx = i < A.nx && j_int && k_int, oky = i_int && j < A.ny && k_int,
             okz = i_int && j_int && k < A.nz;
  int lx = 0, ly = 0, lz = 0;
  const bool px = npml > 0 && i_int && pml_int(i, A.nx, npml, lx);
  const bool py = npml > 0 && j_int && pml_int(j, A.ny, npml, ly);
  const bool pz = npml > 0 && k_int && pml_int(k, A.nz, npml, lz);
  const int64_t iX = ((int64_t)k * A.NY + j) * W + lx, iY = ((int64_t)k * W + ly) * A.PX + i,
                iZ = ((int64_t)lz * A.NY + j) * A.PX + i;
  const int64_t e0 = (int64_t)s * 3 * F;
  double *g = A.gedge + e0;
  // own E multipliers: deferred CPML update (ad = +ce aE for d1, -ce aE for
  // d2) and the gradient product
  if (okx) {
    const T a = Ad.ex[q], ca = A.ce[q] * a;
    if (py) { T &p = Ad.psY[2 * sY + iY]; p = axv(A, 1, AX_BN, j) * (ca + p); }
    if (pz) { T &p = Ad.psZ[2 * sZ + iZ]; p = axv(A, 2, AX_BN, k) * (-ca + p); }
    g[q] += (double)a * ((double)Enew[e0 + q] - (double)Eold[e0 + q]) * tdw[q];
  }
  if (oky) {
    const T a = Ad.ey[q], ca = A.ce[F + q] * a;
    if (pz) { T &p = Ad.psZ[3 * sZ + iZ]; p = axv(A, 2, AX_BN, k) * (ca + p); }
    if (px) { T &p = Ad.psX[2 * sX + iX]; p = axv(A, 0, AX_BN, i) * (-ca + p); }
    g[F + q] += (double)a * ((double)Enew[e0 + F + q] - (double)Eold[e0 + F + q]) * tdw[F + q];
  }
  if (okz) {
    const T a = Ad.ez[q], ca = A.ce[2 * F + q] * a;
    if (px) { T &p = Ad.psX[3 * sX + iX]; p = axv(A, 0, AX_BN, i) * (ca + p); }
    if (py) { T &p = Ad.psY[3 * sY + iY]; p = axv(A, 1, AX_BN, j) * (-ca + p); }
    g[2 * F + q] +=
        (double)a * ((double)Enew[e0 + 2 * F + q] - (double)Eold[e0 + 2 * F + q]) * tdw[2 * F + q];
  }
  // aE += D_e^T aD: E_x is differenced by H_y d1 at k-1, k and H_z d2 at
  // j-1, j; E_y by H_x d2 at k-1, k and H_z d1 at i-1, i; E_z by H_x d1 at
  // j-1, j and H_y d2 at i-1, i
  if constexpr (ORD == 2) {
    if (okx)
      Ad.ex[q] += td_ad_h(A, Ad, 1, 1, i, j, k - 1) - td_ad_h(A, Ad, 1, 1, i, j, k) +
                  td_ad_h(A, Ad, 2, 2, i, j - 1, k) - td_ad_h(A, Ad, 2, 2, i, j, k);
    if (oky)
      Ad.ey[q] += td_ad_h(A, Ad, 0, 2, i, j, k - 1) - td_ad_h(A, Ad, 0, 2, i, j, k) +
                  td_ad_h(A, Ad, 2, 1, i - 1, j, k) - td_ad_h(A, Ad, 2, 1, i, j, k);
    if (okz)
      Ad.ez[q] += td_ad_h(A, Ad, 0, 1, i, j - 1, k) - td_ad_h(A, Ad, 0, 1, i, j, k) +
                  td_ad_h(A, Ad, 1, 2, i - 1, j, k) - td_ad_h(A, Ad, 1, 2, i, j, k);
  } else {
    auto ax = [&](int c, int d) { return [&A, &Ad, c, d, i, j, k](int m) -> T {
      // H_x d1 y, d2 z; H_y d1 z, d2 x; H_z d1 x, d2 y
      const int a = c == 0 ? (d == 1 ? 1 : 2) : c == 1 ? (d == 1 ? 2 : 0) : (d == 1 ? 0 : 1);
      return td_ad_h(A, Ad, c, d, a == 0 ? m : i, a == 1 ? m : j, a == 2 ? m : k);
    }; };
    if (okx) Ad.ex[q] += gather_e4<T>(ax(1, 1), k, A.nz) + gather_e4<T>(ax(2, 2), j, A.ny);
    if (oky) Ad.ey[q] += gather_e4<T>(ax(0, 2), k, A.nz) + gather_e4<T>(ax(2, 1), i, A.nx);
    if (okz) Ad.ez[q] += gather_e4<T>(ax(0, 1), j, A.ny) + gather_e4<T>(ax(1, 2), i, A.nx);
  }
}

// The reverse step of order 2 as rows of waves (where k_leap runs the forward
// steps): one wave a block, 64 nodes of one row; rows, coefficients, layer
// tests and offsets are scalar, and the x neighbour's term comes from the lane
// beside (the wave's edge lane computes it).  The receiver tables of the adjoint
// runs add the receivers' sensitivities to the owner's new multiplier, so the
// two launches are the whole reverse step.  XL, YZ, ENT: as k_leap.
// The same operations in the same order as the general kernels.
// Multipliers and memory on the high walls stay zero: their rows are skipped.
// Measured (one MI355X, 101x101x61 FP32), general -> rows: H multipliers 27.3
// -> 11.8 us, E multipliers and product 35.4 -> 20.7 us (its 94 MB, a third of
// them the FP64 sums, take 13 us at the rate of a cached copy), and the two
// sensitivity launches of 4.8 us a step are gone.

// aD / h of one derivative: ad its multiplier, p its memory's
template <bool P, typename T>
__device__ __forceinline__ T td_ad(T ad, T h, bool in, T p, T kinv, T a) {
  T v = ad;
  if constexpr (P) {
    const T d = ad * kinv + a * (ad + p);
    v = in ? d : v;
  }
  return v * h;
}

// -Re sum_k C_k z_k (k_td_sens) of the lane's nodes of the components K ..
// K + 2, added to v
template <int K, typename T>
__device__ __forceinline__ void td_sens_row(const StepArgs<T> &A, const RowEnt &e, const double2 *C,
                                            const double2 *z, int s, T (&v)[3]) {
  if (max(e.node[K], max(e.node[K + 1], e.node[K + 2])) < 0) return;
  const double2 *q[3];
  double g[3] = {0.0, 0.0, 0.0};
#pragma unroll
  for (int c = 0; c < 3; ++c) q[c] = C + ((int64_t)s * A.nn + max(e.node[K + c], 0)) * A.nf;
#pragma unroll 2
  for (int kf = 0; kf < A.nf; ++kf) {
    const double2 w = z[kf];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const double2 u = q[c][kf];
      g[c] -= u.x * w.x - u.y * w.y;
    }
  }
#pragma unroll
  for (int c = 0; c < 3; ++c) v[c] = e.node[K + c] >= 0 ? v[c] + (T)g[c] : v[c];
}

template <typename T, bool XL, bool YZ, bool ENT>
__device__ __forceinline__ void td_e_wave(const LeapArgs<T> &L, const StepArgs<T> &A, int s, int2 row, int i0,
                                          int j, int k, const double2 *C, const double2 *z) {
  const AxRow<T> yj = L.axr[L.LA + j], yp = L.axr[L.LA + j + 1], zk = L.axr[2 * L.LA + k],
                 zp = L.axr[2 * L.LA + k + 1], xr = L.axr[min(i0 + 64, L.nx)];
  asm volatile("; tde %0" ::"n"(XL * 4 + YZ * 2 + ENT));   // see leap_wave
  const int tid = threadIdx.x, i = i0 + tid;
  RowEnt ent;
  if constexpr (ENT) ent = row_entries(L, A, row, s, tid);
  const int npml = L.npml, W = 2 * npml;
  const uint32_t sz = sizeof(T), x0 = (uint32_t)i0 * sz, o = (uint32_t)tid * sz, Fb = L.Fb;
  const uint32_t q = (uint32_t)k * L.PLb + (uint32_t)j * L.PXb + x0, qj = q + L.PXb, qk = q + L.PLb;
  const __amdgpu_buffer_rsrc_t rA = rsrc_of(L.f0 + (int64_t)s * L.F6), rO = rA,
                               rC = rsrc_of(L.ce), rX = rsrc_of(L.axt);
  const T ax = bload<T>(rA, o, q), ay = bload<T>(rA, o, q + Fb), az = bload<T>(rA, o, q + 2 * Fb);
  const T ax_j = bload<T>(rA, o, qj), az_j = bload<T>(rA, o, qj + 2 * Fb);
  const T ax_k = bload<T>(rA, o, qk), ay_k = bload<T>(rA, o, qk + Fb);
  const T cx = bload<T>(rC, o, q), cy = bload<T>(rC, o, q + Fb), cz = bload<T>(rC, o, q + 2 * Fb);
  const T cx_j = bload<T>(rC, o, qj), cz_j = bload<T>(rC, o, qj + 2 * Fb);
  const T cx_k = bload<T>(rC, o, qk), cy_k = bload<T>(rC, o, qk + Fb);
  const T hx = bload<T>(rA, o, q + 3 * Fb), hy = bload<T>(rA, o, q + 4 * Fb), hz = bload<T>(rA, o, q + 5 * Fb);
  const T ihd = bload<T>(rX, o, x0 + AX_IHD * L.LAb);
  // the edge lane's neighbour at i0 + 64 (edges on the high wall contribute nothing)
  const bool right = i0 + 64 < L.nx;
  T ay_r = T(0), az_r = T(0), cy_r = T(0), cz_r = T(0);
  if (right && tid == 63) {
    ay_r = bload<T>(rA, o, q + Fb + sz);
    az_r = bload<T>(rA, o, q + 2 * Fb + sz);
    cy_r = bload<T>(rC, o, q + Fb + sz);
    cz_r = bload<T>(rC, o, q + 2 * Fb + sz);
  }
  // ---- layers ----
  bool py = false, pz = false, px = false;                  // half nodes: memory of H
  bool nyj = false, nyp = false, nzk = false, nzp = false;  // nodes j, j + 1, k, k + 1: memory of E
  bool nx0 = false, nxr = false;                            // nodes i and, of the edge lane, i0 + 64
  int ly = 0, lz = 0, lyj = 0, lyp = 0, lzk = 0, lzp = 0, lxr = 0;
  uint32_t cxh = 0, cxn = 0;
  if constexpr (YZ) {
    py = pml_half(j, L.ny, npml, ly);
    pz = pml_half(k, L.nz, npml, lz);
    nyj = j >= 1 && pml_int(j, L.ny, npml, lyj);
    nyp = j + 1 < L.ny && pml_int(j + 1, L.ny, npml, lyp);
    nzk = k >= 1 && pml_int(k, L.nz, npml, lzk);
    nzp = k + 1 < L.nz && pml_int(k + 1, L.nz, npml, lzp);
  }
  if constexpr (XL) {
    px = (i < npml) | (i >= L.nx - npml);
    nx0 = (i >= 1) & ((i < npml) | (i > L.nx - npml));
    cxh = (uint32_t)(i < npml ? i : i - L.nx + W) * sz;
    cxn = (uint32_t)(i < npml ? i : i - L.nx + W - 1) * sz;
    nxr = right && pml_int(i0 + 64, L.nx, npml, lxr);
  }
  const int64_t sp = (int64_t)s * L.psi_src;
  const __amdgpu_buffer_rsrc_t rP = rsrc_of(L.p0 + sp);
  const uint32_t r0 = (uint32_t)(k * L.NY + j) * (uint32_t)W * sz;
  const uint32_t oY = L.oYb + x0, oZ = L.oZb + x0;
  auto rowY = [&](int l) { return oY + (uint32_t)(k * W + l) * L.PXb; };
  auto rowZ = [&](int l) { return oZ + (uint32_t)(l * L.NY + j) * L.PXb; };
  T p_hx_y = T(0), p_hz_y = T(0), p_hx_z = T(0), p_hy_z = T(0), p_hy_x = T(0), p_hz_x = T(0);
  T ex_yj = T(0), ez_yj = T(0), ex_yp = T(0), ez_yp = T(0), ex_zk = T(0), ey_zk = T(0), ex_zp = T(0),
    ey_zp = T(0), ey_x = T(0), ez_x = T(0), ey_xr = T(0), ez_xr = T(0);
  T bh = T(0), kn = T(0), an = T(0);
  if constexpr (YZ) {
    if (py) {
      p_hx_y = bload<T>(rP, o, rowY(ly));
      p_hz_y = bload<T>(rP, o, rowY(ly) + L.sYb);
    }
    if (pz) {
      p_hx_z = bload<T>(rP, o, rowZ(lz));
      p_hy_z = bload<T>(rP, o, rowZ(lz) + L.sZb);
    }
    if (nyj) {
      ex_yj = bload<T>(rP, o, rowY(lyj) + 2 * L.sYb);
      ez_yj = bload<T>(rP, o, rowY(lyj) + 3 * L.sYb);
    }
    if (nyp) {
      ex_yp = bload<T>(rP, o, rowY(lyp) + 2 * L.sYb);
      ez_yp = bload<T>(rP, o, rowY(lyp) + 3 * L.sYb);
    }
    if (nzk) {
      ex_zk = bload<T>(rP, o, rowZ(lzk) + 2 * L.sZb);
      ey_zk = bload<T>(rP, o, rowZ(lzk) + 3 * L.sZb);
    }
    if (nzp) {
      ex_zp = bload<T>(rP, o, rowZ(lzp) + 2 * L.sZb);
      ey_zp = bload<T>(rP, o, rowZ(lzp) + 3 * L.sZb);
    }
  }
  if constexpr (XL) {
    if (px) {
      p_hy_x = bload<T>(rP, cxh, r0);
      p_hz_x = bload<T>(rP, cxh, r0 + L.sXb);
      bh = bload<T>(rX, o, x0 + AX_BH * L.LAb);
    }
    if (nx0) {
      ey_x = bload<T>(rP, cxn, r0 + 2 * L.sXb);
      ez_x = bload<T>(rP, cxn, r0 + 3 * L.sXb);
      kn = bload<T>(rX, o, x0 + AX_KN * L.LAb);
      an = bload<T>(rX, o, x0 + AX_AN * L.LAb);
    }
    if (nxr && tid == 63) {
      ey_xr = bload<T>(rP, (uint32_t)lxr * sz, r0 + 2 * L.sXb);
      ez_xr = bload<T>(rP, (uint32_t)lxr * sz, r0 + 3 * L.sXb);
    }
  }
  // own H multipliers: the deferred update of their memory
  const T dtmu = L.dtmu;
  if constexpr (YZ) {
    if (py) {
      bstore<false>(yj.bh * (-dtmu * hx + p_hx_y), rP, o, rowY(ly));
      bstore<false>(yj.bh * (dtmu * hz + p_hz_y), rP, o, rowY(ly) + L.sYb);
    }
    if (pz) {
      bstore<false>(zk.bh * (dtmu * hx + p_hx_z), rP, o, rowZ(lz));
      bstore<false>(zk.bh * (-dtmu * hy + p_hy_z), rP, o, rowZ(lz) + L.sZb);
    }
  }
  if constexpr (XL) {
    if (px) {
      bstore<false>(bh * (dtmu * hy + p_hy_x), rP, cxh, r0);
      bstore<false>(bh * (-dtmu * hz + p_hz_x), rP, cxh, r0 + L.sXb);
    }
  }
  // aD / hd of the E differences (edges that are not updated: dt/eps is zero)
  const T vx = cx * ax, vy = cy * ay, vz = cz * az;
  const T x1 = td_ad<YZ>(vx, yj.ihd, nyj, ex_yj, yj.kn, yj.an);                    // E_x d1 at j
  const T x1p = td_ad<YZ>(cx_j * ax_j, yp.ihd, nyp, ex_yp, yp.kn, yp.an);          // at j + 1
  const T x2 = td_ad<YZ>(-vx, zk.ihd, nzk, ex_zk, zk.kn, zk.an);                   // E_x d2 at k
  const T x2p = td_ad<YZ>(-(cx_k * ax_k), zp.ihd, nzp, ex_zp, zp.kn, zp.an);       // at k + 1
  const T y1 = td_ad<YZ>(vy, zk.ihd, nzk, ey_zk, zk.kn, zk.an);                    // E_y d1 at k
  const T y1p = td_ad<YZ>(cy_k * ay_k, zp.ihd, nzp, ey_zp, zp.kn, zp.an);
  const T y2 = td_ad<XL>(-vy, ihd, nx0, ey_x, kn, an);                             // E_y d2 at i
  const T z1 = td_ad<XL>(vz, ihd, nx0, ez_x, kn, an);                              // E_z d1 at i
  const T z2 = td_ad<YZ>(-vz, yj.ihd, nyj, ez_yj, yj.kn, yj.an);                   // E_z d2 at j
  const T z2p = td_ad<YZ>(-(cz_j * az_j), yp.ihd, nyp, ez_yp, yp.kn, yp.an);
  const T y2r = td_ad<XL>(-(cy_r * ay_r), xr.ihd, nxr, ey_xr, xr.kn, xr.an);
  const T z1r = td_ad<XL>(cz_r * az_r, xr.ihd, nxr, ez_xr, xr.kn, xr.an);
  const T y2p = lane_above(y2r, y2), z1p = lane_above(z1r, z1);
  T nh[3] = {hx + (y1 - y1p + z2 - z2p), hy + (x2 - x2p + z1 - z1p), hz + (x1 - x1p + y2 - y2p)};
  if constexpr (ENT) td_sens_row<3>(A, ent, C, z, s, nh);
  bstore<false>(nh[0], rO, o, q + 3 * Fb);
  bstore<false>(nh[1], rO, o, q + 4 * Fb);
  bstore<false>(nh[2], rO, o, q + 5 * Fb);
}

template <typename T, bool XL, bool YZ, bool ENT>
__device__ __forceinline__ void td_h_wave(const LeapArgs<T> &L, const StepArgs<T> &A, int s, int2 row, int i0,
                                          int j, int k, const T *Enew, const T *Eold, const double *tdw,
                                          const double2 *C, const double2 *z) {
  const bool j_lo = !YZ || j >= 1, k_lo = !YZ || k >= 1, left = !XL || i0 > 0;
  const int jm = j_lo ? j - 1 : j, km = k_lo ? k - 1 : k;
  const AxRow<T> yj = L.axr[L.LA + j], ym = L.axr[L.LA + jm], zk = L.axr[2 * L.LA + k],
                 zm = L.axr[2 * L.LA + km], xl = L.axr[left ? i0 - 1 : 0];
  asm volatile("; tdh %0" ::"n"(XL * 4 + YZ * 2 + ENT));   // see leap_wave
  const int tid = threadIdx.x, i = i0 + tid;
  RowEnt ent;
  if constexpr (ENT) ent = row_entries(L, A, row, s, tid);
  const int npml = L.npml, W = 2 * npml;
  const uint32_t sz = sizeof(T), x0 = (uint32_t)i0 * sz, o = (uint32_t)tid * sz, Fb = L.Fb;
  const uint32_t q = (uint32_t)k * L.PLb + (uint32_t)j * L.PXb + x0;
  // rows below a wall are replaced by the node's own: their values reach no
  // stored result
  const uint32_t qj = j_lo ? q - L.PXb : q, qk = k_lo ? q - L.PLb : q;
  const bool i_lo = !XL || i >= 1;
  const bool okx = j_lo && k_lo, oky = i_lo && k_lo, okz = i_lo && j_lo;
  const __amdgpu_buffer_rsrc_t rA = rsrc_of(L.f0 + (int64_t)s * L.F6), rO = rA,
                               rC = rsrc_of(L.ce), rX = rsrc_of(L.axt);
  const T hx = bload<T>(rA, o, q + 3 * Fb), hy = bload<T>(rA, o, q + 4 * Fb), hz = bload<T>(rA, o, q + 5 * Fb);
  const T hx_j = bload<T>(rA, o, qj + 3 * Fb), hz_j = bload<T>(rA, o, qj + 5 * Fb);
  const T hx_k = bload<T>(rA, o, qk + 3 * Fb), hy_k = bload<T>(rA, o, qk + 4 * Fb);
  const T ax = bload<T>(rA, o, q), ay = bload<T>(rA, o, q + Fb), az = bload<T>(rA, o, q + 2 * Fb);
  const T cx = bload<T>(rC, o, q), cy = bload<T>(rC, o, q + Fb), cz = bload<T>(rC, o, q + 2 * Fb);
  const T ih = bload<T>(rX, o, x0 + AX_IH * L.LAb);
  T hy_l = T(0), hz_l = T(0);
  if (left && tid == 0) {
    hy_l = bload<T>(rA, o, q + 4 * Fb - sz);
    hz_l = bload<T>(rA, o, q + 5 * Fb - sz);
  }
  // gradient product of the own edges
  const int64_t e0 = (int64_t)s * (L.F6 >> 1);
  const __amdgpu_buffer_rsrc_t rN = rsrc_of(Enew + e0), rD = rsrc_of(Eold + e0), rW = rsrc_of(tdw),
                               rG = rsrc_of(A.gedge + e0);
  const T n0 = bload<T>(rN, o, q), n1 = bload<T>(rN, o, q + Fb), n2 = bload<T>(rN, o, q + 2 * Fb);
  const T d0 = bload<T>(rD, o, q), d1 = bload<T>(rD, o, q + Fb), d2 = bload<T>(rD, o, q + 2 * Fb);
  constexpr uint32_t up = 8 / sizeof(T);                    // byte offsets of the FP64 arrays
  const uint32_t og = o * up, qg = q * up, Fg = Fb * up;
  const double w0 = bload<double>(rW, og, qg), w1 = bload<double>(rW, og, qg + Fg),
               w2 = bload<double>(rW, og, qg + 2 * Fg);
  const double g0 = bload<double>(rG, og, qg), g1 = bload<double>(rG, og, qg + Fg),
               g2 = bload<double>(rG, og, qg + 2 * Fg);
  // ---- layers ----
  bool hyj = false, hym = false, hzk = false, hzm = false, hx0 = false, hxl = false;   // memory of H
  bool nyj = false, nzk = false, nx0 = false;                                          // memory of E
  int lyj = 0, lym = 0, lzk = 0, lzm = 0, lxl = 0, ny = 0, nz = 0;
  uint32_t cxh = 0, cxn = 0;
  if constexpr (YZ) {
    hyj = pml_half(j, L.ny, npml, lyj);
    hym = j_lo && pml_half(jm, L.ny, npml, lym);
    hzk = pml_half(k, L.nz, npml, lzk);
    hzm = k_lo && pml_half(km, L.nz, npml, lzm);
    nyj = j_lo && pml_int(j, L.ny, npml, ny);
    nzk = k_lo && pml_int(k, L.nz, npml, nz);
  }
  if constexpr (XL) {
    hx0 = (i < npml) | (i >= L.nx - npml);
    nx0 = i_lo & ((i < npml) | (i > L.nx - npml));
    cxh = (uint32_t)(i < npml ? i : i - L.nx + W) * sz;
    cxn = (uint32_t)(i < npml ? i : i - L.nx + W - 1) * sz;
    hxl = left && pml_half(i0 - 1, L.nx, npml, lxl);
  }
  const __amdgpu_buffer_rsrc_t rP = rsrc_of(L.p0 + (int64_t)s * L.psi_src);
  const uint32_t r0 = (uint32_t)(k * L.NY + j) * (uint32_t)W * sz;
  const uint32_t oY = L.oYb + x0, oZ = L.oZb + x0;
  auto rowY = [&](int l) { return oY + (uint32_t)(k * W + l) * L.PXb; };
  auto rowZ = [&](int l) { return oZ + (uint32_t)(l * L.NY + j) * L.PXb; };
  T hx_yj = T(0), hz_yj = T(0), hx_ym = T(0), hz_ym = T(0), hx_zk = T(0), hy_zk = T(0), hx_zm = T(0),
    hy_zm = T(0), hy_x = T(0), hz_x = T(0), hy_xl = T(0), hz_xl = T(0);
  T ex_y = T(0), ez_y = T(0), ex_z = T(0), ey_z = T(0), ey_x = T(0), ez_x = T(0);
  T kh = T(0), ah = T(0), bn = T(0);
  if constexpr (YZ) {
    if (hyj) {
      hx_yj = bload<T>(rP, o, rowY(lyj));
      hz_yj = bload<T>(rP, o, rowY(lyj) + L.sYb);
    }
    if (hym) {
      hx_ym = bload<T>(rP, o, rowY(lym));
      hz_ym = bload<T>(rP, o, rowY(lym) + L.sYb);
    }
    if (hzk) {
      hx_zk = bload<T>(rP, o, rowZ(lzk));
      hy_zk = bload<T>(rP, o, rowZ(lzk) + L.sZb);
    }
    if (hzm) {
      hx_zm = bload<T>(rP, o, rowZ(lzm));
      hy_zm = bload<T>(rP, o, rowZ(lzm) + L.sZb);
    }
    if (nyj) {
      ex_y = bload<T>(rP, o, rowY(ny) + 2 * L.sYb);
      ez_y = bload<T>(rP, o, rowY(ny) + 3 * L.sYb);
    }
    if (nzk) {
      ex_z = bload<T>(rP, o, rowZ(nz) + 2 * L.sZb);
      ey_z = bload<T>(rP, o, rowZ(nz) + 3 * L.sZb);
    }
  }
  if constexpr (XL) {
    if (hx0) {
      hy_x = bload<T>(rP, cxh, r0);
      hz_x = bload<T>(rP, cxh, r0 + L.sXb);
      kh = bload<T>(rX, o, x0 + AX_KH * L.LAb);
      ah = bload<T>(rX, o, x0 + AX_AH * L.LAb);
    }
    if (hxl && tid == 0) {
      hy_xl = bload<T>(rP, (uint32_t)lxl * sz, r0);
      hz_xl = bload<T>(rP, (uint32_t)lxl * sz, r0 + L.sXb);
    }
    if (nx0) {
      ey_x = bload<T>(rP, cxn, r0 + 2 * L.sXb);
      ez_x = bload<T>(rP, cxn, r0 + 3 * L.sXb);
      bn = bload<T>(rX, o, x0 + AX_BN * L.LAb);
    }
  }
  // own E multipliers: the deferred update of their memory, and the product
  const T vx = cx * ax, vy = cy * ay, vz = cz * az;
  if constexpr (YZ) {
    if (nyj) {
      if (okx) bstore<false>(yj.bn * (vx + ex_y), rP, o, rowY(ny) + 2 * L.sYb);
      if (okz) bstore<false>(yj.bn * (-vz + ez_y), rP, o, rowY(ny) + 3 * L.sYb);
    }
    if (nzk) {
      if (okx) bstore<false>(zk.bn * (-vx + ex_z), rP, o, rowZ(nz) + 2 * L.sZb);
      if (oky) bstore<false>(zk.bn * (vy + ey_z), rP, o, rowZ(nz) + 3 * L.sZb);
    }
  }
  if constexpr (XL) {
    if (nx0) {
      if (oky) bstore<false>(bn * (-vy + ey_x), rP, cxn, r0 + 2 * L.sXb);
      if (okz) bstore<false>(bn * (vz + ez_x), rP, cxn, r0 + 3 * L.sXb);
    }
  }
  if (okx) bstore<false>(g0 + (double)ax * ((double)n0 - (double)d0) * w0, rG, og, qg);
  if (oky) bstore<false>(g1 + (double)ay * ((double)n1 - (double)d1) * w1, rG, og, qg + Fg);
  if (okz) bstore<false>(g2 + (double)az * ((double)n2 - (double)d2) * w2, rG, og, qg + 2 * Fg);
  // aD / h of the H differences: d1 multiplier -dt/mu aH, d2 +dt/mu aH
  const T dtmu = L.dtmu;
  const T x1 = td_ad<YZ>(-dtmu * hx, yj.ih, hyj, hx_yj, yj.kh, yj.ah);             // H_x d1 at j
  const T x1m = td_ad<YZ>(-dtmu * hx_j, ym.ih, hym, hx_ym, ym.kh, ym.ah);          // at j - 1
  const T x2 = td_ad<YZ>(dtmu * hx, zk.ih, hzk, hx_zk, zk.kh, zk.ah);              // H_x d2 at k
  const T x2m = td_ad<YZ>(dtmu * hx_k, zm.ih, hzm, hx_zm, zm.kh, zm.ah);
  const T y1 = td_ad<YZ>(-dtmu * hy, zk.ih, hzk, hy_zk, zk.kh, zk.ah);             // H_y d1 at k
  const T y1m = td_ad<YZ>(-dtmu * hy_k, zm.ih, hzm, hy_zm, zm.kh, zm.ah);
  const T y2 = td_ad<XL>(dtmu * hy, ih, hx0, hy_x, kh, ah);                        // H_y d2 at i
  const T z1 = td_ad<XL>(-dtmu * hz, ih, hx0, hz_x, kh, ah);                       // H_z d1 at i
  const T z2 = td_ad<YZ>(dtmu * hz, yj.ih, hyj, hz_yj, yj.kh, yj.ah);              // H_z d2 at j
  const T z2m = td_ad<YZ>(dtmu * hz_j, ym.ih, hym, hz_ym, ym.kh, ym.ah);
  const T y2l = td_ad<XL>(dtmu * hy_l, xl.ih, hxl, hy_xl, xl.kh, xl.ah);
  const T z1l = td_ad<XL>(-dtmu * hz_l, xl.ih, hxl, hz_xl, xl.kh, xl.ah);
  const T y2m = lane_below(y2l, y2), z1m = lane_below(z1l, z1);
  T ne[3] = {ax + (y1m - y1 + z2m - z2), ay + (x2m - x2 + z1m - z1), az + (x1m - x1 + y2m - y2)};
  if constexpr (ENT) td_sens_row<0>(A, ent, C, z, s, ne);
  if (okx) bstore<false>(ne[0], rO, o, q);
  if (oky) bstore<false>(ne[1], rO, o, q + Fb);
  if (okz) bstore<false>(ne[2], rO, o, q + 2 * Fb);
}

template <typename T>
__global__ void __launch_bounds__(64) k_rows_td_e(LeapArgs<T> L, StepArgs<T> A, const double2 *C,
                                                  const double2 *z) {
  int bx, j, k, s;
  const int b = row_of(L, bx, j, k, s);
  const int i0 = bx * 64;
  if (i0 + (int)threadIdx.x >= L.nx) return;
  bool xl, yz;
  row_kind(L, i0, j, k, xl, yz);
  // z: null where no magnetic receiver is recorded
  int2 row = make_int2(-1, -1);
  if (z) row = row_tables(L, b, bx, j, k, s, 0, 1);
  if (max(row.x, row.y) >= 0)
    td_e_wave<T, true, true, true>(L, A, s, row, i0, j, k, C, z);
  else if (xl) {
    if (yz) td_e_wave<T, true, true, false>(L, A, s, row, i0, j, k, C, z);
    else td_e_wave<T, true, false, false>(L, A, s, row, i0, j, k, C, z);
  } else {
    if (yz) td_e_wave<T, false, true, false>(L, A, s, row, i0, j, k, C, z);
    else td_e_wave<T, false, false, false>(L, A, s, row, i0, j, k, C, z);
  }
}

template <typename T>
__global__ void __launch_bounds__(64) k_rows_td_h(LeapArgs<T> L, StepArgs<T> A, const T *Enew, const T *Eold,
                                                  const double *tdw, const double2 *C, const double2 *z) {
  int bx, j, k, s;
  const int b = row_of(L, bx, j, k, s);
  const int i0 = bx * 64;
  if (i0 + (int)threadIdx.x >= L.nx) return;
  bool xl, yz;
  row_kind(L, i0, j, k, xl, yz);
  // z: null at the first step (no sample before it)
  int2 row = make_int2(-1, -1);
  if (z) row = row_tables(L, b, bx, j, k, s, 0, 1);
  if (max(row.x, row.y) >= 0)
    td_h_wave<T, true, true, true>(L, A, s, row, i0, j, k, Enew, Eold, tdw, C, z);
  else if (xl) {
    if (yz) td_h_wave<T, true, true, false>(L, A, s, row, i0, j, k, Enew, Eold, tdw, C, z);
    else td_h_wave<T, true, false, false>(L, A, s, row, i0, j, k, Enew, Eold, tdw, C, z);
  } else {
    if (yz) td_h_wave<T, false, true, false>(L, A, s, row, i0, j, k, Enew, Eold, tdw, C, z);
    else td_h_wave<T, false, false, false>(L, A, s, row, i0, j, k, Enew, Eold, tdw, C, z);
  }
}

// a[s][node] += -Re sum_k C[s][node][k] z[k]: the sensitivity of the misfit
// to the sample at the receiver nodes of one kind, E (magnetic = 0: the
// sample E^m, z = zE row m-1 = z^m) or H (magnetic = 1: the sample
// H^{n+1/2}, z = zH row n = z^{n+1/2}).  One thread per (source, node).
template <typename T>
__global__ void k_td_sens(T *adj, int64_t F, int ns, int nn, int nf, const int *rn_c,
                          const int64_t *rn_idx, const double2 *C, const double2 *z,
                          int magnetic) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= ns * nn) return;
  const int s = t / nn, node = t % nn;
  if ((rn_c[node] >= 3) != (magnetic != 0)) return;
  double g = 0.0;
  for (int kf = 0; kf < nf; ++kf) {
    const double2 c = C[((int64_t)s * nn + node) * nf + kf];
    g -= c.x * z[kf].x - c.y * z[kf].y;
  }
  T *a = adj + (int64_t)s * 6 * F + (int64_t)rn_c[node] * F + rn_idx[node];
  *a += (T)g;
}

// Magnetic receivers and magnetic adjoint sources, one thread per (source, H
// receiver node); both run beside the step's own launches and read the step
// index like them (n = last completed step + 1).
//   k_hrec, after the fused step n: racc[s][node] += H^{n+1/2} z^{n+1/2}
//     (eq. dtft transforms H' too; H^{n+1/2} is in half (n&1)^1).  The
//     two-kernel schedule records in the E update instead (record_h).
//   k_hinj, before the fused step n (adjoint runs): H^{n-1/2} += (dt/mu)
//     M'^n with M'^n = sum_r coef[s][node][r] F[r][n], the magnetic current
//     of the Faraday row (eq. fictitiouswave) acting at n dt; the step then
//     reads it from half n&1.  The two-kernel schedule adds it inside the H
//     update instead (inject_h).
template <typename T>
__device__ __forceinline__ T *h_comp(const Half<T> &H, int c) {
  return c == 3 ? H.hx : (c == 4 ? H.hy : H.hz);
}

template <typename T>
__global__ void k_hrec(StepArgs<T> A, const int *hn, int nh, const int *rn_c,
                       const int64_t *rn_idx, const double2 *zH) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= A.ns * nh) return;
  const int n = A.step[0] + 1;
  if (n >= A.nt) return;                    // no recording past the run
  const int s = t / nh, node = hn[t - s * nh];
  const T *f = h_comp(half_of(A, (n & 1) ^ 1, s), rn_c[node]);
  const double v = (double)f[rn_idx[node]];
  double2 *a = A.racc + ((int64_t)s * A.nn + node) * A.nf;
  const double2 *z = zH + (int64_t)n * A.nf;
  for (int kf = 0; kf < A.nf; ++kf) {
    double2 x = a[kf];
    x.x = fma(v, z[kf].x, x.x);
    x.y = fma(v, z[kf].y, x.y);
    a[kf] = x;
  }
}

template <typename T>
__global__ void k_hinj(StepArgs<T> A, const int *hn, int nh, const int *rn_c,
                       const int64_t *rn_idx, double dtmu) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= A.ns * nh) return;
  const int n = A.step[0] + 1;
  if (n >= A.nt) return;
  const int s = t / nh, node = hn[t - s * nh];
  const double *cf = A.coef + ((int64_t)s * A.nn + node) * A.nrow;
  double v = 0.0;
  for (int r = 0; r < A.nrow; ++r) v = fma(cf[r], A.Ftab[(int64_t)r * A.nt + n], v);
  T *f = h_comp(half_of(A, n & 1, s), rn_c[node]);
  const int64_t q = rn_idx[node];
  f[q] = (T)((double)f[q] + dtmu * v);
}

// Forward magnetic dipole sources under the fused schedule, one thread per
// injection target, before the fused step n: H^{n-1/2} += (dt/mu) M'^n with
// M'^n = coef * w_n (the arithmetic of inject_h, so every schedule gives the
// same bits).  Targets of the electric kind (c < 3) are skipped.
template <typename T>
__global__ void k_hsrc(StepArgs<T> A, const int *tg_s, const int *tg_c, const int64_t *tg_idx,
                       int ntg, double dtmu) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= ntg) return;
  const int n = A.step[0] + 1;
  if (n >= A.nt || tg_c[t] < 3) return;
  const double v = fma(A.coef[t], A.Ftab[n], 0.0);
  if (v == 0.0) return;                      // as inject_h: a zero leaves the node alone
  T *f = h_comp(half_of(A, n & 1, tg_s[t]), tg_c[t]);
  const int64_t q = tg_idx[t];
  f[q] = (T)((double)f[q] + dtmu * v);
}

// dst [ns][3][F] <- E of every source in half `half` of the double buffer
template <typename T>
__global__ void k_copy_e(T *dst, const T *fields, int64_t fbuf, int half, int ns, int64_t F) {
  const int64_t n3 = 3 * F, total = (int64_t)ns * n3;
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < total;
       t += (int64_t)gridDim.x * blockDim.x) {
    const int s = (int)(t / n3);
    dst[t] = fields[half * fbuf + (int64_t)s * 6 * F + (t - s * n3)];
  }
}

// Coefficients of the adjoint injection (eq. adj2, reading: the electric
// residual is an electric current source carrying sqrt(-i w / 2 w0)), one
// thread per (source, receiver node): the spectrum s_k = fac_k conj(r_k)
// summed over the residual rows touching the node with their trilinear
// weights, as the real vector [Re s_1..Re s_nf, Im s_1..Im s_nf] of eq.
// basis; a magnetic node (H lattice) takes fac_h = z_k^{1/2}, since the
// basis functions reproduce spectra at the injection times (n+1/2) dt of J'
// while M' enters H at n dt.  inc bounds the node's largest injected
// increment: sum_r |t_r| max_n |b_r(n)| times its update factor (dt/eps or
// dt/mu).
__global__ void k_adj_coef(int ns, int nn, int nf, int rows, const double *resid,
                           const int *at_ptr, const int *at_row, const double *at_w,
                           const int *rn_c, const double2 *fac, const double2 *fac_h,
                           const double *bmax, const double *nodefac, double *T, double *inc) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= ns * nn) return;
  const int s = t / nn, node = t - s * nn, m = 2 * nf;
  double *c = T + (int64_t)t * m;
  for (int r = 0; r < m; ++r) c[r] = 0.0;
  const double2 *f = rn_c[node] >= 3 ? fac_h : fac;
  for (int e = at_ptr[node]; e < at_ptr[node + 1]; ++e) {
    const int row = at_row[e];
    const double w = at_w[e];
    for (int k = 0; k < nf; ++k) {
      const double *rr = resid + 2 * (((int64_t)s * rows + row) * nf + k);
      const double a = f[k].x, b = f[k].y, cr = rr[0], ci = -rr[1];
      const double re = a * cr - b * ci, im = a * ci + b * cr;
      c[k] += w * re;
      c[nf + k] += w * im;
    }
  }
  double sum = 0.0;
  for (int r = 0; r < m; ++r) sum += fabs(c[r]) * bmax[r];
  inc[t] = sum * nodefac[node];
}

// The power of two nearest (in log2) to 1 / max inc, so that the injected
// increments stay near 1 (exact scaling); scale_v[k] = 1 / scale for the
// adjoint receiver output.  One block.
__global__ void k_adj_scale(const double *inc, int n, int nf, double *scale, double2 *scale_v) {
  __shared__ double s_big[256];
  double big = 0.0;
  for (int t = threadIdx.x; t < n; t += blockDim.x) big = fmax(big, inc[t]);
  s_big[threadIdx.x] = big;
  __syncthreads();
  for (int h = blockDim.x / 2; h > 0; h >>= 1) {
    if (threadIdx.x < h) s_big[threadIdx.x] = fmax(s_big[threadIdx.x], s_big[threadIdx.x + h]);
    __syncthreads();
  }
  big = s_big[0];
  double sc = 1.0;
  if (big > 0.0) {
    // round(log2(1 / big)) from the exponent and mantissa: 1 / big = m 2^e
    // with m in [1/2, 1), log2 m in [-1, 0) rounds to 0 from m >= 2^-1/2
    int e = 0;
    const double m = frexp(1.0 / big, &e);
    sc = ldexp(1.0, m >= 0.70710678118654752440 ? e : e - 1);
  }
  if (threadIdx.x == 0) scale[0] = sc;
  for (int k = threadIdx.x; k < nf; k += blockDim.x) scale_v[k] = make_double2(1.0 / sc, 0.0);
}

__global__ void k_adj_apply(double *T, int64_t n, const double *scale) {
  const double sc = scale[0];
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < n;
       t += (int64_t)gridDim.x * blockDim.x)
    T[t] *= sc;
}

// receiver output: interpolate node transforms and scale per frequency; a
// row (receiver r, component position ci = row % ncomp) takes scale_h when
// its component is magnetic (rcomp >= 3), scale otherwise
__global__ void k_rec_out(int ns, int nrows, int nn, int nf, const int *ptr, const int *node,
                          const double *w, const double2 *racc, const double2 *scale,
                          const double2 *scale_h, const int *rcomp, int ncomp, double2 *out) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= ns * nrows * nf) return;
  const int kf = t % nf, row = (t / nf) % nrows, s = t / (nf * nrows);
  if (rcomp[row % ncomp] >= 3) scale = scale_h;
  double re = 0, im = 0;
  for (int e = ptr[row]; e < ptr[row + 1]; ++e) {
    const double2 a = racc[((int64_t)s * nn + node[e]) * nf + kf];
    re += w[e] * a.x;
    im += w[e] * a.y;
  }
  const double2 sc = scale[kf];
  out[t] = make_double2(re * sc.x - im * sc.y, re * sc.y + im * sc.x);
}

// gradient per cell from the 12 edges of the cell: with volume-weighted
// edge averaging, dV_e * d sigma_e / d sigma_c = V_c / 4 for every edge of
// the cell, so d phi / d ln rho_c = sigma_c V_c / 4 * sum_edges gacc * gscale
// (gacc summed over the sources).  VTI (Section 3.1): the x and y edges give
// d / d ln rho_h (factor sigma_h V / 4), the z edges d / d ln rho_v (factor
// sigma_v V / 4); split = 1 writes the two as grad[0], grad[1], else their
// sum (rho_h and rho_v scaled together).  With fourth-order differences the
// dual volume of an edge is in metric lengths; vr then holds, per axis, the
// ratios metric / cell width (half nodes) and metric / dual width (nodes) at
// stride LA, and each edge term is scaled by the product of its three.
__global__ void k_grad_cells(int nx, int ny, int nz, int ns, int PX, int NY, int64_t F,
                             const double *gedge, const double *cellfac, const double *cellfac_v,
                             double gscale, const double *gdiv, double *grad, int accumulate,
                             int split, const double *vr, int LA) {
  // gdiv (device, may be null): the scale is 1 / (gscale gdiv[0])
  if (gdiv) gscale = 1.0 / (gscale * gdiv[0]);
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  const int j = blockIdx.y;
  const int k = blockIdx.z;
  if (i >= nx) return;
  const int64_t plane = (int64_t)NY * PX;
  const int64_t q = (int64_t)k * plane + (int64_t)j * PX + i;
  const int64_t ox[4] = {0, PX, plane, plane + PX}, oy[4] = {0, 1, plane, plane + 1},
                oz[4] = {0, 1, PX, PX + 1};
  double ex[4] = {0, 0, 0, 0}, ey[4] = {0, 0, 0, 0}, ez[4] = {0, 0, 0, 0};
  for (int s = 0; s < ns; ++s) {
    const double *gx = gedge + (int64_t)s * 3 * F, *gy = gx + F, *gz = gx + 2 * F;
    for (int e = 0; e < 4; ++e) {
      ex[e] += gx[q + ox[e]];
      ey[e] += gy[q + oy[e]];
      ez[e] += gz[q + oz[e]];
    }
  }
  if (vr) {
    const double *hx = vr, *nxr = vr + LA, *hy = vr + 2 * LA, *nyr = vr + 3 * LA,
                 *hz = vr + 4 * LA, *nzr = vr + 5 * LA;
    for (int e = 0; e < 4; ++e) {
      const int a = e & 1, b = e >> 1;
      ex[e] *= hx[i] * nyr[j + a] * nzr[k + b];
      ey[e] *= hy[j] * nxr[i + a] * nzr[k + b];
      ez[e] *= hz[k] * nxr[i + a] * nyr[j + b];
    }
  }
  const double sx = ex[0] + ex[1] + ex[2] + ex[3];
  const double sy = ey[0] + ey[1] + ey[2] + ey[3];
  const double sz = ez[0] + ez[1] + ez[2] + ez[3];
  const int64_t c = ((int64_t)k * ny + j) * nx + i;
  const double vh = cellfac[c] * (sx + sy) * gscale, vv = cellfac_v[c] * sz * gscale;
  if (split) {
    const int64_t nc = (int64_t)nx * ny * nz;
    grad[c] = accumulate ? grad[c] + vh : vh;
    grad[nc + c] = accumulate ? grad[nc + c] + vv : vv;
  } else {
    grad[c] = accumulate ? grad[c] + (vh + vv) : vh + vv;
  }
}

// normalised volume export: out[s][k][c][z][y][x] = V * scale_k; the
// (s, kf, c, z) planes are walked with a grid-stride loop over blockIdx.z
template <int ACC>
__global__ void k_vol_export(int ns, int nf, int NX, int NY, int NZ, int PX, int64_t F,
                             const void *vol, const double2 *scale, double2 *out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  const int j = blockIdx.y;
  if (i >= NX) return;
  const int total = ns * nf * 3 * NZ;
  for (int zc = blockIdx.z; zc < total; zc += gridDim.z) {
    const int k = zc % NZ;
    const int c = (zc / NZ) % 3;
    const int kf = (zc / (NZ * 3)) % nf;
    const int s = zc / (NZ * 3 * nf);
    const int64_t q = ((int64_t)k * NY + j) * PX + i;
    const double2 v = acc_read<ACC>(vol, (((int64_t)s * nf + kf) * 3 + c) * F + q);
    const double2 sc = scale[kf];
    out[(int64_t)zc * NY * NX + (int64_t)j * NX + i] =
        make_double2(v.x * sc.x - v.y * sc.y, v.x * sc.y + v.y * sc.x);
  }
}

__global__ void k_set_int(int *p, int v) {
  if (threadIdx.x == 0 && blockIdx.x == 0) p[0] = v;
}

// Zero n bytes at p (16-byte stores, then the remaining bytes): a kernel
// rather than a memset node, so that a caller may capture the runs in a
// graph and replay them.
__global__ void k_zero(unsigned char *p, size_t n) {
  const size_t n16 = n / 16, stride = (size_t)gridDim.x * blockDim.x;
  uint4 *q = reinterpret_cast<uint4 *>(p);
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += stride)
    q[i] = make_uint4(0u, 0u, 0u, 0u);
  const size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t < n - n16 * 16) p[n16 * 16 + t] = 0;
}

static void zero_bytes(void *p, size_t n, hipStream_t st) {
  if (n == 0) return;
  const size_t blocks = std::min<size_t>((n / 16 + 255) / 256 + 1, 8192);
  hipLaunchKernelGGL(k_zero, dim3((unsigned)blocks), dim3(256), 0, st,
                     static_cast<unsigned char *>(p), n);
}

// ---------------------------------------------------------------------------
// device tables owned by the plan
// ---------------------------------------------------------------------------
struct DevBuf {
  void *p = nullptr;
  size_t n = 0;
};

struct Dev {
  int device = -1;
  uint64_t model_version = 0, basis_version = 0;
  std::vector<DevBuf> bufs;     // everything allocated for the tables
  // typed views
  void *ce = nullptr;    // [3][F]
  void *axt = nullptr;   // [3][AX_TABLES][LA]
  void *axr = nullptr;   // [3][LA] rows of the same (AxRow)
  int LA = 0;
  double2 *zE = nullptr, *Q = nullptr;
  double *wavelet = nullptr, *basis = nullptr;
  int *src_s = nullptr, *src_c = nullptr, *src_toff = nullptr;
  int64_t *src_idx = nullptr;
  double *src_coef = nullptr;
  int *rn_c = nullptr;
  int64_t *rn_idx = nullptr;
  int *ri_ptr = nullptr, *ri_node = nullptr;
  double *ri_w = nullptr;
  double2 *fwd_scale = nullptr, *adj_scale_v = nullptr, *vol_scale = nullptr;
  // magnetic receivers: the receiver nodes on H lattices (node ids), their
  // twiddles z^{n+1/2}, the forward scale of H rows, and the component of
  // each row position (k_rec_out picks the scale per row)
  int *hn = nullptr;
  int nh = 0;
  double2 *zH = nullptr, *fwd_scale_h = nullptr;
  int *rcomp = nullptr;
  // adjoint injection coefficients (rebuilt per call from the residual on
  // the device): the node -> residual-row table, the spectral factors of E
  // and H nodes, the basis functions' largest values, each node's update
  // factor, per-(source, node) increment bounds and the power-of-two scale
  double *at_coef = nullptr;
  int *at_ptr = nullptr, *at_row = nullptr;
  double *at_w = nullptr, *adj_bmax = nullptr, *adj_nodefac = nullptr, *adj_inc = nullptr;
  double *adj_scale = nullptr;
  double2 *adj_fac = nullptr, *adj_fac_h = nullptr;
  // per-thread entry tables for the current tiling: the E update's forward
  // (index 0) and adjoint (index 1) tables, and the H update's tables of
  // magnetic sources, adjoint (index 2) and forward (index 3; two-kernel and
  // persistent schedules); see build_lists
  int *tile_tab[4] = {nullptr, nullptr, nullptr, nullptr};
  int *tl_off[4] = {nullptr, nullptr, nullptr, nullptr};
  int2 *tl_ent[4] = {nullptr, nullptr, nullptr, nullptr};
  // the same for rows of waves (see build_rows), forward and adjoint runs
  int *row_tab = nullptr, *src_tab = nullptr, *row_rec = nullptr, *row_src = nullptr;
  int rec_mask = 0;
  int ent_box[2][4] = {{0, -1, 0, -1}, {0, -1, 0, -1}};   // rows j and planes k of the E update's entries
  int ntg = 0;                  // forward injection targets (src_s .. src_coef)
  std::string list_key;
  std::vector<DevBuf> list_bufs;
  double *cellfac = nullptr, *cellfac_v = nullptr;   // sigma_h V / 4, sigma_v V / 4
  double *vratio = nullptr;     // order 4: metric / plain dual-volume ratios per axis
  double2 *eadj = nullptr;      // adjoint receiver transform when the caller passes none
  // graphs
  hipStream_t cap = nullptr;
  // time-domain adjoint: 1/(sigma_e dV_e) [3][F], a table of the model built
  // by the first call that needs it (6 of 22 ms of a gradient of 192 steps of
  // 101x101x61 cells were spent building and sending it on each call)
  const double *tdw = nullptr;
  hipGraphExec_t exec = nullptr;
  std::string exec_key;
  // sampled per-kernel timing
  std::vector<hipEvent_t> ev;                  // six per sampled step
  std::vector<uint8_t> kstat_closed;           // bit 0: the sampled step closed a transform block; 1: one launch a step
  double kstat_ms[3] = {0, 0, 0};
  int kstat_n = 0, kstat_ntr = 0;
  int sample_every = 0;
};

static Dev &D(Plan &p) {
  if (!p.dev) p.dev = new Dev();
  return *static_cast<Dev *>(p.dev);
}

static void *dalloc(Dev &d, size_t bytes) {
  void *ptr = nullptr;
  if (bytes == 0) bytes = 16;
  hipError_t e = hipMalloc(&ptr, bytes);
  if (e != hipSuccess) fail(FWD_ERR_OOM, std::string("hipMalloc: ") + hipGetErrorString(e));
  d.bufs.push_back({ptr, bytes});
  return ptr;
}

template <typename V>
static V *upload(Dev &d, const std::vector<V> &h) {
  V *p = static_cast<V *>(dalloc(d, h.size() * sizeof(V)));
  if (!h.empty()) HIP_CHECK(hipMemcpy(p, h.data(), h.size() * sizeof(V), hipMemcpyHostToDevice));
  return p;
}

template <typename T>
static T *upload_as(Dev &d, const std::vector<double> &h) {
  std::vector<T> t(h.begin(), h.end());
  return upload(d, t);
}

// the captured graph holds the lists' addresses and goes with them
static void free_lists(Dev &d) {
  for (auto &b : d.list_bufs) (void)hipFree(b.p);
  if (d.exec) {
    (void)hipGraphExecDestroy(d.exec);
    d.exec = nullptr;
  }
  d.exec_key.clear();
  d.list_bufs.clear();
  d.list_key.clear();
  for (int m = 0; m < 4; ++m) {
    d.tile_tab[m] = d.tl_off[m] = nullptr;
    d.tl_ent[m] = nullptr;
  }
  d.row_tab = d.src_tab = d.row_rec = d.row_src = nullptr;
}

static void free_tables(Dev &d) {
  free_lists(d);
  for (auto &b : d.bufs) (void)hipFree(b.p);
  d.bufs.clear();
}

void dev_release(Plan &p) {
  if (!p.dev) return;
  Dev &d = D(p);
  free_tables(d);
  if (d.cap) (void)hipStreamDestroy(d.cap);
  for (auto e : d.ev) (void)hipEventDestroy(e);
  delete &d;
  p.dev = nullptr;
}

template <typename T>
static void upload_model_tables(Plan &p, Dev &d) {
  const int64_t F = p.field_elems();
  std::vector<double> ce(3 * F);
  for (int c = 0; c < 3; ++c) std::copy(p.ce[c].begin(), p.ce[c].end(), ce.begin() + c * F);
  d.ce = upload_as<T>(d, ce);
  const int LA = std::max(p.nx, std::max(p.ny, p.nz)) + 2;
  std::vector<double> t((size_t)3 * AX_TABLES * LA, 0.0);
  for (int a = 0; a < 3; ++a) {
    const Axis &ax = p.ax[a];
    double *b = t.data() + (size_t)a * AX_TABLES * LA;
    for (int i = 0; i < ax.n; ++i) b[AX_IH * LA + i] = 1.0 / ax.m[i];
    for (int i = 0; i <= ax.n; ++i) b[AX_IHD * LA + i] = 1.0 / ax.md[i];
    std::copy(ax.kinv_n.begin(), ax.kinv_n.end(), b + AX_KN * LA);
    std::copy(ax.b_n.begin(), ax.b_n.end(), b + AX_BN * LA);
    std::copy(ax.a_n.begin(), ax.a_n.end(), b + AX_AN * LA);
    std::copy(ax.kinv_h.begin(), ax.kinv_h.end(), b + AX_KH * LA);
    std::copy(ax.b_h.begin(), ax.b_h.end(), b + AX_BH * LA);
    std::copy(ax.a_h.begin(), ax.a_h.end(), b + AX_AH * LA);
  }
  d.axt = upload_as<T>(d, t);
  std::vector<double> rows(t.size());
  for (int a = 0; a < 3; ++a)
    for (int q = 0; q < AX_TABLES; ++q)
      for (int i = 0; i < LA; ++i)
        rows[((size_t)a * LA + i) * AX_TABLES + q] = t[((size_t)a * AX_TABLES + q) * LA + i];
  d.axr = upload_as<T>(d, rows);
  d.LA = LA;
}

static void ensure_tables(Plan &p, hipStream_t stream) {
  if (!p.have_model) fail(FWD_ERR_STATE, "no model set");
  Dev &d = D(p);
  int dev = 0;
  HIP_CHECK(hipGetDevice(&dev));
  if (d.model_version == p.model_version && d.basis_version == p.basis_version && d.device == dev)
    return;
  HIP_CHECK(hipStreamSynchronize(stream));
  free_tables(d);
  d.vratio = nullptr;
  d.tdw = nullptr;
  d.device = dev;
  if (!d.cap) HIP_CHECK(hipStreamCreateWithFlags(&d.cap, hipStreamNonBlocking));
  if (p.dtype == FWD_F64)
    upload_model_tables<double>(p, d);
  else
    upload_model_tables<float>(p, d);
  const int nf = p.nf();
  std::vector<double2> zE(p.zE.size());
  for (size_t q = 0; q < zE.size(); ++q) zE[q] = make_double2(p.zE[q].real(), p.zE[q].imag());
  d.zE = upload(d, zE);
  d.wavelet = upload(d, p.wavelet);
  // forward injection targets
  {
    std::vector<int> s, c, toff;
    std::vector<int64_t> idx;
    std::vector<double> coef;
    for (size_t t = 0; t < p.src_tg.size(); ++t) {
      s.push_back(p.src_tg[t].s);
      c.push_back(p.src_tg[t].c);
      idx.push_back(p.src_tg[t].idx);
      toff.push_back((int)t);
      coef.push_back(p.src_coef[t] * p.src_scale);
    }
    d.src_s = upload(d, s);
    d.src_c = upload(d, c);
    d.src_idx = upload(d, idx);
    d.src_toff = upload(d, toff);
    d.src_coef = upload(d, coef);
    d.ntg = (int)p.src_tg.size();
  }
  d.rn_c = upload(d, p.rn_c);
  d.rn_idx = upload(d, p.rn_idx);
  d.ri_ptr = upload(d, p.ri_ptr);
  d.ri_node = upload(d, p.ri_node);
  d.ri_w = upload(d, p.ri_w);
  std::vector<double2> sc(nf), vs(nf), sh(nf);
  for (int k = 0; k < nf; ++k) {
    const cplx v = p.norm[k] / p.src_scale, vh = p.norm_h[k] / p.src_scale;
    sc[k] = make_double2(v.real(), v.imag());
    sh[k] = make_double2(vh.real(), vh.imag());
  }
  d.fwd_scale = upload(d, sc);
  d.fwd_scale_h = upload(d, sh);
  d.rcomp = upload(d, p.comp);
  {
    std::vector<int> hn;
    for (size_t node = 0; node < p.rn_c.size(); ++node)
      if (p.rn_c[node] >= 3) hn.push_back((int)node);
    d.nh = (int)hn.size();
    d.hn = upload(d, hn);
    std::vector<double2> zH(p.zH.size());
    for (size_t q = 0; q < zH.size(); ++q) zH[q] = make_double2(p.zH[q].real(), p.zH[q].imag());
    d.zH = upload(d, zH);
  }
  d.vol_scale = d.fwd_scale;
  d.adj_scale_v = static_cast<double2 *>(dalloc(d, nf * sizeof(double2)));
  // adjoint injection coefficients [ns][node][2nf] (filled per adjoint call)
  // and the tables their synthesis reads
  {
    const int nn = (int)p.rn_c.size();
    d.at_coef = static_cast<double *>(dalloc(d, (size_t)p.ns * nn * 2 * nf * sizeof(double)));
    d.eadj = static_cast<double2 *>(dalloc(d, (size_t)p.ns * p.nr * p.ncomp * nf * sizeof(double2)));
    d.at_ptr = upload(d, p.at_ptr);
    d.at_row = upload(d, p.at_row);
    d.at_w = upload(d, p.at_w);
    std::vector<double2> fac(nf), fac_h(nf);
    for (int k = 0; k < nf; ++k) {
      const cplx f = std::sqrt(cplx(0.0, -p.omega[k] / (2.0 * p.omega0)));
      const cplx fh = std::exp(cplx(0.0, 1.0) * p.wprime[k] * (0.5 * p.dt));
      fac[k] = make_double2(f.real(), f.imag());
      fac_h[k] = make_double2(fh.real(), fh.imag());
    }
    d.adj_fac = upload(d, fac);
    d.adj_fac_h = upload(d, fac_h);
    std::vector<double> bmax(2 * nf, 0.0), nodefac(nn);
    if (p.have_basis)
      for (int r = 0; r < 2 * nf; ++r)
        for (int n = 0; n < p.nt; ++n)
          bmax[r] = std::max(bmax[r], std::fabs(p.basis[(size_t)r * p.nt + n]));
    for (int node = 0; node < nn; ++node)
      nodefac[node] = p.rn_c[node] >= 3 ? p.dt / kMu0 : p.ce[p.rn_c[node]][p.rn_idx[node]];
    d.adj_bmax = upload(d, bmax);
    d.adj_nodefac = upload(d, nodefac);
    d.adj_inc = static_cast<double *>(dalloc(d, (size_t)std::max(1, p.ns * nn) * sizeof(double)));
    d.adj_scale = static_cast<double *>(dalloc(d, sizeof(double)));
  }
  // per-cell factors sigma_h V / 4 and sigma_v V / 4 (zero for cells above
  // the resistivity cap)
  {
    std::vector<double> cf((size_t)p.nx * p.ny * p.nz), cv(cf.size());
    for (int k = 0; k < p.nz; ++k)
      for (int j = 0; j < p.ny; ++j)
        for (int i = 0; i < p.nx; ++i) {
          const size_t c = ((size_t)k * p.ny + j) * p.nx + i;
          const double V = p.ax[0].h[i] * p.ax[1].h[j] * p.ax[2].h[k];
          cf[c] = p.capped[c] ? 0.0 : p.sigma[c] * V * 0.25;
          cv[c] = p.capped_v[c] ? 0.0 : p.sigma_v[c] * V * 0.25;
        }
    d.cellfac = upload(d, cf);
    d.cellfac_v = upload(d, cv);
  }
  // order 4: the dual volume of an edge in metric lengths over the one the
  // cell factors assume (cell and dual widths), per axis: [axis][half n |
  // node n+1] at stride LA; the ratio of an edge is a product of three
  if (p.fd_order == 4) {
    const int LA = d.LA;
    std::vector<double> r((size_t)3 * 2 * LA, 1.0);
    for (int a = 0; a < 3; ++a) {
      const Axis &ax = p.ax[a];
      for (int i = 0; i < ax.n; ++i) r[(size_t)(2 * a) * LA + i] = ax.m[i] / ax.h[i];
      for (int i = 0; i <= ax.n; ++i) r[(size_t)(2 * a + 1) * LA + i] = ax.md[i] / ax.hd[i];
    }
    d.vratio = upload(d, r);
  }
  if (p.have_basis) {
    d.basis = upload(d, p.basis);
    // Q_k^n = (Omega_k / w'_k) * norm_k * z_k^{n+1}: the discrete-time
    // gradient factor, the forward normalisation and the twiddle
    std::vector<double2> Q((size_t)p.nt * nf);
    for (int k = 0; k < nf; ++k) {
      const cplx f = p.Omega[k] / p.wprime[k] * p.norm[k];
      for (int n = 0; n < p.nt; ++n) {
        const cplx v = f * p.zE[(size_t)n * nf + k];
        Q[(size_t)n * nf + k] = make_double2(v.real(), v.imag());
      }
    }
    d.Q = upload(d, Q);
  }
  d.model_version = p.model_version;
  d.basis_version = p.basis_version;
}

// ---------------------------------------------------------------------------
// workspace carving
// ---------------------------------------------------------------------------
struct WS {
  void *fields, *psi;   // two halves each
  double2 *racc;
  int *step;            // [2] step counters (last completed step)
  int *flushed;         // last sample already added by a flush
  unsigned *bar;        // persistent schedule: barrier counter and generation
  int *abort;           // persistent schedule: a barrier wait was abandoned
  int *bad;             // a non-finite value in the final fields or the gradient
  void *hist;
  double *gedge;
};

static size_t a256(size_t b) { return (b + 255) & ~size_t(255); }

static WS carve(const Plan &p, void *ws) {
  WS w;
  char *b = static_cast<char *>(ws);
  w.fields = b;
  b += a256(2 * (size_t)p.ns * 6 * p.field_elems() * p.tsize());
  w.psi = b;
  b += a256(2 * (size_t)p.ns * p.psi_elems_per_source() * p.tsize());
  w.racc = reinterpret_cast<double2 *>(b);
  b += a256((size_t)p.ns * p.rn_c.size() * p.nf() * 16);
  w.step = reinterpret_cast<int *>(b);
  w.flushed = w.step + 2;
  w.bar = reinterpret_cast<unsigned *>(w.step + 4);
  w.abort = w.step + 6;
  w.bad = w.step + 7;
  b += 256;
  w.hist = b;
  b += a256((size_t)p.ns * p.hist_elems_per_source() * p.tsize());
  w.gedge = reinterpret_cast<double *>(b);
  return w;
}

// ---------------------------------------------------------------------------
// one step = one launch (k_leap), two launches (H, E) or one fused launch
// ---------------------------------------------------------------------------
// Tiling: (bx x by) threads over x-y; tile b = (bz * nby + by) * nbx + bx.
// Rows of waves: 64 x nodes of one row.  Two kernels: each thread a vector of VX
// x nodes, one plane per tile row (bz = k).  Fused: one x node per thread, kz planes per tile (bz = chunk).
struct Tiling {
  int nbx, nby, nbz, nblocks, vx;
  int bx, by;   // threads of a tile along x and y
  size_t lds;   // dynamic LDS bytes per block (fused)
};

// Schedule 0 with one node per thread runs as rows of waves: the one-launch
// step k_leap at order 2, k_rows_h4 and k_rows_e4 at order 4.  It is left to
// the general kernels where 32-bit byte offsets do not reach (a source's
// fields, CPML memory or history slot of 4 GB and more) and where magnetic
// nodes lie on the high walls (the rows of those walls are skipped).
// The two general kernels on one node per thread, as a plan starts, are slower
// on every grid measured (us a step; order 2, FP32: 101x101x61 30.1 against
// 17.2, 200x200x100 with 8 sources 967 against 644, 800x800x60 950 against
// 642; FP64: 32x32x32 13.4 against 5.5, 128x128x96 90.5 against 63.4,
// 400x400x200 1395 against 1299; order 4, FP32, 101x101x61: 31.5 against
// 22.0).  Without the XCD remap, FP64 grids of more than 90,000 nodes a plane
// ran 2 to 8 % faster on them (400x400x200 1220 against 1320), but their
// 16-byte vector forms, a choice of the caller and the autotuner's there, are
// faster than either (1080).
static bool rows_fit(const Plan &p) {
  const uint64_t lim = (uint64_t)1 << 32;
  return !p.h_on_walls && 6 * (uint64_t)p.field_elems() * p.tsize() < lim &&
         (uint64_t)p.psi_elems_per_source() * p.tsize() < lim;
}
static bool wave_rows(const Plan &p) {
  return p.sched == 0 && p.vx == 1 && p.vxh == 1 && rows_fit(p);
}
static bool one_launch(const Plan &p) { return p.fd_order == 2 && wave_rows(p); }

static Tiling tiling(const Plan &p, bool h_update = false) {
  if (p.bx * p.by > 256) fail(FWD_ERR_INVALID_ARG, "block x * block y must be <= 256");
  Tiling t;
  t.bx = p.bx;
  t.by = p.by;
  if (wave_rows(p)) {
    // one wave a block: 64 nodes of a row (the nodes of the high walls are
    // skipped, see k_leap)
    t.vx = 1;
    t.bx = 64;
    t.by = 1;
    t.nbx = (p.nx + 63) / 64;
    t.nby = p.ny;
    t.nbz = p.nz;
    t.lds = 0;
  } else if (p.sched == 1) {
    t.vx = 1;
    t.nbx = (p.NX + p.bx - 1) / p.bx;
    t.nby = (p.NY + p.by - 1) / p.by;
    t.nbz = (p.nz + p.kz - 1) / p.kz;
    t.lds = 3 * ((size_t)(p.bx + 2) * (p.by + 2) + (size_t)(p.bx + 1) * (p.by + 1)) * p.tsize();
  } else {
    // the H update has its own vector width; the persistent schedule runs
    // one node per thread
    const int v = p.sched == 2 ? 1 : (h_update ? p.vxh : p.vx);
    t.vx = v == 1 ? 1 : (int)(16 / p.tsize());
    t.nbx = (p.NX + p.bx * t.vx - 1) / (p.bx * t.vx);
    t.nby = (p.NY + p.by - 1) / p.by;
    t.nbz = p.NZ;
    t.lds = 0;
  }
  t.nblocks = t.nbx * t.nby * t.nbz;
  return t;
}

// Per-thread entry tables of the E update.  An entry is an injection target
// (kind 0: component c of source s; ref = first coefficient row) or a
// receiver node (kind 1: component c; ref = node index), attached to the
// thread of the tiling that owns its edge (with the element of that
// thread's vector, or the plane within the fused chunk), so that the E
// update finds its own entries with two loads and no search.
static std::string lists_key(const Plan &p) {
  char key[128];
  snprintf(key, sizeof key, "%d/%d/%d/%d/%d/%d/%d/%llu", p.bx, p.by, p.vx, p.vxh, p.sched, p.kz,
           p.order, (unsigned long long)p.model_version);
  return key;
}

template <typename V>
static V *upload_list(Dev &d, const std::vector<V> &h) {
  void *ptr = nullptr;
  const size_t bytes = h.size() * sizeof(V);
  HIP_CHECK(hipMalloc(&ptr, bytes ? bytes : 16));
  d.list_bufs.push_back({ptr, bytes});
  if (bytes) HIP_CHECK(hipMemcpy(ptr, h.data(), bytes, hipMemcpyHostToDevice));
  return static_cast<V *>(ptr);
}

// Injections and receivers of rows of waves: a table of 64 lanes and six
// components for every row with receiver nodes (an adjoint run injects at the
// same nodes), and one of the three E components for every row and source
// with an edge of that source (forward runs; a table a row for all sources
// would grow with their square).  Also the rows and planes that the entries
// of either run span (ent_box); the rows' source tables are listed for the
// forward run's box alone, as no other row asks (18 MB of -1 on 400x400x200
// cells with 8 sources otherwise, at every new model).
static void build_rows(Plan &p, Dev &d) {
  const Tiling t = tiling(p);
  const int nn = (int)p.rn_c.size();
  const int64_t plane = (int64_t)p.NY * p.PX;
  for (int m = 0; m < 2; ++m) {
    int *box = d.ent_box[m];
    box[0] = p.NY;
    box[2] = p.NZ;
    box[1] = box[3] = -1;
  }
  struct Node {
    int bx, j, k, lane;
  };
  auto at = [&](int64_t idx) {
    const int k = (int)(idx / plane), j = (int)((idx % plane) / p.PX), i = (int)(idx % p.PX);
    if (i >= p.nx || j >= p.ny || k >= p.nz) fail(FWD_ERR_INVALID_ARG, "entry outside the grid");
    return Node{i >> 6, j, k, i & 63};
  };
  auto span = [&](int64_t idx, int run) {
    const Node q = at(idx);
    int *box = d.ent_box[run];
    box[0] = std::min(box[0], q.j);
    box[1] = std::max(box[1], q.j);
    box[2] = std::min(box[2], q.k);
    box[3] = std::max(box[3], q.k);
  };
  for (int node = 0; node < nn; ++node)
    for (int run : {0, 1}) span(p.rn_idx[node], run);
  for (const Target &tg : p.src_tg)
    if (tg.c < 3) span(tg.idx, 0);            // the others go into H before the step
  const int *box = d.ent_box[0];
  const int ejn = std::max(0, box[1] - box[0] + 1), ekn = std::max(0, box[3] - box[2] + 1);
  std::vector<int> tab(t.nblocks, -1), stab((size_t)ekn * ejn * t.nbx * p.ns, -1), rec, src;
  d.rec_mask = 0;
  for (int node = 0; node < nn; ++node) {
    const Node q = at(p.rn_idx[node]);
    int &r = tab[p.order ? (q.j * t.nbx + q.bx) * t.nbz + q.k : (q.k * t.nby + q.j) * t.nbx + q.bx];
    if (r < 0) {
      r = (int)(rec.size() / 384);
      rec.resize(rec.size() + 384, -1);
    }
    rec[((size_t)r * 6 + p.rn_c[node]) * 64 + q.lane] = node;
    d.rec_mask |= 1 << p.rn_c[node];
  }
  for (size_t e = 0; e < p.src_tg.size(); ++e) {
    const Target &tg = p.src_tg[e];
    if (tg.c >= 3) continue;
    const Node q = at(tg.idx);
    int &r = stab[(((size_t)(q.k - box[2]) * ejn + (q.j - box[0])) * t.nbx + q.bx) * p.ns + tg.s];
    if (r < 0) {
      r = (int)(src.size() / 192);
      src.resize(src.size() + 192, -1);
    }
    src[((size_t)r * 3 + tg.c) * 64 + q.lane] = (int)e;
  }
  d.row_tab = upload_list(d, tab);
  d.src_tab = upload_list(d, stab);
  d.row_rec = upload_list(d, rec);
  d.row_src = upload_list(d, src);
}

static void build_lists(Plan &p, Dev &d) {
  const std::string key = lists_key(p);
  if (d.list_key == key) return;
  free_lists(d);
  const bool rows = wave_rows(p);
  if (rows) build_rows(p, d);
  const int nn = (int)p.rn_c.size(), nf = p.nf();
  // the one-launch step has no H update, so no entries of one
  for (int mode = one_launch(p) ? 4 : rows ? 2 : 0; mode < 4; ++mode) {
    const Tiling t = tiling(p, mode >= 2);   // modes 2 and 3 live on the H update's grid
    const bool own_h = p.sched != 1;         // the H update adds magnetic sources
    const int slots = t.bx * t.by;
    struct E {
      int b, slot;
      int2 v;
    };
    std::vector<E> ents;
    auto place = [&](int c, int kind, int s, int64_t idx, int ref) {
      const int64_t plane = (int64_t)p.NY * p.PX;
      const int k = (int)(idx / plane), j = (int)((idx % plane) / p.PX), i = (int)(idx % p.PX);
      if (i > p.nx || j > p.ny || k > p.nz) fail(FWD_ERR_INVALID_ARG, "entry outside the grid");
      int bxi, byi, bzi, slot, sub;
      if (p.sched == 1) {
        if (k >= p.nz) return;   // no E update on the top plane: never used
        bzi = k / p.kz;
        sub = k % p.kz;
        bxi = i / p.bx;
        slot = (j % p.by) * p.bx + (i % p.bx);
      } else {
        const int tx = i / t.vx;
        sub = i % t.vx;
        bzi = k;
        bxi = tx / t.bx;
        slot = (j % t.by) * t.bx + (tx % t.bx);
      }
      byi = j / t.by;
      const int b = p.order ? (byi * t.nbx + bxi) * t.nbz + bzi : (bzi * t.nby + byi) * t.nbx + bxi;
      ents.push_back({b, slot, make_int2(c | (kind << 2) | (sub << 3) | (s << 9), ref)});
    };
    if (mode == 0) {
      for (size_t q = 0; q < p.src_tg.size(); ++q)
        if (p.src_tg[q].c < 3) place(p.src_tg[q].c, 0, p.src_tg[q].s, p.src_tg[q].idx, (int)q);
    } else if (mode == 3) {
      // forward magnetic sources M'^n, added by the H update; the fused
      // schedule uses k_hsrc instead
      if (own_h)
        for (size_t q = 0; q < p.src_tg.size(); ++q)
          if (p.src_tg[q].c >= 3)
            place(p.src_tg[q].c - 3, 0, p.src_tg[q].s, p.src_tg[q].idx, (int)q);
    } else if (mode == 1) {
      for (int s = 0; s < p.ns; ++s)
        for (int node = 0; node < nn; ++node)
          if (p.rn_c[node] < 3) place(p.rn_c[node], 0, s, p.rn_idx[node], (s * nn + node) * 2 * nf);
    } else if (own_h) {
      // magnetic adjoint sources M'^n, added by the H update (component c of
      // H = rn_c - 3); the fused schedule uses k_hinj instead
      for (int s = 0; s < p.ns; ++s)
        for (int node = 0; node < nn; ++node)
          if (p.rn_c[node] >= 3)
            place(p.rn_c[node] - 3, 0, s, p.rn_idx[node], (s * nn + node) * 2 * nf);
    }
    // H receiver nodes: recorded by the E update (entry c = 3; the node's
    // table gives the component), or by k_hrec under the fused schedule
    if (mode < 2)
      for (int node = 0; node < nn; ++node) {
        if (p.rn_c[node] < 3) place(p.rn_c[node], 1, 0, p.rn_idx[node], node);
        else if (p.sched != 1) place(3, 1, 0, p.rn_idx[node], node);
      }
    std::stable_sort(ents.begin(), ents.end(), [](const E &a, const E &b) {
      return a.b != b.b ? a.b < b.b : a.slot < b.slot;
    });
    std::vector<int> tab(t.nblocks, -1), off;
    std::vector<int2> ev;
    size_t e = 0;
    while (e < ents.size()) {
      const int b = ents[e].b;
      tab[b] = (int)off.size();
      const size_t base = off.size();
      off.resize(base + slots + 1, 0);
      size_t f = e;
      while (f < ents.size() && ents[f].b == b) ++f;
      // counts per slot, then prefix offsets into the global entry array
      std::vector<int> cnt(slots, 0);
      for (size_t g = e; g < f; ++g) cnt[ents[g].slot]++;
      int acc = (int)ev.size();
      for (int sl = 0; sl < slots; ++sl) {
        off[base + sl] = acc;
        acc += cnt[sl];
      }
      off[base + slots] = acc;
      for (size_t g = e; g < f; ++g) ev.push_back(ents[g].v);
      e = f;
    }
    d.tile_tab[mode] = upload_list(d, tab);
    d.tl_off[mode] = upload_list(d, off);
    d.tl_ent[mode] = upload_list(d, ev);
  }
  d.list_key = key;
}

// r: which step counter holds the last completed step (the launches read
// counter r and write counter r ^ 1)
// grid of a launch: tile counts, the block count (tiles * sources) and the
// dividers of the block decode (A.ns must be set)
template <typename T>
static void set_grid(StepArgs<T> &A, int nbx, int nby, int nbz) {
  A.nbx = nbx;
  A.nby = nby;
  A.nbz = nbz;
  const int64_t nb = (int64_t)nbx * nby * nbz * A.ns;
  if (nb >= ((int64_t)1 << 31)) fail(FWD_ERR_INVALID_ARG, "too many blocks for one launch");
  A.nblocks = (int)nb;
  A.dns = fdiv_make((uint32_t)A.ns);
  A.dnbx = fdiv_make((uint32_t)nbx);
  A.dnby = fdiv_make((uint32_t)nby);
  A.dnbz = fdiv_make((uint32_t)nbz);
}

template <typename T>
static StepArgs<T> make_args(Plan &p, Dev &d, const WS &w, void *vol, bool adj, int r = 0) {
  StepArgs<T> A{};
  A.nx = p.nx;
  A.ny = p.ny;
  A.nz = p.nz;
  A.npml = p.npml;
  A.PX = p.PX;
  A.NY = p.NY;
  A.NZ = p.NZ;
  A.ns = p.ns;
  A.F = p.field_elems();
  A.psi_src = p.psi_elems_per_source();
  A.fields = static_cast<T *>(w.fields);
  A.psi = static_cast<T *>(w.psi);
  A.ce = static_cast<const T *>(d.ce);
  A.axt = static_cast<const T *>(d.axt);
  A.LA = d.LA;
  A.fbuf = (int64_t)p.ns * 6 * A.F;
  A.pbuf = (int64_t)p.ns * A.psi_src;
  {
    const int64_t W = 2 * p.npml;
    A.plane = (int64_t)p.NY * p.PX;
    A.sX = (int64_t)p.NZ * p.NY * W;
    A.sY = (int64_t)p.NZ * W * p.PX;
    A.sZ = W * p.NY * p.PX;
    A.F6 = 6 * A.F;
    A.oY = 4 * A.sX;
    A.oZ = 4 * A.sX + 4 * A.sY;
  }
  A.dtmu = (T)(p.dt / kMu0);
  A.step = w.step + r;
  A.step_w = w.step + (r ^ 1);
  const Tiling t = tiling(p);
  set_grid(A, t.nbx, t.nby, t.nbz);
  A.xcd = p.xcd;
  A.kz = p.kz;
  A.order = p.order;
  A.lean = p.npml >= 1 && p.lean ? 1 : 0;
  A.kb = p.kb;
  A.dl = adj ? 0 : p.dec_log2;   // the adjoint's gradient product takes every sample
  A.nts = p.streaming(vol != nullptr) ? 1 : 0;
  A.dplane = fdiv_make((uint32_t)A.plane);
  A.dpx = fdiv_make((uint32_t)p.PX);
  A.nf = p.nf();
  A.zE = d.zE;
  A.vol = vol;
  A.Q = d.Q;
  A.gedge = adj ? w.gedge : nullptr;
  A.hist = static_cast<T *>(w.hist);
  A.hist_src = p.hist_elems_per_source();
  A.flushed = w.flushed;
  const int m = adj ? 1 : 0;   // tables built by build_lists before any launch or capture
  A.tile_tab = d.tile_tab[m];
  A.tl_off = d.tl_off[m];
  A.tl_ent = d.tl_ent[m];
  A.nt = p.nt;
  if (adj) {
    A.nrow = 2 * p.nf();
    A.coef = d.at_coef;
    A.Ftab = d.basis;
  } else {
    A.nrow = 1;
    A.coef = d.src_coef;
    A.Ftab = d.wavelet;
  }
  A.racc = w.racc;
  A.nn = (int)p.rn_c.size();
  A.rn_c = d.rn_c;
  A.zH = d.zH;
  A.dtmu64 = p.dt / kMu0;
  return A;
}

// start/stop events of one timed launch; hipExtLaunchKernel stamps them
// from the kernel's own dispatch, so the interval covers the kernel alone
// (no event-marker or dispatch latency around it)
struct KTime {
  hipEvent_t start, stop;
};

template <typename F, typename... Args>
static void go(F kernel, dim3 grid, dim3 block, size_t lds, hipStream_t st, const KTime *kt,
               Args... args) {
  if (kt) hipExtLaunchKernelGGL(kernel, grid, block, (std::uint32_t)lds, st, kt->start, kt->stop,
                                0u, args...);
  else hipLaunchKernelGGL(kernel, grid, block, lds, st, args...);
}

// E update (order 2 or 4); hist: the run keeps every sample for the block
// transform
template <typename T>
static void launch_e(const StepArgs<T> &A, int vx, bool hist, dim3 grid, dim3 block,
                     hipStream_t st, const KTime *kt = nullptr, bool o4 = false) {
  constexpr int VV = (int)(16 / sizeof(T));
  if (o4) {
    if (hist) go(k_update_e4<T, true>, grid, block, 0, st, kt, A);
    else go(k_update_e4<T, false>, grid, block, 0, st, kt, A);
  } else if (vx == 1) {
    if (A.nts) {
      if constexpr (std::is_same<T, float>::value) {
        if (hist) go(k_update_e_s<true>, grid, block, 0, st, kt, A);
        else go(k_update_e_s<false>, grid, block, 0, st, kt, A);
      } else {
        if (hist) go(k_update_e<T, true, 1, true>, grid, block, 0, st, kt, A);
        else go(k_update_e<T, false, 1, true>, grid, block, 0, st, kt, A);
      }
    } else {
      if (hist) go(k_update_e<T, true, 1, false>, grid, block, 0, st, kt, A);
      else go(k_update_e<T, false, 1, false>, grid, block, 0, st, kt, A);
    }
  } else {
    if (A.nts) {
      if (hist) go(k_update_e<T, true, VV, true>, grid, block, 0, st, kt, A);
      else go(k_update_e<T, false, VV, true>, grid, block, 0, st, kt, A);
    } else {
      if (hist) go(k_update_e<T, true, VV, false>, grid, block, 0, st, kt, A);
      else go(k_update_e<T, false, VV, false>, grid, block, 0, st, kt, A);
    }
  }
}

// the block transform: grid (nodes of the padded layout / 256, sources)
template <typename T, int KB, bool FLUSH>
static void launch_transform_kb(const StepArgs<T> &A, int acc, bool adj, hipStream_t st,
                                const KTime *kt) {
  const dim3 grid((unsigned)((A.F + 255) / 256), A.ns, 3), block(256);
  const size_t lds = (size_t)A.nf * KB * sizeof(double2);
#define FWD_TR(ACCV) \
  do { \
    if (adj) go(k_transform<T, ACCV, true, KB, FLUSH>, grid, block, lds, st, kt, A); \
    else go(k_transform<T, ACCV, false, KB, FLUSH>, grid, block, lds, st, kt, A); \
  } while (0)
  switch (acc) {
    case FWD_ACC_F64: FWD_TR(ACC_F64); break;
    case FWD_ACC_KAHAN: FWD_TR(ACC_KAHAN); break;
    default: FWD_TR(ACC_F32);
  }
#undef FWD_TR
}
template <typename T, bool FLUSH>
static void launch_transform(const StepArgs<T> &A, int kb, int acc, bool adj, hipStream_t st,
                             const KTime *kt = nullptr) {
  switch (kb) {
    case 1: launch_transform_kb<T, 1, FLUSH>(A, acc, adj, st, kt); break;
    case 2: launch_transform_kb<T, 2, FLUSH>(A, acc, adj, st, kt); break;
    case 4: launch_transform_kb<T, 4, FLUSH>(A, acc, adj, st, kt); break;
    case 8: launch_transform_kb<T, 8, FLUSH>(A, acc, adj, st, kt); break;
    case 16: launch_transform_kb<T, 16, FLUSH>(A, acc, adj, st, kt); break;
    default: launch_transform_kb<T, 32, FLUSH>(A, acc, adj, st, kt);
  }
}

template <typename T>
static void launch_step(const StepArgs<T> &A, bool hist, dim3 grid, dim3 block, size_t lds,
                        hipStream_t st, const KTime *kt = nullptr) {
  if (hist) go(k_step<T, true>, grid, block, lds, st, kt, A);
  else go(k_step<T, false>, grid, block, lds, st, kt, A);
}

// n: the step by the host's count, which places the sample in its transform
// block and nothing else.  keep: E^{n+1} of every source also goes there,
// [ns][3][F] (runs without a volume transform)
template <typename T>
static LeapArgs<T> leap_args(Plan &p, Dev &d, const StepArgs<T> &A, bool vol, bool adj, int n,
                             T *keep = nullptr) {
  LeapArgs<T> L{};
  L.f0 = A.fields;
  L.f1 = A.fields + A.fbuf;
  L.p0 = A.psi;
  L.p1 = A.psi + A.pbuf;
  L.ce = A.ce;
  L.axt = A.axt;
  L.axr = static_cast<const AxRow<T> *>(d.axr);
  L.step = A.step;
  L.step_w = A.step_w;
  L.F6 = A.F6;
  L.psi_src = A.psi_src;
  L.hist_src = A.hist_src;
  const size_t sz = sizeof(T);
  L.PXb = (uint32_t)(A.PX * sz);
  L.PLb = (uint32_t)(A.plane * sz);
  L.Fb = (uint32_t)(A.F * sz);
  L.LAb = (uint32_t)(A.LA * sz);
  L.sXb = (uint32_t)(A.sX * sz);
  L.sYb = (uint32_t)(A.sY * sz);
  L.sZb = (uint32_t)(A.sZ * sz);
  L.oYb = (uint32_t)(A.oY * sz);
  L.oZb = (uint32_t)(A.oZ * sz);
  L.nx = A.nx;
  L.ny = A.ny;
  L.nz = A.nz;
  L.npml = A.npml;
  L.LA = A.LA;
  L.NY = A.NY;
  L.dtmu = A.dtmu;
  L.order = A.order;
  L.ns = A.ns;
  L.runs = A.xcd ? (uint32_t)A.nblocks >> (3 + XCD_RUN_LOG2) << (3 + XCD_RUN_LOG2) : 0;
  L.dns = A.dns;
  L.d1 = A.order ? A.dnbz : A.dnbx;
  L.d2 = A.order ? A.dnbx : A.dnby;
  // differences reach one node past the layer's edge rows, and two past a
  // wall at order 4
  const int np = p.fd_order == 4 ? std::max(A.npml, 2) : A.npml;
  auto window = [&](int n, int width, uint32_t &first, uint32_t &count) {
    first = (uint32_t)np + 1;
    count = A.lean ? (uint32_t)std::max(0, n - 2 * np - width) : 0;
  };
  window(A.nx, 64, L.xs, L.xn);
  window(A.ny, 1, L.ys, L.yn);
  window(A.nz, 1, L.zs, L.zn);
  L.row_tab = d.row_tab;
  L.src_tab = adj ? nullptr : d.src_tab;
  L.row_rec = d.row_rec;
  L.row_src = d.row_src;
  L.rec_mask = d.rec_mask;
  L.adj = adj ? 1 : 0;
  const int *box = d.ent_box[adj ? 1 : 0];
  L.ej = (uint32_t)box[0];
  L.ejn = (uint32_t)std::max(0, box[1] - box[0] + 1);
  L.ek = (uint32_t)box[2];
  L.ekn = (uint32_t)std::max(0, box[3] - box[2] + 1);
  L.nbx = (uint32_t)A.nbx;
  const int D = adj ? 1 : p.dec, m = n + 1, r = m / D & (p.kb - 1);
  const bool hist = vol && m % D == 0 && r != 0;
  if (hist) L.hist = A.hist + (int64_t)(r - 1) * 3 * A.F;
  if (keep) {
    L.hist = keep;
    L.hist_src = 3 * A.F;
  }
  return L;
}

template <typename T>
static void launch_leap(Plan &p, Dev &d, const StepArgs<T> &A, bool vol, bool adj, int n,
                        hipStream_t st, const KTime *kt, T *keep) {
  const LeapArgs<T> L = leap_args<T>(p, d, A, vol, adj, n, keep);
  const bool hist = L.hist != nullptr;
  const dim3 grid(A.nblocks), block(64);
  if (A.nts) {
    if (hist) go(k_leap<T, true, true>, grid, block, 0, st, kt, L, A);
    else go(k_leap<T, false, true>, grid, block, 0, st, kt, L, A);
  } else {
    if (hist) go(k_leap<T, true, false>, grid, block, 0, st, kt, L, A);
    else go(k_leap<T, false, false>, grid, block, 0, st, kt, L, A);
  }
}

template <typename T>
static void launch_h(const StepArgs<T> &A, int vx, dim3 grid, dim3 block, hipStream_t st,
                     const KTime *kt = nullptr, bool o4 = false, bool inj = false) {
  constexpr int VV = (int)(16 / sizeof(T));
  if (o4) {
    if (inj) go(k_update_h4<T, true>, grid, block, 0, st, kt, A);
    else go(k_update_h4<T, false>, grid, block, 0, st, kt, A);
    return;
  }
#define FWD_H(VXV, INJV)                                                   \
  do {                                                                     \
    if (A.nts) go(k_update_h<T, VXV, INJV, true>, grid, block, 0, st, kt, A); \
    else go(k_update_h<T, VXV, INJV, false>, grid, block, 0, st, kt, A);   \
  } while (0)
  if (inj) {
    if (vx == 1) FWD_H(1, true);
    else FWD_H(VV, true);
  } else {
    if (vx == 1) FWD_H(1, false);
    else FWD_H(VV, false);
  }
#undef FWD_H
}

// enqueue step n (one launch; H update, E update; or the fused step), followed by the
// block transform when sample n+1 closes a transform block.  If ev !=
// nullptr, ev[0..1] time the H kernel, ev[2..3] the E kernel (one launch or
// fused: the one kernel in ev[2..3], ev[0..1] recorded back to back) and ev[4..5] the block
// transform (recorded back to back when there is none); *closed says which.
// keep: see leap_args (rows of waves only).
template <typename T>
static void enqueue_step(Plan &p, Dev &d, const WS &w, void *vol, bool adj, hipStream_t st,
                         hipEvent_t *ev, int r, int n, bool *closed = nullptr, T *keep = nullptr) {
  StepArgs<T> A = make_args<T>(p, d, w, vol, adj, r);
  const dim3 block(p.bx, p.by), grid(A.nblocks);
  const KTime th_ev = ev ? KTime{ev[0], ev[1]} : KTime{}, te_ev = ev ? KTime{ev[2], ev[3]} : KTime{};
  const KTime *kh = ev ? &th_ev : nullptr, *ke = ev ? &te_ev : nullptr;
  const bool one = one_launch(p), hpre = one || p.sched == 1;
  // magnetic nodes of the one-launch and fused steps: their sources go into H
  // before the launch (every wave that recomputes a node then reads it); the
  // fused step's H transform follows it (the E update does not touch H)
  const dim3 hgrid((p.ns * d.nh + 63) / 64), hblock(64);
  if (d.nh > 0 && adj && hpre)
    hipLaunchKernelGGL((k_hinj<T>), hgrid, hblock, 0, st, A, d.hn, d.nh, d.rn_c, d.rn_idx,
                       p.dt / kMu0);
  if (!adj && p.src_kind == 1 && hpre)
    hipLaunchKernelGGL((k_hsrc<T>), dim3((d.ntg + 63) / 64), dim3(64), 0, st, A, d.src_s, d.src_c,
                       d.src_idx, d.ntg, p.dt / kMu0);
  if (one) {
    if (ev) {
      (void)hipEventRecord(ev[0], st);
      (void)hipEventRecord(ev[1], st);
    }
    launch_leap<T>(p, d, A, vol != nullptr, adj, n, st, ke, keep);
  } else if (p.sched == 1) {
    if (ev) {
      (void)hipEventRecord(ev[0], st);
      (void)hipEventRecord(ev[1], st);
    }
    launch_step<T>(A, vol != nullptr, grid, block, tiling(p).lds, st, ke);
    if (d.nh > 0)
      hipLaunchKernelGGL((k_hrec<T>), hgrid, hblock, 0, st, A, d.hn, d.nh, d.rn_c, d.rn_idx, d.zH);
  } else {
    // the E update records the H receiver nodes itself; the H update adds
    // the magnetic sources (adjoint runs with magnetic data, forward runs of
    // magnetic dipoles) from its own entry table
    StepArgs<T> Ah = A;
    const Tiling th = tiling(p, true);
    set_grid(Ah, th.nbx, th.nby, th.nbz);
    const bool hinj = adj ? d.nh > 0 : p.src_kind == 1;
    const int hm = adj ? 2 : 3;
    Ah.tile_tab = hinj ? d.tile_tab[hm] : nullptr;
    Ah.tl_off = hinj ? d.tl_off[hm] : nullptr;
    Ah.tl_ent = hinj ? d.tl_ent[hm] : nullptr;
    const bool o4 = p.fd_order == 4;
    if (o4 && wave_rows(p)) {
      const LeapArgs<T> L = leap_args<T>(p, d, A, vol != nullptr, adj, n, keep);
      const dim3 row(64);
      if (hinj) go(k_rows_h4<T, true>, grid, row, 0, st, kh, L, Ah);
      else go(k_rows_h4<T, false>, grid, row, 0, st, kh, L, Ah);
      if (L.hist) go(k_rows_e4<T, true>, grid, row, 0, st, ke, L, A);
      else go(k_rows_e4<T, false>, grid, row, 0, st, ke, L, A);
    } else {
      launch_h<T>(Ah, p.vxh, dim3(Ah.nblocks), block, st, kh, o4, hinj);
      // with a decimated volume transform only the steps whose sample enters
      // it keep history
      const int D = adj ? 1 : p.dec;
      launch_e<T>(A, p.vx, vol != nullptr && (n + 1) % D == 0, grid, block, st, ke, o4);
    }
  }
  // the block transform after the step whose sample closes a block; it reads
  // the counter the E update has just written (step n)
  const bool close = vol != nullptr && (n + 1) % (p.kb * (adj ? 1 : p.dec)) == 0;
  if (closed) *closed = close;
  if (close) {
    StepArgs<T> At = A;
    At.step = A.step_w;
    const KTime tt_ev = ev ? KTime{ev[4], ev[5]} : KTime{};
    launch_transform<T, false>(At, p.kb, p.acc, adj, st, ev ? &tt_ev : nullptr);
  } else if (ev) {
    (void)hipEventRecord(ev[4], st);
    (void)hipEventRecord(ev[5], st);
  }
}

// Add the samples of an incomplete last transform block (the host's step
// count says whether there is one); the device reads the newest sample's
// index from the equalised counters.
template <typename T>
static void flush_t(Plan &p, Dev &d, const WS &w, void *vol, bool adj, hipStream_t st) {
  // decimated samples taken so far (every step's sample when D = 1)
  const int taken = p.host_step / (adj ? 1 : p.dec);
  // no sample, so no block transform has written the volume buffer yet
  if (!adj && vol && taken == 0) zero_bytes(vol, p.volume_bytes(), st);
  if (p.kb == 1 || !vol || taken % p.kb == 0) return;
  build_lists(p, d);
  hipLaunchKernelGGL(k_equalize, dim3(1), dim3(64), 0, st, w.step);
  StepArgs<T> A = make_args<T>(p, d, w, vol, adj);
  launch_transform<T, true>(A, p.kb, p.acc, adj, st);
  hipLaunchKernelGGL(k_set_flushed, dim3(1), dim3(64), 0, st, w.flushed, (const int *)w.step);
  HIP_CHECK(hipGetLastError());
}

static void flush_any(Plan &p, Dev &d, const WS &w, void *vol, bool adj, hipStream_t st) {
  if (p.dtype == FWD_F64)
    flush_t<double>(p, d, w, vol, adj, st);
  else
    flush_t<float>(p, d, w, vol, adj, st);
}

// The persistent schedule: cooperative launches of up to 4096 steps each,
// the grid sized from the occupancy of the instantiation (at most one block
// per tile of the largest phase).
template <typename T, bool HIST, int ACC, bool ADJ, int KB, bool INJ>
static void launch_persist(const StepArgs<T> &A, const StepArgs<T> &Ah, int nsteps, const Bar &B,
                           dim3 block, size_t lds, hipStream_t st, int cap) {
  const void *fn = reinterpret_cast<const void *>(&k_persist<T, HIST, ACC, ADJ, KB, INJ>);
  int dev = 0, per_cu = 0, cus = 0;
  HIP_CHECK(hipGetDevice(&dev));
  HIP_CHECK(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
  HIP_CHECK(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, (int)(block.x * block.y), lds));
  if (per_cu < 1) fail(FWD_ERR_UNSUPPORTED, "persistent schedule: no block fits on a compute unit");
  if (cap > 0) per_cu = std::min(per_cu, cap);
  const int64_t tiles = std::max<int64_t>(A.nblocks, Ah.nblocks);
  const unsigned grid = (unsigned)std::min<int64_t>((int64_t)per_cu * cus, tiles);
  StepArgs<T> a = A, ah = Ah;
  Bar b = B;
  for (int done = 0; done < nsteps;) {
    int m = std::min(4096, nsteps - done);
    void *args[] = {&a, &ah, &m, &b};
    HIP_CHECK(hipLaunchCooperativeKernel(fn, dim3(grid), block, args, (unsigned)lds, st));
    done += m;
  }
}

template <typename T, bool HIST, int ACC, bool ADJ, bool INJ>
static void launch_persist_kb(const StepArgs<T> &A, const StepArgs<T> &Ah, int nsteps,
                              const Bar &B, dim3 block, size_t lds, hipStream_t st, int kb,
                              int cap) {
  if (kb == 8) launch_persist<T, HIST, ACC, ADJ, 8, INJ>(A, Ah, nsteps, B, block, lds, st, cap);
  else if (kb == 16) launch_persist<T, HIST, ACC, ADJ, 16, INJ>(A, Ah, nsteps, B, block, lds, st, cap);
  else fail(FWD_ERR_UNSUPPORTED, "persistent schedule: transform block 8 or 16");
}

template <typename T>
static void run_persistent(Plan &p, Dev &d, const WS &w, void *vol, bool adj, int nsteps,
                           hipStream_t st) {
  if (nsteps <= 0) return;
  if (p.fd_order != 2) fail(FWD_ERR_UNSUPPORTED, "persistent schedule: order 2 only");
  StepArgs<T> A = make_args<T>(p, d, w, vol, adj, 0);
  StepArgs<T> Ah = A;
  const Tiling th = tiling(p, true);
  set_grid(Ah, th.nbx, th.nby, th.nbz);
  const bool inj = adj ? d.nh > 0 : p.src_kind == 1;
  const int hm = adj ? 2 : 3;
  Ah.tile_tab = inj ? d.tile_tab[hm] : nullptr;
  Ah.tl_off = inj ? d.tl_off[hm] : nullptr;
  Ah.tl_ent = inj ? d.tl_ent[hm] : nullptr;
  A.xcd = Ah.xcd = 0;                      // virtual blocks: no dispatch-order remap
  int dev = 0, khz = 0;
  HIP_CHECK(hipGetDevice(&dev));
  HIP_CHECK(hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev));
  const Bar B{w.bar, w.bar + 1, w.abort, (uint64_t)(p.barrier_us * (double)khz / 1000.0),
              p.barrier_sleep};
  const int cap = p.persist_blocks;
  const dim3 block(p.bx, p.by);
  const bool hist = vol != nullptr;
  const size_t lds = hist ? (size_t)p.nf() * p.kb * sizeof(double2) : 0;
  if (!hist) {
    if (inj) launch_persist<T, false, ACC_F64, false, 8, true>(A, Ah, nsteps, B, block, lds, st, cap);
    else launch_persist<T, false, ACC_F64, false, 8, false>(A, Ah, nsteps, B, block, lds, st, cap);
  } else {
#define FWD_PERSIST(ACCV)                                                                   \
  do {                                                                                      \
    if (!adj && inj) launch_persist_kb<T, true, ACCV, false, true>(A, Ah, nsteps, B, block, lds, st, p.kb, cap); \
    else if (!adj) launch_persist_kb<T, true, ACCV, false, false>(A, Ah, nsteps, B, block, lds, st, p.kb, cap); \
    else if (!inj) launch_persist_kb<T, true, ACCV, true, false>(A, Ah, nsteps, B, block, lds, st, p.kb, cap); \
    else launch_persist_kb<T, true, ACCV, true, true>(A, Ah, nsteps, B, block, lds, st, p.kb, cap); \
  } while (0)
    switch (p.acc) {
      case FWD_ACC_F64: FWD_PERSIST(ACC_F64); break;
      case FWD_ACC_KAHAN: FWD_PERSIST(ACC_KAHAN); break;
      default: FWD_PERSIST(ACC_F32);
    }
#undef FWD_PERSIST
  }
  p.host_step += nsteps;
}

// A persistent run abandoned at a barrier (its wait exceeded the limit) is an
// error of the call that ran it.
static void check_abort(Plan &p, const WS &w, hipStream_t st) {
  if (p.sched != 2) return;
  int bad = 0;
  HIP_CHECK(hipMemcpyAsync(&bad, w.abort, sizeof bad, hipMemcpyDeviceToHost, st));
  HIP_CHECK(hipStreamSynchronize(st));
  if (bad)
    fail(FWD_ERR_HIP, "persistent schedule: a grid barrier wait exceeded " +
                          std::to_string(p.barrier_us) + " us; the run was abandoned");
}

// Run nsteps steps from the current position.  The device counters hold the
// step index for the kernels; the host keeps the same count (p.host_step)
// to know which steps close a transform block.
// plain: every step launched eagerly, no timing (no graph or event is
// created: the path of the entry point that allocates nothing)
template <typename T>
static void run_steps_t(Plan &p, Dev &d, const WS &w, void *vol, bool adj, int nsteps,
                        hipStream_t st, bool plain = false) {
  build_lists(p, d);
  // both counters hold the last completed step; the steps then alternate
  // (r = counter read by the next step)
  const int D = adj ? 1 : p.dec;
  if (D > 1 && vol && p.sched != 0)
    fail(FWD_ERR_UNSUPPORTED, "a decimated volume transform runs with schedule 0");
  hipLaunchKernelGGL(k_equalize, dim3(1), dim3(64), 0, st, w.step);
  if (p.sched == 2) {
    run_persistent<T>(p, d, w, vol, adj, nsteps, st);
    return;
  }
  int r = 0;
  // graphs hold an even number of steps (they start and end at r = 0) and a
  // whole number of transform blocks (every replay starts at the same phase);
  // a block of D-decimated samples spans kb * D steps
  const int unit = std::max(2, p.kb * D);
  const int Kg = p.graph_steps & ~1;
  const int K = plain || Kg < 2 ? 0 : std::max(unit, Kg / unit * unit);
  const int sample = plain ? 0 : d.sample_every;
  // eager launches of m steps, each bracketed by events if asked
  auto eager = [&](int m, bool timed) {
    for (int t = 0; t < m; ++t) {
      hipEvent_t *ev = nullptr;
      if (timed) {
        const size_t need = (size_t)(d.kstat_n + 1) * 6;
        while (d.ev.size() < need) {
          hipEvent_t e;
          HIP_CHECK(hipEventCreate(&e));
          d.ev.push_back(e);
        }
        ev = &d.ev[(size_t)d.kstat_n * 6];
      }
      bool closed = false;
      enqueue_step<T>(p, d, w, vol, adj, st, ev, r, p.host_step, &closed);
      if (timed) {
        d.kstat_closed.resize((size_t)d.kstat_n + 1);
        d.kstat_closed[d.kstat_n] = (closed ? 1 : 0) | (one_launch(p) || p.sched == 1 ? 2 : 0);
        d.kstat_n++;
      }
      p.host_step++;
      r ^= 1;
    }
    HIP_CHECK(hipGetLastError());
  };
  if (K < 2 || nsteps < K) {
    for (int t = 0; t < nsteps; ++t) eager(1, sample > 0 && t % sample == 0);
    return;
  }
  // graph of K steps, captured on a private stream and replayed on st
  const int phase = p.host_step % (p.kb * D);
  char key[256];
  snprintf(key, sizeof key, "%p/%p/%d/%d/%d/%d/%d/%d/%d/%d/%d/%d/%d/%d/%d/%d/%llu/%llu", w.fields,
           vol, (int)adj, K, phase, p.bx, p.by, p.xcd, p.kb * 64 + D, p.vx, p.vxh, p.sched, p.kz, p.order,
           p.lean, p.streaming(vol != nullptr) ? 1 : 0, (unsigned long long)p.model_version,
           (unsigned long long)p.basis_version);
  if (!d.exec || d.exec_key != key) {
    if (d.exec) {
      HIP_CHECK(hipGraphExecDestroy(d.exec));
      d.exec = nullptr;
    }
    hipGraph_t g = nullptr;
    HIP_CHECK(hipStreamBeginCapture(d.cap, hipStreamCaptureModeRelaxed));
    for (int t = 0; t < K; ++t)
      enqueue_step<T>(p, d, w, vol, adj, d.cap, nullptr, t & 1, p.host_step + t);
    const hipError_t le = hipGetLastError();
    const hipError_t ce = hipStreamEndCapture(d.cap, &g);   // always end the capture
    if (le != hipSuccess || ce != hipSuccess) {
      if (g) (void)hipGraphDestroy(g);
      fail(FWD_ERR_HIP, std::string("graph capture failed: ") +
                            hipGetErrorString(le != hipSuccess ? le : ce));
    }
    HIP_CHECK(hipGraphInstantiate(&d.exec, g, nullptr, nullptr, 0));
    HIP_CHECK(hipGraphDestroy(g));
    d.exec_key = key;
  }
  // with sampling on, one chunk in every max(1, sample/K) runs eagerly and
  // times each of its steps (all phases of the transform block); all others
  // replay the graph
  const int every = sample > 0 ? std::max(1, sample / K) : 0;
  int done = 0, chunk = 0;
  while (nsteps - done >= K) {
    if (every && chunk % every == 0) {
      eager(K, true);
    } else {
      HIP_CHECK(hipGraphLaunch(d.exec, st));
      p.host_step += K;
    }
    done += K;
    ++chunk;
  }
  eager(nsteps - done, false);
}

static void run_steps_any(Plan &p, Dev &d, const WS &w, void *vol, bool adj, int nsteps,
                          hipStream_t st, bool plain = false) {
  if (p.dtype == FWD_F64)
    run_steps_t<double>(p, d, w, vol, adj, nsteps, st, plain);
  else
    run_steps_t<float>(p, d, w, vol, adj, nsteps, st, plain);
}

// averages over the sampled steps: H update, E update (every sampled step),
// block transform (the sampled steps that closed a block)
static void collect_kernel_stats(Dev &d) {
  double tot[3] = {0, 0, 0};
  int ntr = 0;
  for (int s = 0; s < d.kstat_n; ++s) {
    hipEvent_t *ev = &d.ev[(size_t)s * 6];
    for (int k = 0; k < 3; ++k) {
      if (k == 2 && !(d.kstat_closed[s] & 1)) continue;
      if (k == 0 && (d.kstat_closed[s] & 2)) continue;   // one launch: no H update of its own
      float ms = 0;
      HIP_CHECK(hipEventElapsedTime(&ms, ev[2 * k], ev[2 * k + 1]));
      tot[k] += ms;
    }
    ntr += d.kstat_closed[s] & 1;
  }
  for (int k = 0; k < 2; ++k) d.kstat_ms[k] = d.kstat_n ? tot[k] / d.kstat_n : 0.0;
  d.kstat_ms[2] = ntr ? tot[2] / ntr : 0.0;
  d.kstat_ntr = ntr;
}

// A run starts from zero fields, CPML memory, receiver sums and counters
// (and, in adjoint runs, zero gradient accumulators).  The transform-block
// history is not cleared: every slot a block transform reads was written
// earlier in the same run (slots of samples past the run are masked by a
// select), and on the large grids it is the largest part of the workspace.
// Neither is the volume buffer: the run's first block transform writes all
// of it (and a run that ends before its first sample clears it at the
// flush).
static void zero_state(Plan &p, const WS &w, void *ws, int mode, hipStream_t st) {
  p.host_step = 0;
  p.host_ws = ws;
  char *b = static_cast<char *>(ws);
  zero_bytes(b, p.core_state_bytes(), st);
  zero_bytes(b + p.state_bytes(), p.workspace_bytes(mode) - p.state_bytes(), st);
  hipLaunchKernelGGL(k_set_int, dim3(1), dim3(64), 0, st, w.step, -1);
  hipLaunchKernelGGL(k_set_int, dim3(1), dim3(64), 0, st, w.step + 1, -1);
  HIP_CHECK(hipGetLastError());
}

static void check_sizes(Plan &p, size_t ws_bytes, int mode, void *vol, size_t vol_bytes) {
  if (ws_bytes < p.workspace_bytes(mode)) fail(FWD_ERR_INVALID_ARG, "workspace too small");
  if (vol && vol_bytes < p.volume_bytes()) fail(FWD_ERR_INVALID_ARG, "volume buffer too small");
}

// Sets *flag when any of n values at v (16-byte aligned) is Inf or NaN:
// 16-byte loads, then the last n % W values one by one.
template <typename T>
__global__ void k_nonfinite_v(const T *v, size_t n, int *flag) {
  using V = Vec<T, 16 / sizeof(T)>;
  constexpr int W = 16 / sizeof(T);
  const size_t nv = n / W, stride = (size_t)gridDim.x * blockDim.x;
  const size_t t0 = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  bool bad = false;
  for (size_t i = t0; i < nv; i += stride) {
    const V x = *reinterpret_cast<const V *>(v + i * W);
#pragma unroll
    for (int e = 0; e < W; ++e) bad |= !isfinite(x.v[e]);
  }
  if (t0 < n - nv * W) bad |= !isfinite(v[nv * W + t0]);
  if (bad) flag[0] = 1;
}

template <typename T>
static void flag_nonfinite(const T *v, size_t n, int *flag, hipStream_t st) {
  constexpr int W = 16 / sizeof(T);
  const size_t blocks = std::min<size_t>((n / W + 255) / 256 + 1, 4096);
  if (n == 0) return;
  hipLaunchKernelGGL((k_nonfinite_v<T>), dim3((unsigned)blocks), dim3(256), 0, st, v, n, flag);
}

// The fields of the last completed step (the half step n wrote, n = host
// step count - 1) to the workspace's flag: a blow-up anywhere in the grid
// (inside a CPML layer, far from every receiver) shows up there.
static void flag_final_fields(Plan &p, const WS &w, hipStream_t st) {
  const size_t half = (size_t)p.ns * 6 * p.field_elems();
  const int h = p.host_step & 1;
  if (p.dtype == FWD_F64)
    flag_nonfinite(static_cast<const double *>(w.fields) + h * half, half, w.bad, st);
  else
    flag_nonfinite(static_cast<const float *>(w.fields) + h * half, half, w.bad, st);
}

// Receiver output (host copy) and the device flag, one synchronisation.
static void check_finite(const double2 *dptr, size_t n, const int *flag_dev, hipStream_t st) {
  std::vector<double2> h(n);
  int bad = 0;
  HIP_CHECK(hipMemcpyAsync(h.data(), dptr, n * sizeof(double2), hipMemcpyDeviceToHost, st));
  if (flag_dev) HIP_CHECK(hipMemcpyAsync(&bad, flag_dev, sizeof bad, hipMemcpyDeviceToHost, st));
  HIP_CHECK(hipStreamSynchronize(st));
  for (auto &v : h)
    if (!std::isfinite(v.x) || !std::isfinite(v.y)) bad = 1;
  if (bad) fail(FWD_ERR_NONFINITE, "non-finite field: unstable run (dt above the CFL bound?)");
}

// The host's step count from a workspace's counters (last completed step: the
// larger of the two).  Waits for the stream.
static void read_host_step(Plan &p, const void *ws, hipStream_t st) {
  int cnt[2] = {0, 0};
  const WS w = carve(p, const_cast<void *>(ws));
  HIP_CHECK(hipMemcpyAsync(cnt, w.step, sizeof cnt, hipMemcpyDeviceToHost, st));
  HIP_CHECK(hipStreamSynchronize(st));
  p.host_step = std::max(cnt[0], cnt[1]) + 1;
  p.host_ws = ws;
}

// The host's count decides which steps of a run with a volume close a
// transform block: where it was taken on another workspace (a plan may step
// several in turn) it is read again.  Steps without a volume need no count, so
// they wait for nothing and leave it without a workspace.  A stream that is
// being captured cannot be waited for; there the count stands.
static void follow_workspace(Plan &p, const void *ws, const void *vol, hipStream_t st) {
  if (ws == p.host_ws) return;
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  if (vol) HIP_CHECK(hipStreamIsCapturing(st, &cs));
  if (vol && cs == hipStreamCaptureStatusNone) read_host_step(p, ws, st);
  else p.host_ws = nullptr;
}

// ---------------------------------------------------------------------------
// entry points used by the C ABI
// ---------------------------------------------------------------------------
void dev_run_begin(Plan &p, void *ws, size_t ws_bytes, void *vol, size_t vol_bytes, void *stream) {
  hipStream_t st = static_cast<hipStream_t>(stream);
  check_sizes(p, ws_bytes, FWD_MODE_FORWARD, vol, vol_bytes);
  ensure_tables(p, st);
  zero_state(p, carve(p, ws), ws, FWD_MODE_FORWARD, st);
}

void dev_run_steps(Plan &p, void *ws, void *vol, int nsteps, void *stream) {
  hipStream_t st = static_cast<hipStream_t>(stream);
  ensure_tables(p, st);
  if (nsteps < 0 || nsteps > p.nt) fail(FWD_ERR_INVALID_ARG, "nsteps outside [0, nt]");
  Dev &d = D(p);
  follow_workspace(p, ws, vol, st);
  run_steps_any(p, d, carve(p, ws), vol, false, nsteps, st);
  check_abort(p, carve(p, ws), st);
}

void dev_run_receivers(Plan &p, void *ws, double *E_rec, void *stream) {
  hipStream_t st = static_cast<hipStream_t>(stream);
  ensure_tables(p, st);
  Dev &d = D(p);
  WS w = carve(p, ws);
  const int nrows = p.nr * p.ncomp, nn = (int)p.rn_c.size(), n = p.ns * nrows * p.nf();
  hipLaunchKernelGGL(k_rec_out, dim3((n + 127) / 128), dim3(128), 0, st, p.ns, nrows, nn, p.nf(),
                     d.ri_ptr, d.ri_node, d.ri_w, w.racc, d.fwd_scale, d.fwd_scale_h, d.rcomp,
                     p.ncomp, reinterpret_cast<double2 *>(E_rec));
  HIP_CHECK(hipGetLastError());
}

void dev_run_flush(Plan &p, void *ws, void *vol, void *stream) {
  hipStream_t st = static_cast<hipStream_t>(stream);
  ensure_tables(p, st);
  follow_workspace(p, ws, vol, st);
  flush_any(p, D(p), carve(p, ws), vol, false, st);
}

void dev_forward(Plan &p, void *ws, size_t ws_bytes, void *vol, size_t vol_bytes, double *E_rec,
                 void *stream) {
  hipStream_t st = static_cast<hipStream_t>(stream);
  dev_run_begin(p, ws, ws_bytes, vol, vol_bytes, stream);
  Dev &d = D(p);
  d.kstat_n = 0;
  hipEvent_t e0, e1;
  HIP_CHECK(hipEventCreate(&e0));
  HIP_CHECK(hipEventCreate(&e1));
  HIP_CHECK(hipEventRecord(e0, st));
  run_steps_any(p, d, carve(p, ws), vol, false, p.nt, st);
  flush_any(p, d, carve(p, ws), vol, false, st);
  HIP_CHECK(hipEventRecord(e1, st));
  dev_run_receivers(p, ws, E_rec, stream);
  HIP_CHECK(hipEventSynchronize(e1));
  float ms = 0;
  HIP_CHECK(hipEventElapsedTime(&ms, e0, e1));
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  p.last_ms = ms;
  p.last_steps = p.nt;
  collect_kernel_stats(d);
  check_abort(p, carve(p, ws), st);
  const WS w = carve(p, ws);
  flag_final_fields(p, w, st);
  check_finite(reinterpret_cast<double2 *>(E_rec), (size_t)p.ns * p.nr * p.ncomp * p.nf(), w.bad,
               st);
}

// ---------------------------------------------------------------------------
// Forward run with the workspace in a static device array, for callers that
// cannot allocate (code under stream capture, serving loops).  One array per
// device, shared by every call on that device (overlapping calls race);
// its device address is taken once per device with hipGetSymbolAddress.
// ---------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[FWD_STATIC_SCRATCH_BYTES];

namespace {
std::mutex g_scratch_mu;
void *g_scratch_ptr[64] = {};
}  // namespace

static void *static_scratch(int dev) {
  if (dev < 0 || dev >= 64) fail(FWD_ERR_UNSUPPORTED, "device index above 63");
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void *ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !ptr)
      fail(FWD_ERR_HIP, std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e));
    g_scratch_ptr[dev] = ptr;
  }
  return g_scratch_ptr[dev];
}

__global__ void k_or_flag(int *flag, const int *other) {
  if (threadIdx.x == 0 && blockIdx.x == 0 && other[0]) flag[0] = 1;
}

__global__ void k_nonfinite(const double *v, size_t n, int *flag) {
  const size_t st = (size_t)gridDim.x * blockDim.x;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += st)
    if (!isfinite(v[i])) flag[0] = 1;
}

void dev_forward_static(Plan &p, void *vol, size_t vol_bytes, double *E_rec, void *stream) {
  hipStream_t st = static_cast<hipStream_t>(stream);
  int dev = 0;
  HIP_CHECK(hipGetDevice(&dev));
  void *ws = static_scratch(dev);
  const size_t need = p.workspace_bytes(FWD_MODE_FORWARD), flag_off = a256(need);
  if (flag_off + 256 > (size_t)FWD_STATIC_SCRATCH_BYTES)
    fail(FWD_ERR_INVALID_ARG, "forward workspace of " + std::to_string(need) +
                                  " bytes exceeds the static scratch of " +
                                  std::to_string((size_t)FWD_STATIC_SCRATCH_BYTES) + " bytes");
  if (vol && vol_bytes < p.volume_bytes()) fail(FWD_ERR_INVALID_ARG, "volume buffer too small");
  // everything the run uses must already be on this device: building the
  // tables or the entry lists would allocate
  Dev *dp = static_cast<Dev *>(p.dev);
  if (!dp || dp->device != dev || dp->model_version != p.model_version ||
      dp->basis_version != p.basis_version || dp->list_key != lists_key(p))
    fail(FWD_ERR_STATE, "plan tables not resident on this device for the current model and "
                        "tiling: run fwd_forward once first");
  Dev &d = *dp;
  const WS w = carve(p, ws);
  zero_state(p, w, ws, FWD_MODE_FORWARD, st);
  run_steps_any(p, d, w, vol, false, p.nt, st, true);
  flush_any(p, d, w, vol, false, st);
  dev_run_receivers(p, ws, E_rec, stream);
  int *flag = reinterpret_cast<int *>(static_cast<char *>(ws) + flag_off);
  hipLaunchKernelGGL(k_set_int, dim3(1), dim3(64), 0, st, flag, 0);
  const size_t n = 2 * (size_t)p.ns * p.nr * p.ncomp * p.nf();
  hipLaunchKernelGGL(k_nonfinite, dim3((unsigned)std::min<size_t>((n + 255) / 256, 1024)),
                     dim3(256), 0, st, E_rec, n, flag);
  flag_final_fields(p, w, st);                 // into w.bad, cleared by zero_state
  hipLaunchKernelGGL(k_or_flag, dim3(1), dim3(64), 0, st, flag, (const int *)w.bad);
  HIP_CHECK(hipGetLastError());
  int bad = 0;
  HIP_CHECK(hipMemcpyAsync(&bad, flag, sizeof bad, hipMemcpyDeviceToHost, st));
  HIP_CHECK(hipStreamSynchronize(st));
  if (bad) fail(FWD_ERR_NONFINITE, "non-finite field: unstable run (dt above the CFL bound?)");
}

void dev_checkpoint(Plan &p, const void *ws, const void *vol, void *snap, int save, void *stream) {
  hipStream_t st = static_cast<hipStream_t>(stream);
  const size_t sb = p.state_bytes();
  char *sn = static_cast<char *>(snap);
  if (save) {
    HIP_CHECK(hipMemcpyAsync(sn, ws, sb, hipMemcpyDeviceToDevice, st));
    if (vol) HIP_CHECK(hipMemcpyAsync(sn + sb, vol, p.volume_bytes(), hipMemcpyDeviceToDevice, st));
  } else {
    HIP_CHECK(hipMemcpyAsync(const_cast<void *>(ws), sn, sb, hipMemcpyDeviceToDevice, st));
    if (vol)
      HIP_CHECK(hipMemcpyAsync(const_cast<void *>(vol), sn + sb, p.volume_bytes(),
                               hipMemcpyDeviceToDevice, st));
    read_host_step(p, ws, st);             // follows the restored counters
  }
}

void dev_volume_export(Plan &p, const void *vol, double *out, void *stream) {
  hipStream_t st = static_cast<hipStream_t>(stream);
  ensure_tables(p, st);
  Dev &d = D(p);
  if (p.NY > 65535) fail(FWD_ERR_UNSUPPORTED, "volume export: ny too large");
  const dim3 block(64), grid((p.NX + 63) / 64, p.NY, std::min(p.ns * p.nf() * 3 * p.NZ, 4096));
  double2 *o = reinterpret_cast<double2 *>(out);
  switch (p.acc) {
    case FWD_ACC_F64:
      hipLaunchKernelGGL((k_vol_export<ACC_F64>), grid, block, 0, st, p.ns, p.nf(), p.NX, p.NY, p.NZ,
                         p.PX, p.field_elems(), vol, d.vol_scale, o);
      break;
    case FWD_ACC_KAHAN:
      hipLaunchKernelGGL((k_vol_export<ACC_KAHAN>), grid, block, 0, st, p.ns, p.nf(), p.NX, p.NY,
                         p.NZ, p.PX, p.field_elems(), vol, d.vol_scale, o);
      break;
    default:
      hipLaunchKernelGGL((k_vol_export<ACC_F32>), grid, block, 0, st, p.ns, p.nf(), p.NX, p.NY, p.NZ,
                         p.PX, p.field_elems(), vol, d.vol_scale, o);
  }
  HIP_CHECK(hipGetLastError());
}

void dev_adjoint(Plan &p, void *ws, size_t ws_bytes, const void *vol, const double *resid,
                 double *grad, int accumulate, double *E_adj, void *stream) {
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (!p.have_basis) fail(FWD_ERR_BASIS, "build the basis functions first (fwd_basis_build)");
  if (!vol) fail(FWD_ERR_INVALID_ARG, "adjoint needs the forward volume transform");
  check_sizes(p, ws_bytes, FWD_MODE_ADJOINT, const_cast<void *>(vol), p.volume_bytes());
  ensure_tables(p, st);
  Dev &d = D(p);
  WS w = carve(p, ws);
  // adjoint coefficients from the residual, on the device: spectrum ->
  // nodes, the power-of-two scale, then the scaled coefficients
  const int nn = (int)p.rn_c.size(), nsn = p.ns * nn;
  if (nsn > 0) {
    hipLaunchKernelGGL(k_adj_coef, dim3((nsn + 127) / 128), dim3(128), 0, st, p.ns, nn, p.nf(),
                       p.nr * p.ncomp, resid, d.at_ptr, d.at_row, d.at_w, d.rn_c, d.adj_fac,
                       d.adj_fac_h, d.adj_bmax, d.adj_nodefac, d.at_coef, d.adj_inc);
  }
  hipLaunchKernelGGL(k_adj_scale, dim3(1), dim3(256), 0, st, d.adj_inc, nsn, p.nf(), d.adj_scale,
                     d.adj_scale_v);
  {
    const int64_t nc = (int64_t)nsn * 2 * p.nf();
    if (nc > 0)
      hipLaunchKernelGGL(k_adj_apply, dim3((unsigned)std::min<int64_t>((nc + 255) / 256, 1024)),
                         dim3(256), 0, st, d.at_coef, nc, (const double *)d.adj_scale);
  }
  HIP_CHECK(hipGetLastError());
  zero_state(p, w, ws, FWD_MODE_ADJOINT, st);
  d.kstat_n = 0;
  hipEvent_t e0, e1;
  HIP_CHECK(hipEventCreate(&e0));
  HIP_CHECK(hipEventCreate(&e1));
  HIP_CHECK(hipEventRecord(e0, st));
  run_steps_any(p, d, w, const_cast<void *>(vol), true, p.nt, st);
  flush_any(p, d, w, const_cast<void *>(vol), true, st);
  HIP_CHECK(hipEventRecord(e1, st));
  // gradient on cells, scaled by 1 / (src_scale adj_scale)
  hipLaunchKernelGGL(k_grad_cells, dim3((p.nx + 127) / 128, p.ny, p.nz), dim3(128), 0, st, p.nx,
                     p.ny, p.nz, p.ns, p.PX, p.NY, p.field_elems(), w.gedge, d.cellfac,
                     d.cellfac_v, p.src_scale, (const double *)d.adj_scale, grad, accumulate,
                     p.vti_grad, d.vratio, d.LA);
  HIP_CHECK(hipGetLastError());
  const int nrows = p.nr * p.ncomp, n = p.ns * nrows * p.nf();
  double2 *dst = E_adj ? reinterpret_cast<double2 *>(E_adj) : d.eadj;
  hipLaunchKernelGGL(k_rec_out, dim3((n + 127) / 128), dim3(128), 0, st, p.ns, nrows, nn, p.nf(),
                     d.ri_ptr, d.ri_node, d.ri_w, w.racc, d.adj_scale_v, d.adj_scale_v, d.rcomp,
                     p.ncomp, dst);
  HIP_CHECK(hipGetLastError());
  HIP_CHECK(hipEventSynchronize(e1));
  float ms = 0;
  HIP_CHECK(hipEventElapsedTime(&ms, e0, e1));
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  p.last_ms = ms;
  p.last_steps = p.nt;
  collect_kernel_stats(d);
  check_abort(p, w, st);
  flag_final_fields(p, w, st);
  flag_nonfinite(grad, (size_t)p.nx * p.ny * p.nz * (p.vti_grad ? 2 : 1), w.bad, st);
  check_finite(dst, (size_t)n, w.bad, st);
}

// ---------------------------------------------------------------------------
// time-domain adjoint: forward with checkpoints of the core state every
// `segment` steps; then, from the last segment to the first, replay the
// segment forward (keeping E after every step) and run its reverse steps.
// ---------------------------------------------------------------------------
template <typename T>
static void adjoint_td_t(Plan &p, Dev &d, const WS &w, void *ws, char *scratch, int L,
                         const std::vector<double> &C, double gscale, double *grad, int accumulate, hipStream_t st) {
  const int64_t F = p.field_elems();
  const int nt = p.nt, ns = p.ns, nn = (int)p.rn_c.size(), nf = p.nf();
  const int nseg = (nt + L - 1) / L;
  const size_t core = p.core_state_bytes(), ckb = a256(core);
  char *b = scratch;
  char *ckpt = b;
  b += (size_t)nseg * ckb;
  T *eseg = reinterpret_cast<T *>(b);
  b += a256((size_t)(L + 1) * ns * 3 * F * sizeof(T));
  T *afld = reinterpret_cast<T *>(b);
  const size_t afld_b = (size_t)ns * 6 * F * sizeof(T);
  b += a256(afld_b);
  T *apsi = reinterpret_cast<T *>(b);
  const size_t apsi_b = (size_t)ns * p.psi_elems_per_source() * sizeof(T);
  b += a256(apsi_b);
  double *gedge = reinterpret_cast<double *>(b);
  b += a256((size_t)ns * 3 * F * 8);
  double2 *coef = reinterpret_cast<double2 *>(b);
  HIP_CHECK(hipMemcpyAsync(coef, C.data(), C.size() * sizeof(double), hipMemcpyHostToDevice, st));
  T *fields = static_cast<T *>(w.fields);
  const int64_t fbuf = (int64_t)ns * 6 * F, eslice = (int64_t)ns * 3 * F;
  const int cgrid = (int)std::min<int64_t>(((int64_t)ns * 3 * F + 255) / 256, 65536);
  auto copy_e = [&](int t, int half) {
    hipLaunchKernelGGL((k_copy_e<T>), dim3(cgrid), dim3(256), 0, st, eseg + t * eslice, fields, fbuf,
                       half, ns, F);
  };
  // the len steps from n0 on, keeping E^{n0} .. E^{n0+len} in eseg: rows of
  // waves store it with the step (a copy after each took 6.8 us on the marine
  // grid, of 22 us a step), the general kernels' is copied
  const bool keep = wave_rows(p);
  auto segment = [&](int n0, int len) {
    hipLaunchKernelGGL(k_equalize, dim3(1), dim3(64), 0, st, w.step);
    copy_e(0, n0 & 1);
    int r = 0;
    for (int t = 1; t <= len; ++t) {
      enqueue_step<T>(p, d, w, nullptr, false, st, nullptr, r, n0 + t - 1, nullptr,
                      keep ? eseg + t * eslice : nullptr);
      r ^= 1;
      if (!keep) copy_e(t, (n0 + t) & 1);
    }
  };
  // forward run, checkpointing the core state at the start of every segment;
  // the last one is kept at once where no kernel times are sampled
  zero_state(p, w, ws, FWD_MODE_FORWARD, st);
  const bool last_kept = d.sample_every <= 0 && p.sched != 2;
  for (int sg = 0; sg < nseg; ++sg) {
    const int n0 = sg * L, len = std::min(L, nt - n0);
    if (last_kept && sg == nseg - 1) {
      segment(n0, len);
      p.host_step = nt;
      break;
    }
    HIP_CHECK(hipMemcpyAsync(ckpt + (size_t)sg * ckb, ws, core, hipMemcpyDeviceToDevice, st));
    run_steps_t<T>(p, d, w, nullptr, false, len, st);
  }
  // adjoint state at zero; the sensitivity to the last sample E^nt
  HIP_CHECK(hipMemsetAsync(afld, 0, afld_b, st));
  HIP_CHECK(hipMemsetAsync(apsi, 0, apsi_b, st));
  HIP_CHECK(hipMemsetAsync(gedge, 0, (size_t)ns * 3 * F * 8, st));
  StepArgs<T> A = make_args<T>(p, d, w, nullptr, false);
  {
    // one node per thread on the plan's block shape
    const int nbx = (p.NX + p.bx - 1) / p.bx, nby = (p.NY + p.by - 1) / p.by;
    set_grid(A, nbx, nby, p.NZ);
  }
  A.fields = afld;
  A.fbuf = 0;
  A.psi = apsi;
  A.pbuf = 0;
  A.gedge = gedge;
  const dim3 block(p.bx, p.by), sgrid((ns * nn + 127) / 128), sblock(128);
  auto sens = [&](int m) {
    hipLaunchKernelGGL((k_td_sens<T>), sgrid, sblock, 0, st, afld, F, ns, nn, nf, d.rn_c, d.rn_idx,
                       coef, d.zE + (int64_t)(m - 1) * nf, 0);
  };
  // magnetic receivers: d phi / d H^{n+1/2} joins the H multipliers after
  // k_td_e (whose deferred CPML update still needs the previous value) and
  // before k_td_h reads them
  const bool rows = one_launch(p);
  LeapArgs<T> R{};
  if (rows) {
    const Tiling t = tiling(p);
    set_grid(A, t.nbx, t.nby, t.nbz);
    R = leap_args<T>(p, d, A, false, true, 0);
  }
  auto hsens = [&](int n) {
    if (d.nh > 0)
      hipLaunchKernelGGL((k_td_sens<T>), sgrid, sblock, 0, st, afld, F, ns, nn, nf, d.rn_c,
                         d.rn_idx, coef, d.zH + (int64_t)n * nf, 1);
  };
  sens(nt);
  const dim3 grid(A.nblocks), row(64);
  for (int sg = nseg - 1; sg >= 0; --sg) {
    const int n0 = sg * L, len = std::min(L, nt - n0);
    if (!last_kept || sg < nseg - 1) {   // replay the segment from its checkpoint
      HIP_CHECK(hipMemcpyAsync(ws, ckpt + (size_t)sg * ckb, core, hipMemcpyDeviceToDevice, st));
      segment(n0, len);
    }
    // reverse steps n0 + len - 1 .. n0
    for (int n = n0 + len - 1; n >= n0; --n) {
      const int t = n - n0;
      if (rows) {
        const double2 *zh = d.nh > 0 ? d.zH + (int64_t)n * nf : nullptr;
        const double2 *ze = n >= 1 ? d.zE + (int64_t)(n - 1) * nf : nullptr;
        hipLaunchKernelGGL((k_rows_td_e<T>), grid, row, 0, st, R, A, coef, zh);
        hipLaunchKernelGGL((k_rows_td_h<T>), grid, row, 0, st, R, A, eseg + (t + 1) * eslice,
                           eseg + t * eslice, d.tdw, coef, ze);
        continue;
      }
      if (p.fd_order == 4) {
        hipLaunchKernelGGL((k_td_e<T, 4>), grid, block, 0, st, A);
        hsens(n);
        hipLaunchKernelGGL((k_td_h<T, 4>), grid, block, 0, st, A, eseg + (t + 1) * eslice,
                           eseg + t * eslice, d.tdw);
      } else {
        hipLaunchKernelGGL((k_td_e<T, 2>), grid, block, 0, st, A);
        hsens(n);
        hipLaunchKernelGGL((k_td_h<T, 2>), grid, block, 0, st, A, eseg + (t + 1) * eslice,
                           eseg + t * eslice, d.tdw);
      }
      if (n >= 1) sens(n);
    }
    HIP_CHECK(hipGetLastError());
  }
  hipLaunchKernelGGL(k_grad_cells, dim3((p.nx + 127) / 128, p.ny, p.nz), dim3(128), 0, st, p.nx,
                     p.ny, p.nz, p.ns, p.PX, p.NY, p.field_elems(), gedge, d.cellfac, d.cellfac_v,
                     gscale, (const double *)nullptr, grad, accumulate, p.vti_grad, d.vratio,
                     d.LA);
  HIP_CHECK(hipGetLastError());
}

void dev_adjoint_td(Plan &p, void *ws, size_t ws_bytes, void *scratch, size_t scratch_bytes,
                    int segment, const double *resid, double *grad, int accumulate, void *stream) {
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (segment < 1) fail(FWD_ERR_INVALID_ARG, "segment must be >= 1");
  check_sizes(p, ws_bytes, FWD_MODE_FORWARD, nullptr, 0);
  if (scratch_bytes < p.td_scratch_bytes(segment))
    fail(FWD_ERR_INVALID_ARG, "time-domain adjoint scratch too small");
  if (p.bx * p.by > 256) fail(FWD_ERR_INVALID_ARG, "block x * block y must be <= 256");
  ensure_tables(p, st);
  Dev &d = D(p);
  WS w = carve(p, ws);
  const size_t nres = (size_t)p.ns * p.nr * p.ncomp * p.nf();
  std::vector<double> rh(2 * nres);
  HIP_CHECK(hipMemcpyAsync(rh.data(), resid, rh.size() * sizeof(double), hipMemcpyDeviceToHost, st));
  HIP_CHECK(hipStreamSynchronize(st));
  std::vector<double> C;
  double scale = 1.0;
  td_coefficients(p, rh.data(), C, scale);
  if (!d.tdw) {
    std::vector<double> W;
    td_edge_weights(p, W);
    d.tdw = upload(d, W);
  }
  build_lists(p, d);
  d.kstat_n = 0;
  const double gscale = 1.0 / (p.src_scale * scale);
  hipEvent_t e0, e1;
  HIP_CHECK(hipEventCreate(&e0));
  HIP_CHECK(hipEventCreate(&e1));
  HIP_CHECK(hipEventRecord(e0, st));
  if (p.dtype == FWD_F64)
    adjoint_td_t<double>(p, d, w, ws, static_cast<char *>(scratch), segment, C, gscale, grad,
                         accumulate, st);
  else
    adjoint_td_t<float>(p, d, w, ws, static_cast<char *>(scratch), segment, C, gscale, grad,
                        accumulate, st);
  HIP_CHECK(hipEventRecord(e1, st));
  HIP_CHECK(hipEventSynchronize(e1));   // C (host) stays alive until here
  float ms = 0;
  HIP_CHECK(hipEventElapsedTime(&ms, e0, e1));
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  p.last_ms = ms;
  p.last_steps = p.nt;
}

// ---------------------------------------------------------------------------
// autotuner: time candidate schedules and tilings on the real buffers.  A
// staged search (coordinate descent) instead of the full product: the rows of
// waves, or where they do not apply block shapes; vector widths; tile order x
// XCD remap; the fused schedule's shapes and planes per block; the transform
// block K (8 or 16, when the workspace holds the longer history).  Each candidate first runs `steps` steps
// untimed (its HIP graph is captured and instantiated there), then the same
// number timed, so the timed interval holds the replays only.  Results are
// cached for the process, keyed by everything that shapes the work.
// ---------------------------------------------------------------------------
namespace {
struct TuneCand {
  int sched, bx, by, vx, vxh, kz, order, xcd, kb;
};
struct TuneHit {
  TuneCand c;
  double ms;
};
std::mutex g_tune_mu;
std::map<std::string, TuneHit> g_tune_cache;

TuneCand cand_of(const Plan &p) {
  return {p.sched, p.bx, p.by, p.vx, p.vxh, p.kz, p.order, p.xcd, p.kb};
}
void apply_cand(Plan &p, const TuneCand &c) {
  p.sched = c.sched;
  p.bx = c.bx;
  p.by = c.by;
  p.vx = c.vx;
  p.vxh = c.vxh;
  p.kz = c.kz;
  p.order = c.order;
  p.xcd = c.xcd;
  p.kb = c.kb;
}
}  // namespace

double dev_autotune(Plan &p, void *ws, size_t ws_bytes, void *vol, size_t vol_bytes, int mode,
                    int steps, void *stream) {
  hipStream_t st = static_cast<hipStream_t>(stream);
  const bool adj = mode == FWD_MODE_ADJOINT;
  if (adj && (!p.have_basis || !vol)) fail(FWD_ERR_STATE, "adjoint tuning needs basis and volume");
  check_sizes(p, ws_bytes, mode, vol, vol_bytes);
  ensure_tables(p, st);
  Dev &d = D(p);
  const bool o4 = p.fd_order == 4;      // order 4: two-kernel schedule, scalar threads
  // a decimated forward volume transform runs on the two-kernel schedule only
  const bool sched0_only = o4 || (vol && !adj && p.dec > 1);
  // transform blocks the caller's workspace can hold (the history grows with K)
  std::vector<int> kbs{p.kb};
  if (vol) {
    const int keep = p.kb;
    for (int kb : {8, 16, 32}) {
      p.kb = kb;
      if (kb != keep && p.workspace_bytes(mode) <= ws_bytes) kbs.push_back(kb);
    }
    p.kb = keep;
  }
  char key[256];
  snprintf(key, sizeof key, "%d/%d/%d/%d/%d/%d/%d/%d/%d/%d/%d/%d/%d/%d/%d/%d/%d/%d", p.nx, p.ny,
           p.nz, p.npml, p.ns, p.nf(), p.dtype, p.acc, p.fd_order, mode, vol ? 1 : 0,
           (int)kbs.size(), (int)p.rn_c.size(), steps, adj ? 1 : p.dec, p.stream_stores,
           rows_fit(p) ? 1 : 0, p.src_kind);
  {
    std::lock_guard<std::mutex> lk(g_tune_mu);
    auto it = g_tune_cache.find(key);
    if (it != g_tune_cache.end()) {
      apply_cand(p, it->second.c);
      return it->second.ms;
    }
  }
  const int save_sample = d.sample_every;
  d.sample_every = 0;
  hipEvent_t e0, e1;
  HIP_CHECK(hipEventCreate(&e0));
  HIP_CHECK(hipEventCreate(&e1));
  // one clean state (the whole workspace: a longer transform block lays the
  // history out further); between candidates only the step counters and
  // the flush marker are reset (stepping on from any state costs the same)
  HIP_CHECK(hipMemsetAsync(ws, 0, ws_bytes, st));
  p.host_ws = ws;
  if (vol && !adj) HIP_CHECK(hipMemsetAsync(vol, 0, p.volume_bytes(), st));
  auto time_cand = [&](const TuneCand &c, int nsteps) {
    apply_cand(p, c);
    const WS wc = carve(p, ws);
    for (int t = 0; t < 2; ++t) {
      hipLaunchKernelGGL(k_set_int, dim3(1), dim3(64), 0, st, wc.step, -1);
      hipLaunchKernelGGL(k_set_int, dim3(1), dim3(64), 0, st, wc.step + 1, -1);
      hipLaunchKernelGGL(k_set_int, dim3(1), dim3(64), 0, st, wc.flushed, 0);
      p.host_step = 0;
      if (t == 1) HIP_CHECK(hipEventRecord(e0, st));
      run_steps_any(p, d, wc, vol, adj, nsteps, st);
    }
    HIP_CHECK(hipEventRecord(e1, st));
    HIP_CHECK(hipEventSynchronize(e1));
    float ms = 0;
    HIP_CHECK(hipEventElapsedTime(&ms, e0, e1));
    return (double)ms / nsteps;
  };
  TuneCand best = cand_of(p);
  best.sched = 0;
  best.vx = best.vxh = 1;
  double best_ms = 1e300;
  auto consider = [&](const TuneCand &c) {
    const double ms = time_cand(c, steps);
    if (ms < best_ms) {
      best_ms = ms;
      best = c;
    }
    return ms;
  };
  // stage 1: rows of waves, which have no shape to choose; otherwise block
  // shapes of the two kernels, one node per thread
  const int shapes[][2] = {{64, 4}, {64, 2}, {64, 1}, {32, 8}, {32, 4}, {16, 16},
                           {16, 8}, {16, 4}, {128, 2}, {256, 1}};
  apply_cand(p, best);
  const bool leap = wave_rows(p);
  if (leap) {
    consider(TuneCand(best));
  } else {
    const TuneCand base = best;
    for (auto &sh : shapes) {
      TuneCand c = base;
      c.bx = sh[0];
      c.by = sh[1];
      consider(c);
    }
  }
  // stage 2: 16-byte vectors (both updates, then H only).  Where stage 1 had
  // no shapes, on each of them, and the best with the other remap: the pair
  // loses to the one-launch step on every FP32 grid measured and up to some
  // 10^7 FP64 nodes, and gains beyond (us a step, one launch against the best
  // pair: 101x101x61 FP32 16 and 27, 400x400x200 FP32 with 8 sources 4350 and
  // 5040; FP64: 128x128x96 61 and 69, 300x300x200 with 2 sources 1430 and
  // 1200, 400x400x200 1290 and 1080).
  if (!o4) {
    TuneCand pair = best;
    pair.vxh = pair.vx = 4;
    double pair_ms = 1e300;
    const TuneCand base = pair;
    for (size_t q = 0; q < (leap ? std::size(shapes) : 1); ++q) {
      TuneCand c = base;
      if (leap) {
        c.bx = shapes[q][0];
        c.by = shapes[q][1];
      }
      const double ms = consider(c);
      if (ms < pair_ms) {
        pair_ms = ms;
        pair = c;
      }
    }
    if (leap) {                          // stage 3 sees the better form only
      TuneCand c = pair;
      c.xcd ^= 1;
      if (consider(c) < pair_ms) pair = c;
    }
    pair.vx = 1;
    consider(pair);
  }
  // stage 3: tile order and XCD remap
  {
    const TuneCand base = best;
    for (int order : {0, 1})
      for (int xc : {0, 1}) {
        if (order == base.order && xc == base.xcd) continue;
        TuneCand c = base;
        c.order = order;
        c.xcd = xc;
        consider(c);
      }
  }
  // stage 4: the fused schedule
  if (!sched0_only) {
    const TuneCand base = best;
    const int fused[][2] = {{64, 4}, {32, 8}, {16, 16}, {16, 8}};
    for (auto &sh : fused)
      for (int kz : {2, 4, 8}) {
        TuneCand c = base;
        c.sched = 1;
        c.bx = sh[0];
        c.by = sh[1];
        c.vx = c.vxh = 1;
        c.kz = kz;
        consider(c);
      }
  }
  // the persistent schedule (transform blocks of 8 or 16 only)
  if (!sched0_only && (!vol || p.kb == 8 || p.kb == 16)) {
    const TuneCand base = best;
    const int pers[][2] = {{64, 4}, {32, 8}};
    for (auto &sh : pers) {
      TuneCand c = base;
      c.sched = 2;
      c.bx = sh[0];
      c.by = sh[1];
      c.vx = c.vxh = 1;
      consider(c);
    }
  }
  // stage 5: the transform block, every candidate over the same whole
  // number of the longest block (each closes its blocks inside the timing)
  if (kbs.size() > 1) {
    const TuneCand base = best;
    int kmax = 1;
    for (int kb : kbs) kmax = std::max(kmax, kb);
    const int ksteps = (std::max(steps, kmax) + kmax - 1) / kmax * kmax;
    double kbest = 1e300;
    for (int kb : kbs) {
      if (base.sched == 2 && kb != 8 && kb != 16) continue;   // the persistent kernel's blocks
      TuneCand c = base;
      c.kb = kb;
      const double ms = time_cand(c, ksteps);
      if (ms < kbest) {
        kbest = ms;
        best = c;
      }
    }
    best_ms = kbest;
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  apply_cand(p, best);
  d.sample_every = save_sample;
  {
    std::lock_guard<std::mutex> lk(g_tune_mu);
    g_tune_cache[key] = {best, best_ms};
  }
  return best_ms;
}

// option plumbing for the sampled timing lives with the device state
void dev_set_sampling(Plan &p, int every) { D(p).sample_every = every; }
int dev_get_sampling(Plan &p) { return p.dev ? D(p).sample_every : 0; }
void dev_kernel_stats(Plan &p, double *ms3, int *count) {
  if (!p.dev) {
    for (int k = 0; k < 3; ++k) ms3[k] = 0;
    *count = 0;
    return;
  }
  Dev &d = D(p);
  for (int k = 0; k < 3; ++k) ms3[k] = d.kstat_ms[k];
  *count = d.kstat_n;
}

}  // namespace fwdem
