// Device pieces shared by the kernels that march through a block's planes
// with a depth-3 halo: the fused rhs + RK stage and its adjoint.
#pragma once

#include <mutex>
#include <type_traits>

#include "resolve.h"
#include "wacm_internal.h"

namespace wacm {

__device__ __forceinline__ void load_tab(const Tab* __restrict__ g, Tab& s) {
  const int32_t* src = reinterpret_cast<const int32_t*>(g);
  int32_t* dst = reinterpret_cast<int32_t*>(&s);
  for (int q = threadIdx.x; q < (int)(sizeof(Tab) / 4); q += blockDim.x) dst[q] = src[q];
}

// Barrier that orders LDS traffic only: global loads issued before it stay in
// flight (they are the next plane's prefetch).
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  // s_waitcnt lgkmcnt(0): this wave's LDS writes have completed before it
  // arrives (the fence alone need not wait for them)
  __builtin_amdgcn_s_waitcnt(0xC07F);
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Persistent loop over the work items (block b, tile t) = item b nty + t of
// the Morton-ordered block list.  With xcd_map, workgroup w (dispatched to XCD
// w % 8) walks a contiguous eighth of the items, so blocks that share faces
// are processed close in time on the same L2; otherwise items go round-robin.
struct BlockIter {
  int64_t ib, end, step;
  __device__ BlockIter(int64_t n, int xcd_map) {
    const int64_t G = gridDim.x, w = blockIdx.x;
    if (xcd_map && G % 8 == 0 && n >= G) {
      const int64_t per = G / 8, xcd = w % 8, lw = w / 8;
      const int64_t chunk = (n + 7) / 8;
      const int64_t start = xcd * chunk;
      end = start + chunk < n ? start + chunk : n;
      ib = start + lw;
      step = per;
    } else {
      ib = w;
      end = n;
      step = G;
    }
  }
};

// The plate's mask on a block, by factors.  In the body frame the box's x and
// z coordinates depend on (x, z) of the point alone and its y coordinate on y
// alone, so a block has BS^2 + BS factor values for its BS^3 points: a
// workgroup evaluates them once into LDS (4 tanh per thread of a whole block
// instead of 6 per point, FP64 tanh being what bounded the kernels with a
// mask) and forms chi = f0 f1 f2 per point, in mask_point's order.
template <int BS>
struct PlateTab {
  double f0[BS * BS], f2[BS * BS];  // [z][x]
  double f1[BS];
};
struct NoTab {};

// tanh of FP64 is +-1 exactly from |x| = 20 on (1 - tanh x < 9e-18, a
// twelfth of the last place); whole waves often lie there
__device__ __forceinline__ double tanh_sat(double x) {
  double r = copysign(1.0, x);
  if (!(fabs(x) >= 20.0)) r = tanh(x);
  return r;
}

// The sphere's mask at a point, as mask_point evaluates it.  SAT: by tanh_sat,
// whose branch pays in the time stepping's kernels; a kernel that does little
// else waits for it (force_adj_kernel, 372 blocks of 32^3, FP64: 335 us for 308).
template <bool SAT = true>
__device__ __forceinline__ double sphere_chi(const wacm_params& p, double x, double y, double z) {
  const double dx = x - p.sph_c[0], dy = y - p.sph_c[1], dz = z - p.sph_c[2];
  const double d = sqrt(fma(dx, dx, fma(dy, dy, dz * dz))) - p.sph_r;
  const double chi = 0.5 * (1.0 - (SAT ? tanh_sat(d / p.w) : tanh(d / p.w)));
  return p.clip && chi < 1e-8 ? 0.0 : chi;
}

__device__ __forceinline__ double box_factor(double b, double lo, double hi, double w) {
  return 0.5 * (tanh_sat((b - lo) / w) - tanh_sat((b - hi) / w));
}

template <int BS>
__device__ __forceinline__ void plate_tab_fill(const wacm_params& p, const MaskTime& mt,
                                               const int32_t* meta, double h, PlateTab<BS>& t,
                                               int z0 = 0, int nz = BS) {
  for (int q = z0 * BS + threadIdx.x; q < (z0 + nz) * BS; q += blockDim.x) {  // nz planes
    const int x = q % BS, z = q / BS;
    const double rx = (double)(meta[2] * BS + x) * h - p.x_le[0];
    const double rz = (double)(meta[4] * BS + z) * h - p.x_le[2];
    t.f0[q] = box_factor(fma(mt.ca, rx, -(mt.sa * rz)), p.lo[0], p.hi[0], p.w);
    t.f2[q] = box_factor(fma(mt.sa, rx, mt.ca * rz), p.lo[2], p.hi[2], p.w);
  }
  for (int y = threadIdx.x; y < BS; y += blockDim.x)
    t.f1[y] = box_factor((double)(meta[3] * BS + y) * h - p.x_le[1], p.lo[1], p.hi[1], p.w);
}

template <int BS>
__device__ __forceinline__ double plate_tab_chi(const wacm_params& p, const PlateTab<BS>& t,
                                                int x, int y, int z) {
  double chi = t.f0[z * BS + x];
  chi *= t.f1[y];
  chi *= t.f2[z * BS + x];
  return p.clip && chi < 1e-8 ? 0.0 : chi;
}

// The same with each factor's derivative in its body coordinate (adjoint).
template <int BS>
struct PlateAdjTab {
  double f0[BS * BS], f2[BS * BS], g0[BS * BS], g2[BS * BS];  // [z][x]
  double f1[BS];
};

__device__ __forceinline__ void box_factor_adj(double b, double lo, double hi, double w,
                                               double& f, double& g) {
  const double ta = tanh_sat((b - lo) / w), tb = tanh_sat((b - hi) / w);
  f = 0.5 * (ta - tb);
  g = 0.5 * ((1.0 - ta * ta) - (1.0 - tb * tb)) / w;
}

template <int BS>
__device__ __forceinline__ void plate_adj_tab_fill(const wacm_params& p, const PlateAdjTime& m,
                                                   const int32_t* meta, double h, int z0, int z1,
                                                   PlateAdjTab<BS>& t) {
  for (int q = z0 * BS + threadIdx.x; q < z1 * BS; q += blockDim.x) {  // planes z0..z1-1
    const int x = q % BS, z = q / BS;
    const double rx = (double)(meta[2] * BS + x) * h - p.x_le[0];
    const double rz = (double)(meta[4] * BS + z) * h - p.x_le[2];
    box_factor_adj(m.ca * rx - m.sa * rz, p.lo[0], p.hi[0], p.w, t.f0[q], t.g0[q]);
    box_factor_adj(m.sa * rx + m.ca * rz, p.lo[2], p.hi[2], p.w, t.f2[q], t.g2[q]);
  }
  for (int y = threadIdx.x; y < BS; y += blockDim.x)
    t.f1[y] = box_factor((double)(meta[3] * BS + y) * h - p.x_le[1], p.lo[1], p.hi[1], p.w);
}

// chi, its derivative in the pitch angle (the body frame turns about y: d b0 =
// -b2, d b2 = b0) and the solid velocity with its derivative in the pitch rate
template <int BS>
__device__ __forceinline__ void plate_adj_tab_point(const wacm_params& p, const PlateAdjTime& m,
                                                    const PlateAdjTab<BS>& t, int x, int y, int z,
                                                    double xg, double zg, double& chi,
                                                    double& dchi, double us[3], double dusd[3]) {
  const int q = z * BS + x;
  const double rx = xg - p.x_le[0], rz = zg - p.x_le[2];
  const double b0 = m.ca * rx - m.sa * rz, b2 = m.sa * rx + m.ca * rz;
  const double f0 = t.f0[q], f1 = t.f1[y], f2 = t.f2[q];
  chi = f0 * f1 * f2;
  dchi = t.g0[q] * -b2 * f1 * f2 + f0 * f1 * t.g2[q] * b0;
  if (p.clip && chi < 1e-8) {
    chi = 0.0;
    dchi = 0.0;
  }
  us[0] = m.ad * rz;
  us[1] = 0.0;
  us[2] = -m.ad * rx;
  dusd[0] = rz;
  dusd[1] = 0.0;
  dusd[2] = -rx;
}

// Whether the mask (bit 0) and the sponge (bit 1) reach a block at the time
// whose pitch angle has cosine ca and sine sa: elsewhere they are exactly 0
// at every point (pen_far).
__device__ __forceinline__ int pen_reach(const wacm_params& p, double L, int bs,
                                         const int32_t* meta, double ca, double sa) {
  wacm_params q = p;
  q.sponge = 0;
  int r = p.mask && !pen_far(q, L, bs, meta, PitchWindow{ca, sa, 1e-9, true}) ? 1 : 0;
  q.mask = 0;
  q.sponge = p.sponge;
  if (p.sponge && !pen_far(q, L, bs, meta, PitchWindow{ca, sa, 1e-9, true})) r |= 2;
  return r;
}

// Where the depth-3 halo of one face of the current block lives: element
// (field c, depth d away from the face, tangential t0 < t1 by axis order) is
// ptr[c fs + d sd + t0 s0 + t1 s1].  Same-level neighbours are read in place
// (their interior next to the face); faces next to a coarser or finer leaf
// point into the halo buffer filled by nlface_kernel; the rhs-only mode reads
// the block's own synchronised ghost layers.  With an x-split input the
// x faces stay affine (the neighbour's side columns); for the y and z faces
// mode = 1 and ptr is the neighbour's origin: each thread addresses its own
// column with xsplit_offset.
template <typename T>
struct FaceDesc {
  const T* ptr;
  int32_t fs, sd, s0, s1, mode;
};

// Where a stage reads the depth-3 halo of a face: HALO_NB same-level faces
// from the neighbour's interior, the others from the face-halo buffer;
// HALO_OWN every face from the input's own ghost layers; HALO_MIX same-level
// faces from the neighbour's interior, the others from the own ghost layers.
enum { HALO_NB = 0, HALO_OWN = 1, HALO_MIX = 2 };

// in, L: the stage input and its layout (xin: x-split); hb: the face-halo buffer.
template <typename T, int BS, int HALO>
__device__ __forceinline__ FaceDesc<T> face_desc(const Tab& tb, const T* in, const Layout& L,
                                                 const T* hb, int f, bool xin) {
  const int axis = f >> 1, side = f & 1;
  const int sx[3] = {1, L.P, L.P * L.P};
  const int sa = sx[axis], st0 = sx[axis == 0 ? 1 : 0], st1 = sx[axis == 2 ? 1 : 2];
  const int slot = tb.meta[0];
  const int64_t org = ((int64_t)L.ng * L.P + L.ng) * L.P + L.ng;  // local (0,0,0)
  const int r = (axis == 0 ? 2 * side : 1) + 3 * (axis == 1 ? 2 * side : 1) +
                9 * (axis == 2 ? 2 * side : 1);
  FaceDesc<T> fd;
  fd.mode = 0;
  if (HALO == HALO_OWN || (HALO == HALO_MIX && tb.kind[r] != 0)) {
    fd.ptr = in + (int64_t)slot * L.bstride + org + (int64_t)(side ? BS : -1) * sa;
    fd.fs = (int)L.fstride;
    fd.sd = side ? sa : -sa;
    fd.s0 = st0;
    fd.s1 = st1;
    return fd;
  }
  if (tb.kind[r] == 0 && xin) {
    const T* nb = in + (int64_t)tb.slot[r][0] * L.bstride;
    fd.fs = (int)L.fstride;
    if (axis == 0) {
      // side 0 reads the neighbour's last columns from the top, side 1 its
      // first ones
      fd.ptr = nb + (side ? BS * BS * (BS - 2 * XS_H) : BS * BS * (BS - XS_H) + XS_H - 1);
      fd.sd = side ? 1 : -1;
      fd.s0 = XS_H;
      fd.s1 = XS_H * BS;
    } else {
      fd.ptr = nb;
      fd.sd = fd.s0 = fd.s1 = 0;
      fd.mode = 1;
    }
  } else if (tb.kind[r] == 0) {
    fd.ptr = in + (int64_t)tb.slot[r][0] * L.bstride + org + (int64_t)(side ? 0 : BS - 1) * sa;
    fd.fs = (int)L.fstride;
    fd.sd = side ? sa : -sa;
    fd.s0 = st0;
    fd.s1 = st1;
  } else {
    fd.ptr = hb + ((int64_t)slot * 6 + f) * 12 * BS * BS;
    fd.fs = 3 * BS * BS;
    fd.sd = BS * BS;
    fd.s0 = 1;
    fd.s1 = BS;
  }
  return fd;
}

// A value the compiler takes as it is (nothing is fused into its use).
template <typename T>
__device__ __forceinline__ T opaque(T v) {
  asm("" : "+v"(v));
  return v;
}

// Streaming operands (U^n, the accumulator) are touched once per stage: load
// and store them non-temporally so the caches keep the stage input, whose
// face layers neighbouring blocks read again.
template <typename T>
__device__ __forceinline__ T ntload(const T* p, int nt) {
  return nt ? __builtin_nontemporal_load(p) : *p;
}
template <typename T>
__device__ __forceinline__ void ntstore(T v, T* p, int nt) {
  if (nt)
    __builtin_nontemporal_store(v, p);
  else
    *p = v;
}


template <typename T>
__device__ __forceinline__ T wave_max(T v) {
  for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
  return v;
}
// |u|^2 in FP64 with one fixed operation order: the maximum fused into the
// last RK4 stage and the stand-alone reduction agree bit for bit.
__device__ __forceinline__ double speed2(double u, double v, double w) {
  return __builtin_fma(w, w, __builtin_fma(v, v, u * u));
}
template <typename T>
__device__ __forceinline__ T wave_min(T v) {
  for (int o = 32; o > 0; o >>= 1) v = fmin(v, __shfl_xor(v, o, 64));
  return v;
}

template <typename T>
struct StageArgs {
  const Tab* tab;
  int64_t nb;
  const T* in;  // stage input register
  Layout Lin;
  const T* hb;  // halo buffer of faces next to other levels [slot][6][4][3][bs][bs]
  T* un;        // U^n register (the pool)
  Layout Lun;
  T* acc;  // accumulator (compact)
  Layout Lacc;
  T* out;  // next stage input, or dU for the rhs-only mode
  Layout Lout;
  const T* dus;  // extra solid velocity [slot][3][bs^3] or null
  const double* t_dev;  // step time and size on the device, or null:
  const double* dt_dev;  // t_host and dt_host
  int64_t* nmax;      // host: where the launcher leaves the number of umax_part entries
  double* umax_part;  // stage 4: per work item max |u|^2 of the new U^n, or null
  // optional block list: the blocks of this launch are blist[off + i],
  // i < bcnt[bsel], off = bsel ? bcnt[0] : 0 (the list holds the blocks
  // without penalization first, then the others; null: every block)
  const int32_t* blist;
  const int32_t* bcnt;
  int bsel;
  double t_host;
  double dt_host;
  double kscale;  // MODE 3: out = U^n + kscale dt k (1; 1/2 gives stage 2 without W)
  double L;
  int xcd_map;  // 1: give each XCD a contiguous run of work items
  int* queue;   // xcd_map 2: per-XCD work counters (QSTRIDE apart), zero at launch
  int nt;       // 1: non-temporal loads/stores of the streaming operands
  wacm_params p;
};

// Dynamic per-XCD work queues (xcd_map 2): the Morton-ordered items are cut
// into 8 contiguous chunks, one per XCD; workgroup w (on XCD w % 8) takes the
// next item of its own chunk from that chunk's counter, so the tiles of one
// block and neighbouring blocks run together on one L2, and when its chunk is
// empty it takes items from the following chunks, so no XCD idles while
// another still has work.  Each counter increment that finds a chunk empty
// moves on to the next chunk: at most 8 misses per workgroup, so every
// workgroup ends.  Thread 0 only.
constexpr int QSTRIDE = 32;  // ints between counters: one 128-byte line each
__device__ __forceinline__ int queue_take(int* ctr, int& q, int chunk, int n, int v) {
  for (int miss = 0;;) {
    const int lo = q * chunk;
    const int hi = lo + chunk < n ? lo + chunk : n;
    if (lo + v < hi) return lo + v;
    if (++miss == 8) return n;
    q = (q + 1) & 7;
    v = atomicAdd(ctr + q * QSTRIDE, 1);
  }
}

[[maybe_unused]] static __global__ void queue_clear(int* ctr) {
  if (threadIdx.x < 8 * QSTRIDE) ctr[threadIdx.x] = 0;
}

// compute units of the current device (asked once)
inline int num_cus() {
  static int cus = 0;
  static std::once_flag once;
  std::call_once(once, [] {
    int dev = 0;
    hipDeviceProp_t prop;
    if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess)
      cus = prop.multiProcessorCount;
    if (cus <= 0) cus = 256;
  });
  return cus;
}

// One launch of the stage kernel (stage_kernel.h; instantiated per element type
// in stage_f32.hip and stage_f64.hip): mode 0 rhs only, 1..4 RK stage, 10 + 1..4
// RK stage on padded registers.
template <typename T>
hipError_t stage_run(int mode, int bs, const StageArgs<T>& a, const wacm_schedule& s,
                     hipStream_t st);

}  // namespace wacm
