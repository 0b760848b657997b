// CDF 4/4 lifted restriction (Sec. 3.2) on the device: the second phase of
// the ghost synchronisation (ghost points whose owner is finer) and the
// parents of merged families.
//
// Lifting the interpolating CDF 4/0 wavelet to 4 vanishing moments turns
// restriction from decimation into a low-pass filter.  Along one axis the
// coarse value at an even fine point is
//   c = u_0 + sum_m U_m (u_m - P u_m),  m = -3, -1, 1, 3,
// P the DD4 prediction from the neighbours m-3, m-1, m+1, m+3 and
// U = (-1, 9, 9, -1)/32; expanded, a 13-tap filter on the offsets -6..6
// (zero at +-5).  In 3D it is applied along x, y and z.  The fine values are
// read from the finer leaf's padded array after the CDF 4/0 ghost fill, whose
// ghost layers must be at least 6 deep.
#include <hip/hip_runtime.h>

#include "resolve.h"
#include "stage.h"
#include "wacm_internal.h"

namespace wacm {

// Expanded lifted low-pass, offsets -6..6.
constexpr double LIFT_TAP[13] = {-1.0 / 512,  0.0,         18.0 / 512,  -16.0 / 512, -63.0 / 512,
                                 144.0 / 512, 348.0 / 512, 144.0 / 512, -63.0 / 512, -16.0 / 512,
                                 18.0 / 512,  0.0,         -1.0 / 512};

// One work item: a box of nx x ny x nz coarse outputs.  Source: the padded
// array of pool slot `sslot`; the output (dx, dy, dz) is centred on the
// source's fine point (fx0 + 2 dx, fy0 + 2 dy, fz0 + 2 dz).  Items of the
// ghost phase write into a staging buffer (4 fields, [c][dz][dy][dx], at 4 *
// base values), so that no item reads a ghost value another item rewrites;
// items of a merge write the parent's interior directly (parent slots are
// fresh).
//
// mode 0: `items` holds 12 int32 per item (dst slot, i0, j0, k0, nx, ny, nz,
//         src slot, fx0, fy0, fz0, base); outputs to `out` at 4 * base.
// mode 1: `items` is the merge list (10 int32 per parent: parent slot, 8
//         child slots, unused); item w is octant w % 8 of parent w / 8, a box
//         of (bs/2)^3 outputs at the octant's offset, centred on the child's
//         even points from (0, 0, 0); outputs into U at the parent.
struct LiftItem {
  int dslot, i0, j0, k0, nx, ny, nz, sslot, fx0, fy0, fz0;
  int64_t base;
};

template <int BS, int NF>
struct LiftDims {
  static constexpr int NM = BS / 2;           // largest box edge
  static constexpr int NROW = 2 * NM + 11;    // fine points a box needs along an axis
  static constexpr int NPT = NROW * NROW;     // fine points of a plane
  static constexpr int PER = (NPT + NT_GEN - 1) / NT_GEN;
  static constexpr int XC = 4;                // outputs of the x pass per task
  static constexpr int XI = (NF * NROW * (NM / XC) + NT_GEN - 1) / NT_GEN;
  static_assert(NM % XC == 0, "whole chunks");
};

// v += h[q] w[q] over the nonzero taps, in their order
template <typename T>
__device__ __forceinline__ T lift_taps(const T* w) {
  T v = T(0);
#pragma unroll
  for (int q = 0; q < 13; ++q)
    if (q != 1 && q != 11) v = fma(T(LIFT_TAP[q]), w[q], v);
  return v;
}

// One item: a march over its fine z planes.  Per plane: the points, loaded
// into registers one plane ahead, go to LDS; x pass in chunks of 4 outputs,
// whose tap windows overlap; y pass in chunks of YC outputs, each thread
// keeping its columns for the whole march; the z pass adds the plane to the
// sums of the at most 7 outputs that it belongs to.  Two barriers per plane,
// which wait for LDS only; where a thread's points, tasks and columns lie is
// found once per item.
template <typename T, int BS, int NF, bool INPLACE, int YC>
__device__ __forceinline__ void lift_march(const LiftItem& m, int c0, const T* U, const Layout& L,
                                           T* out, int mode, const Tab& ft, T* raw, T* xq) {
  using D = LiftDims<BS, NF>;
  constexpr int NM = D::NM, PER = D::PER, XC = D::XC, XI = D::XI;
  const int tid = threadIdx.x;
  const int nrow = 2 * m.ny + 11, ncol = 2 * m.nx + 11, nplane = 2 * m.nz + 11;
  const int npt = nrow * ncol, nxc = (m.nx + XC - 1) / XC, nxt = NF * nrow * nxc;
  // x tasks: where the window starts in raw and the outputs in xq; the latter
  // negative past the last task, the outputs present in the low 3 bits
  int xs[XI], xd[XI];
#pragma unroll
  for (int k = 0; k < XI; ++k) {
    const int t = tid + k * NT_GEN, row = t / nxc, ch = t - row * nxc;  // row: of all fields
    const int c = row / nrow;
    xs[k] = row * ncol + 2 * XC * ch;
    const int left = m.nx - XC * ch;
    xd[k] = t < nxt ? ((c * D::NROW + row - c * nrow) * NM + XC * ch) * 8 + (left < XC ? left : XC)
                    : -1;
  }
  // this thread's columns: YC outputs along y of one field and dx
  const int nyc = (m.ny + YC - 1) / YC;
  const int yt = tid / m.nx, dx = tid - yt * m.nx, yfld = yt / nyc, dy0 = (yt - yfld * nyc) * YC;
  const bool own = yfld < NF;
  const T* yq = xq + (own ? (yfld * D::NROW + 2 * dy0) * NM + dx : 0);
  T acc[YC][7];
#pragma unroll
  for (int e = 0; e < YC; ++e)
#pragma unroll
    for (int j = 0; j < 7; ++j) acc[e][j] = T(0);
  const T* src = U + c0 * L.fstride;
  const int64_t zs = (int64_t)L.P * L.P;
  const T* ptr[PER];
  T v[PER][NF];
  // Addresses of this thread's points in plane z.  INPLACE: values of the
  // finer leaf's ghost regions whose level-J box is a leaf are read from that
  // leaf's interior (the same values its ghost fill would copy there); the
  // other ghost regions from its array.
  auto locate = [&](int z) {
    const int rz = z < 0 ? 0 : (z < BS ? 1 : 2);
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      int p = tid + k * NT_GEN;
      p = p < npt ? p : 0;
      const int yf = p / ncol, x = m.fx0 - 6 + (p - yf * ncol), y = m.fy0 - 6 + yf;
      int64_t slot = m.sslot;
      int sx = 0, sy = 0, sz = 0;
      if constexpr (INPLACE) {
        const int rx = x < 0 ? 0 : (x < BS ? 1 : 2), ry = y < 0 ? 0 : (y < BS ? 1 : 2);
        const int r = rx + 3 * ry + 9 * rz;
        if (r != 13 && ft.kind[r] == 0) {
          slot = ft.slot[r][0];
          sx = (1 - rx) * BS, sy = (1 - ry) * BS, sz = (1 - rz) * BS;
        }
      }
      ptr[k] = src + slot * L.bstride +
               ((int64_t)(z + sz + L.ng) * L.P + (y + sy + L.ng)) * L.P + (x + sx + L.ng);
    }
  };
  auto load = [&]() {
#pragma unroll
    for (int k = 0; k < PER; ++k)
#pragma unroll
      for (int c = 0; c < NF; ++c) v[k][c] = ptr[k][c * L.fstride];
  };
  locate(m.fz0 - 6);
  load();
  for (int zf = 0; zf < nplane; ++zf) {
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int p = tid + k * NT_GEN;
      if (p < npt)
#pragma unroll
        for (int c = 0; c < NF; ++c) raw[c * npt + p] = v[k][c];
    }
    lds_barrier();
    if (zf + 1 < nplane) {
      const int z = m.fz0 - 5 + zf;
      if (INPLACE && (z == 0 || z == BS)) {
        locate(z);
      } else {
#pragma unroll
        for (int k = 0; k < PER; ++k) ptr[k] += zs;
      }
      load();
    }
#pragma unroll
    for (int k = 0; k < XI; ++k)
      if (xd[k] >= 0) {
        T w[2 * (XC - 1) + 13];
#pragma unroll
        for (int q = 0; q < 2 * (XC - 1) + 13; ++q) w[q] = raw[xs[k] + q];
        T* o = xq + (xd[k] >> 3);
        const int no = xd[k] & 7;
#pragma unroll
        for (int e = 0; e < XC; ++e) {
          const T s = lift_taps(w + 2 * e);
          if (e < no) o[e] = s;
        }
      }
    lds_barrier();
    if (own) {
      T w[2 * (YC - 1) + 13], s[YC];
#pragma unroll
      for (int q = 0; q < 2 * (YC - 1) + 13; ++q) w[q] = yq[q * NM];
#pragma unroll
      for (int e = 0; e < YC; ++e) s[e] = lift_taps(w + 2 * e);
      if ((zf & 1) == 0) {
        // the outputs zf/2 - 6 .. zf/2, of which the first is complete
        const int k = zf / 2 - 6;
#pragma unroll
        for (int e = 0; e < YC; ++e) {
#pragma unroll
          for (int j = 0; j < 7; ++j) acc[e][j] = fma(T(LIFT_TAP[12 - 2 * j]), s[e], acc[e][j]);
          if (k >= 0 && dy0 + e < m.ny) {
            const int cf = c0 + yfld, dy = dy0 + e;
            if (mode == 0)
              out[m.base + ((int64_t)(cf * m.nz + k) * m.ny + dy) * m.nx + dx] = acc[e][0];
            else
              out[(int64_t)m.dslot * L.bstride + cf * L.fstride +
                  ((int64_t)(m.k0 + k + L.ng) * L.P + (m.j0 + dy + L.ng)) * L.P +
                  (m.i0 + dx + L.ng)] = acc[e][0];
          }
#pragma unroll
          for (int j = 0; j < 6; ++j) acc[e][j] = acc[e][j + 1];
          acc[e][6] = T(0);
        }
      } else {
#pragma unroll
        for (int e = 0; e < YC; ++e)
#pragma unroll
          for (int j = 1; j < 5; ++j) acc[e][j] = fma(T(LIFT_TAP[11 - 2 * j]), s[e], acc[e][j]);
      }
    }
  }
}

// A work unit is a pair of fields of an item: all 4 at once make the units too
// few and too unequal for the chip (587 us against 448, the bound being the
// memory latency of each plane), one alone halves the loads in flight (497).
// Before, the x pass loaded its 11 taps per output from memory: 668 us; all on
// 2000 blocks of 24^3, FP64, where it fetches 1.1 GB.  Boxes thin along x or y
// give every output column a thread of its own.
template <typename T, int BS, bool INPLACE>
__global__ __launch_bounds__(NT_GEN) void lift_box_kernel(const int32_t* __restrict__ items,
                                                          int64_t n, const T* U, Layout L,
                                                          T* out, int mode,
                                                          const Tab* __restrict__ tab,
                                                          const int32_t* __restrict__ stab) {
  constexpr int NF = 2, NM = BS / 2, YC = 2;
  using D = LiftDims<BS, NF>;
  static_assert(NF * NM * (NM / YC) <= NT_GEN && NM % YC == 0, "one thread per chunk of columns");
  // a fine plane (a chunk's unused outputs read up to 6 values past it)
  __shared__ T raw[NF * D::NPT + 8];
  __shared__ T xq[NF * D::NROW * NM];  // its x pass
  __shared__ Tab ft;                   // the finer leaf's table (in-place reads)
  for (int64_t u = blockIdx.x; u < 2 * n; u += gridDim.x) {
    const int64_t w = u >> 1;
    LiftItem m;
    if (mode == 0) {
      const int32_t* e = items + 12 * w;
      m = {e[0], e[1], e[2], e[3], e[4], e[5], e[6], e[7], e[8], e[9], e[10], (int64_t)e[11] * 4};
    } else {
      const int32_t* e = items + 10 * (w >> 3);
      const int oc = (int)(w & 7);
      m = {e[0], (oc & 1) * NM, ((oc >> 1) & 1) * NM, (oc >> 2) * NM, NM, NM, NM,
           e[1 + oc], 0, 0, 0, 0};
    }
    __syncthreads();  // the last unit's tables and planes are free again
    if constexpr (INPLACE) {
      load_tab(tab + stab[m.sslot], ft);
      __syncthreads();
    }
    const int c0 = NF * (int)(u & 1);
    if (NF * m.nx * m.ny <= NT_GEN)
      lift_march<T, BS, NF, INPLACE, 1>(m, c0, U, L, out, mode, ft, raw, xq);
    else
      lift_march<T, BS, NF, INPLACE, YC>(m, c0, U, L, out, mode, ft, raw, xq);
  }
}

// Staged ghost values (mode 0 items) into the ghost layers.
template <typename T>
__global__ __launch_bounds__(NT_GEN) void lift_scatter_kernel(const int32_t* __restrict__ items,
                                                              int64_t n, const T* __restrict__ tmp,
                                                              T* __restrict__ U, Layout L) {
  for (int64_t w = blockIdx.x; w < n; w += gridDim.x) {
    const int32_t* e = items + 12 * w;
    const int dslot = e[0], i0 = e[1], j0 = e[2], k0 = e[3], nx = e[4], ny = e[5], nz = e[6];
    const int64_t base = (int64_t)e[11] * 4;
    const int np = nx * ny * nz;
    T* dst = U + (int64_t)dslot * L.bstride;
    for (int p = threadIdx.x; p < 4 * np; p += blockDim.x) {
      const int c = p / np, q = p - c * np;
      const int dx = q % nx, dy = (q / nx) % ny, dz = q / (nx * ny);
      dst[c * L.fstride + ((int64_t)(k0 + dz + L.ng) * L.P + (j0 + dy + L.ng)) * L.P +
          (i0 + dx + L.ng)] = tmp[base + p];
    }
  }
}

static Layout lift_layout(const wacm_grid* g) {
  Layout L;
  L.P = g->P;
  L.ng = g->d.ng;
  L.fstride = (int64_t)g->P * g->P * g->P;
  L.bstride = 4 * L.fstride;
  return L;
}

static unsigned lift_grid(int64_t n) {
  const int64_t cap = 16384;
  return (unsigned)(n < cap ? (n > 0 ? n : 1) : cap);
}

template <typename T, int BS>
static hipError_t lift_box_t(const wacm_grid* g, const int32_t* items, int64_t n, T* U, T* out,
                             int mode, bool inplace, hipStream_t st) {
  if (inplace)
    lift_box_kernel<T, BS, true><<<lift_grid(2 * n), NT_GEN, 0, st>>>(
        items, n, U, lift_layout(g), out, mode, g->d_tab, lift_slot_tab(g));
  else
    lift_box_kernel<T, BS, false><<<lift_grid(2 * n), NT_GEN, 0, st>>>(
        items, n, U, lift_layout(g), out, mode, nullptr, nullptr);
  return hipGetLastError();
}

template <typename T>
static hipError_t lift_box(const wacm_grid* g, const int32_t* items, int64_t n, T* U, T* out,
                           int mode, bool inplace, hipStream_t st) {
  switch (g->d.bs) {
    case 24:
      return lift_box_t<T, 24>(g, items, n, U, out, mode, inplace, st);
    case 32:
      return lift_box_t<T, 32>(g, items, n, U, out, mode, inplace, st);
    default:
      return hipErrorInvalidValue;  // CDF 4/4 needs ng >= 6, hence bs >= 18
  }
}

// the first n items of the list (all of them, or the face star's); inplace:
// same-level values read from the neighbours' interiors
template <typename T>
static hipError_t lift_sync_t(const wacm_grid* g, T* U, int64_t n, bool inplace, hipStream_t st) {
  if (g->n_lift < 0) return hipErrorOutOfMemory;  // the last item build failed
  if (n == 0) return hipSuccess;
  if (inplace && !lift_slot_tab(g)) return hipErrorInvalidValue;
  T* tmp = (T*)g->d_lift_tmp;
  hipError_t e = lift_box<T>(g, g->d_lift, n, U, tmp, 0, inplace, st);
  if (e != hipSuccess) return e;
  lift_scatter_kernel<T><<<lift_grid(n), NT_GEN, 0, st>>>(g->d_lift, n, tmp, U, lift_layout(g));
  return hipGetLastError();
}

hipError_t launch_lift_sync(const wacm_grid* g, void* U, hipStream_t st) {
  return g->d.dtype == WACM_F64 ? lift_sync_t(g, (double*)U, g->n_lift, false, st)
                                : lift_sync_t(g, (float*)U, g->n_lift, false, st);
}

hipError_t launch_lift_sync_face(const wacm_grid* g, void* U, hipStream_t st) {
  return g->d.dtype == WACM_F64 ? lift_sync_t(g, (double*)U, g->n_lift_face, true, st)
                                : lift_sync_t(g, (float*)U, g->n_lift_face, true, st);
}

hipError_t launch_lift_coarsen(const wacm_grid* g, void* U, int64_t nparents, hipStream_t st) {
  if (nparents == 0) return hipSuccess;
  return g->d.dtype == WACM_F64
             ? lift_box<double>(g, g->d_list, 8 * nparents, (double*)U, (double*)U, 1, false, st)
             : lift_box<float>(g, g->d_list, 8 * nparents, (float*)U, (float*)U, 1, false, st);
}

// --------------------------------------------------------------------------
// Classical RK4 with CDF 4/4 ghosts.  The CDF 4/0 step reads same-level
// halos in place and fills face halos next to other levels itself; with the
// lifted restriction each stage input's ghost layers are filled first (the
// CDF 4/0 values of the regions in a coarser leaf and of the boxes the
// face-star lifted values read from finer leaves' padded arrays; then the
// lifted phase of the face star), and the fused stage kernel reads
// same-level halos in place and the others from those ghost layers: per
// stage a fill and one stage kernel, with the CDF 4/0 step's register
// arrangement (Y2/Y4, Y3 and W) in `work`, Y2/Y4 and Y3 in the padded pool
// layout, W compact.
// --------------------------------------------------------------------------
struct LiftWork {
  size_t y, k, a, total;
};
static LiftWork lift_work(const wacm_grid* g) {
  const size_t es = g->d.dtype == WACM_F64 ? 8 : 4;
  const size_t reg = (size_t)g->d.capacity * 4 * (size_t)g->P * g->P * g->P * es;
  const size_t up = (reg + 255) / 256 * 256;
  return LiftWork{0, up, 2 * up, 3 * up};
}

size_t lift_work_bytes(const wacm_grid* g) { return lift_work(g).total; }

__global__ void lift_advance_time(double* t_dev, const double* dt_dev) {
  if (threadIdx.x == 0) t_dev[0] += dt_dev[0];
}

template <typename T>
static hipError_t rk4_lifted_t(const wacm_grid* g, const wacm_params* p, double* t_dev,
                               double* dt_dev, T* U, void* work, const void* dus, int dt_mode,
                               int64_t nsteps, hipStream_t st) {
  if (g->nb == 0) return hipSuccess;
  const LiftWork wp = lift_work(g);
  T* Ya = (T*)((char*)work + wp.y);  // Y2, then Y4
  T* Yb = (T*)((char*)work + wp.k);  // Y3
  T* Wr = (T*)((char*)work + wp.a);  // W = (U^n + Y2)/3 + dt/3 k2, compact layout
  hipError_t e;
  // per stage: the CDF 4/0 fill of the input's ghosts that the stage and the
  // face-star lifted values read, the lifted values of the face star, then
  // the fused stage (same-level halos in place, the others from the ghost
  // layers); t and dt stay on the device
  auto stage = [&](int s, T* in, T* out) {
    hipError_t r = launch_sync_lifted_stage(g, in, g->d_lift_mask, st);
    if (r == hipSuccess) r = launch_lift_sync_face(g, in, st);
    if (r == hipSuccess) r = launch_stage_owng(g, p, s, t_dev, dt_dev, in, U, out, Wr, dus, st);
    return r;
  };
  for (int64_t n = 0; n < nsteps; ++n) {
    if (dt_mode == WACM_DT_CFL && (e = launch_dt(g, p, U, dt_dev, st)) != hipSuccess) return e;
    if ((e = stage(1, U, Ya)) != hipSuccess || (e = stage(2, Ya, Yb)) != hipSuccess ||
        (e = stage(3, Yb, Ya)) != hipSuccess || (e = stage(4, Ya, U)) != hipSuccess)
      return e;
    lift_advance_time<<<1, 64, 0, st>>>(t_dev, dt_dev);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_rk4_lifted(const wacm_grid* g, const wacm_params* p, double* t_dev,
                             double* dt_dev, void* U, void* work, const void* dus, int dt_mode,
                             int64_t nsteps, hipStream_t st) {
  return g->d.dtype == WACM_F64
             ? rk4_lifted_t(g, p, t_dev, dt_dev, (double*)U, work, dus, dt_mode, nsteps, st)
             : rk4_lifted_t(g, p, t_dev, dt_dev, (float*)U, work, dus, dt_mode, nsteps, st);
}

}  // namespace wacm
