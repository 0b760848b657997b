// HIP kernels of libwacm for gfx950 (MI355X).
//
// Data: the block pool U[slot][4][P][P][P] (x fastest, P = bs + 2 ng), RK
// registers in the same padded layout or compact (bs^3 per field), and the
// per-block neighbour tables (Tab) built on the host.  All kernels are
// memory-bound stencils: no MFMA; wave64 reductions; LDS slabs.
#include <algorithm>
#include <cmath>
#include <mutex>

#include "resolve.h"
#include "schedule.h"
#include "stage.h"
#include "wacm_internal.h"

namespace wacm {

// --------------------------------------------------------------------------
// ghost synchronisation
// --------------------------------------------------------------------------
// Point-wise ghost fill of all ng layers.  With skip_coarser, points of regions
// that lie in a coarser leaf are left to sync_coarser_kernel.  With `box` (the
// lifted step's read boxes, LIFT_BOX_WORDS per block): only the points inside the
// boxes of regions in a finer leaf; the lifted phase reads same-level values from
// the neighbours' interiors, and what it reads in a coarser leaf is
// sync_coarser_kernel's.
template <typename T>
__global__ __launch_bounds__(NT_GEN) void sync_kernel(const Tab* __restrict__ tab, int64_t nb,
                                                      T* __restrict__ U, Layout L, int bs,
                                                      int skip_coarser,
                                                      const int32_t* __restrict__ box) {
  __shared__ Tab st;
  __shared__ int32_t sbox[LIFT_BOX_WORDS];
  const int npts = L.P * L.P * L.P - bs * bs * bs;
  for (int64_t ib = blockIdx.x; ib < nb; ib += gridDim.x) {
    __syncthreads();
    load_tab(tab + ib, st);
    if (box && threadIdx.x < LIFT_BOX_WORDS)
      sbox[threadIdx.x] = box[ib * LIFT_BOX_WORDS + threadIdx.x];
    __syncthreads();
    T* dst = U + (int64_t)st.meta[0] * L.bstride;
    int32_t have = 0;  // boxes of regions in a finer leaf (uniform)
    if (box) {
      for (int r = 0; r < 27; ++r)
        if (r != 13 && st.kind[r] > 0) have |= sbox[13] & (int32_t(1) << r);
      if (have == 0) continue;
    }
    for (int p = threadIdx.x; p < npts; p += blockDim.x) {
      int i, j, k;
      shell_point(p, bs, L.ng, L.P, 0, i, j, k);
      const int r = region_of(i, bs) + 3 * region_of(j, bs) + 9 * region_of(k, bs);
      if (skip_coarser && st.kind[r] < 0) continue;
      if (box) {
        if (!((have >> r) & 1)) continue;
        const int32_t b = sbox[r];
        const int q[3] = {i, j, k};
        bool in = true;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
          const int o = q[d] - (q[d] < 0 ? -L.ng : (q[d] < bs ? 0 : bs));
          in = in && o >= ((b >> (10 * d)) & 31) && o <= ((b >> (10 * d + 5)) & 31);
        }
        if (!in) continue;
      }
      T v[4];
      ghost_value<T>(st, bs, L, U, i, j, k, v);
      const int64_t o = ((int64_t)(k + L.ng) * L.P + (j + L.ng)) * L.P + (i + L.ng);
#pragma unroll
      for (int c = 0; c < 4; ++c) dst[o + c * L.fstride] = v[c];
    }
  }
}

// Ghost points of the even lattice within 3 of the block: (i, j, k) all even
// in [-2, bs+2]^3 outside the interior, the points the wavelet details read
// (detail_kernel).  Each is a copy: an even point is a lattice point of a
// coarser leaf and coincides with a point of a finer one (Sec. 3.1), and
// every source is an interior point of its leaf, so no write is read.
template <typename T, int BS>
__global__ __launch_bounds__(NT_GEN) void sync_lattice_kernel(const Tab* __restrict__ tab,
                                                              int64_t nb, T* __restrict__ U,
                                                              Layout L) {
  constexpr int S = BS / 2 + 3, S3 = S * S * S;  // even positions -2, 0, ..., bs+2
  __shared__ Tab st;
  for (int64_t ib = blockIdx.x; ib < nb; ib += gridDim.x) {
    __syncthreads();
    load_tab(tab + ib, st);
    __syncthreads();
    T* dst = U + (int64_t)st.meta[0] * L.bstride;
    for (int q = threadIdx.x; q < S3; q += NT_GEN) {
      const int a = q % S, b = (q / S) % S, c = q / (S * S);
      const int i = 2 * a - 2, j = 2 * b - 2, k = 2 * c - 2;
      if (i >= 0 && i < BS && j >= 0 && j < BS && k >= 0 && k < BS) continue;
      const int64_t so = point_offset(st, BS, L, i, j, k);
      const int64_t o = ((int64_t)(k + L.ng) * L.P + (j + L.ng)) * L.P + (i + L.ng);
      T v[4];
#pragma unroll
      for (int f = 0; f < 4; ++f) v[f] = U[so + f * L.fstride];
#pragma unroll
      for (int f = 0; f < 4; ++f) dst[o + f * L.fstride] = v[f];
    }
  }
}

// Ghost regions that lie in a coarser leaf (Sec. 3.1 prediction, Sec. 4.2):
// one work item per (block, region).  The region's box of ghost points is
// predicted separably: the even lattice box around it (read from whichever
// leaves hold it) is gathered for all 4 fields at once into registers, then,
// one field at a time, predicted along x through LDS, in pairs of an even and
// an odd point that share the lattice values, and along y and z by one thread
// per column (i, j), which marches along z with the last 4 lattice layers in
// registers and writes the ghost points.  The same tensor-product DD4 values
// as the point-wise fill, summed in another order.  Requires ng <= SC_MAXG
// (checked by the launcher).  Bound: its ghost layers lie in partly written
// cache lines; it moves 1.25 GB in 411 us on 2000 blocks of 24^3, FP64 (561 us
// with a pass per axis through LDS and hardware divisions), 304 us on 1500
// blocks of 32^3, FP32 (481 before).
constexpr int SC_MAXG = 6;
template <int BS>
struct SyncCoarseDims {
  static constexpr int S = BS / 2 + 3;       // lattice points along an interior axis
  static constexpr int MG = SC_MAXG;         // lattice points along a ghost axis, ng <= 6
  static constexpr int NSRC = MG * S * S;    // largest lattice box (a face region)
  static constexpr int NA = MG * S * BS;     // largest x-pass box
};

// p / d for p d < 2^32, d > 1: the box edges are known at run time only, and a
// division of the hardware's instruction set costs some 25 operations.
struct FastDiv {
  uint32_t inv;
  __device__ explicit FastDiv(int d) : inv(0xffffffffu / (uint32_t)d + 1u) {}
  __device__ int operator()(int p) const { return (int)__umulhi((uint32_t)p, inv); }
};

template <typename T, int BS>
__global__ __launch_bounds__(NT_GEN) void sync_coarser_kernel(const Tab* __restrict__ tab,
                                                              const int32_t* __restrict__ cr,
                                                              int64_t n, T* __restrict__ U,
                                                              Layout L) {
  using D = SyncCoarseDims<BS>;
  constexpr int PER = (D::NSRC + NT_GEN - 1) / NT_GEN;
  __shared__ Tab st;
  __shared__ T buf0[D::NSRC];  // lattice box of one field
  __shared__ T buf1[D::NA];    // after the x pass: [az][ay][i]
  const T w0 = T(DDW0), w1 = T(DDW1);
  const int tid = threadIdx.x, ng = L.ng, P = L.P;
  const int64_t fs = L.fstride, zs = (int64_t)P * P;
  auto odd = [&](T a0, T a1, T a2, T a3) {
    return fma(w0, a3, fma(w1, a2, fma(w1, a1, w0 * a0)));
  };
  for (int64_t wk = blockIdx.x; wk < n; wk += gridDim.x) {
    const int32_t ib = cr[2 * wk], r = cr[2 * wk + 1];
    __syncthreads();
    load_tab(tab + ib, st);
    __syncthreads();
    T* dst = U + (int64_t)st.meta[0] * L.bstride;
    // box lo..lo+n-1 per axis, and its even lattice e0, e0+2, ... (m points)
    int lo[3], nn[3], e0[3], m[3];
    const int rd[3] = {r % 3, (r / 3) % 3, r / 9};
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      lo[d] = rd[d] == 0 ? -ng : (rd[d] == 1 ? 0 : BS);
      nn[d] = rd[d] == 1 ? BS : ng;
      const int hi = lo[d] + nn[d] - 1;
      e0[d] = (lo[d] & ~1) - 2;
      m[d] = (hi + ((hi & 1) ? 3 : 2) - e0[d]) / 2 + 1;
    }
    const int nsrc = m[0] * m[1] * m[2];
    const FastDiv by_m0(m[0]), by_m1(m[1]), by_n0(nn[0]);
    T v[PER][4];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int p = tid + q * NT_GEN;
      if (p < nsrc) {
        const int rest = by_m0(p), ax = p - rest * m[0];
        const int az = by_m1(rest), ay = rest - az * m[1];
        const int64_t o = point_offset(st, BS, L, e0[0] + 2 * ax, e0[1] + 2 * ay, e0[2] + 2 * az);
#pragma unroll
        for (int c = 0; c < 4; ++c) v[q][c] = U[o + c * fs];
      }
    }
    // pairs (2t, 2t + 1) along x: the lattice values a .. a + 3 with a = t - 1
    // - e0/2 give the even point (a + 1) and the odd one
    const int t0 = lo[0] >> 1, npx = ((lo[0] + nn[0] - 1) >> 1) - t0 + 1;
    const FastDiv by_npx(npx);
    const int nxp = m[2] * m[1] * npx, hi0 = lo[0] + nn[0] - 1;
    // a z axis along the interior is marched in two runs: more threads
    const int ncol = nn[1] * nn[0], nrun = rd[2] == 1 ? 2 : 1, len = nn[2] / nrun;
    const int rowz = m[1] * nn[0];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
#pragma unroll
      for (int q = 0; q < PER; ++q) {
        const int p = tid + q * NT_GEN;
        if (p < nsrc) buf0[p] = v[q][c];
      }
      lds_barrier();
      for (int p = tid; p < nxp; p += NT_GEN) {
        const int row = by_npx(p), t = t0 + (p - row * npx), i = 2 * t;
        const T* s = buf0 + row * m[0] + (t - 1 - e0[0] / 2);
        T* o = buf1 + row * nn[0] + (i - lo[0]);
        if (i >= lo[0]) o[0] = s[1];
        if (i < hi0) o[1] = odd(s[0], s[1], s[2], s[3]);
      }
      lds_barrier();
      for (int p = tid; p < nrun * ncol; p += NT_GEN) {
        const int run = p >= ncol ? 1 : 0, col = p - run * ncol;
        const int jj = by_n0(col), ii = col - jj * nn[0], j = lo[1] + jj;
        const bool je = (j & 1) == 0;
        const T* sy = buf1 + ((je ? j : j - 3) - e0[1]) / 2 * nn[0] + ii;
        auto y = [&](int az) -> T {  // after the y pass, at lattice layer az
          const T* q = sy + az * rowz;
          if (je) return q[0];
          return odd(q[0], q[nn[0]], q[2 * nn[0]], q[3 * nn[0]]);
        };
        const int kA = lo[2] + run * len, kB = kA + len;
        T* out = dst + c * fs + (int64_t)(j + ng) * P + (lo[0] + ii + ng);
        int az = (kA >> 1) - 1 - e0[2] / 2;
        T a0 = y(az), a1 = y(az + 1), a2 = y(az + 2);
        for (int k = kA & ~1; k < kB; k += 2) {
          T* ok = out + (k + ng) * zs;
          if (k >= kA) ok[0] = a1;
          if (k + 1 < kB) {
            const T a3 = y(az + 3);
            ok[zs] = odd(a0, a1, a2, a3);
            a0 = a1;
            a1 = a2;
            a2 = a3;
            ++az;
          }
        }
      }
    }
  }
}

// --------------------------------------------------------------------------
// fused rhs + RK4 stage (Sec. 2.2-2.3)
// --------------------------------------------------------------------------
// Faces next to a coarser or finer leaf: the depth-3 face halo of the stage
// input into the halo buffer the stage kernel reads.  A finer neighbour gives
// its coincident point (decimation, Sec. 3.1).  A coarser neighbour gives the
// tensor-product DD4 prediction (Sec. 3.1), computed separably: each thread
// gathers the 4 or 5 coarse values along the normal at its tangential lattice
// position (even local indices, read from whichever leaves hold them) for all
// 4 fields at once, so that one memory latency per face is exposed, and
// predicts along the normal in registers; then t0 through LDS in pairs of an
// even and an odd point, and t1 by one thread per column with the last 4
// lattice values in registers.  Two barriers for NF fields, which wait for LDS
// only.  With `queue` (schedule xcd_map 2) the faces, listed in the blocks'
// Morton order, are taken from per-XCD work counters like the stage kernel's
// items, so the faces of sister blocks, which read the same coarse data, meet
// in one L2.
// Bound: the gather's latency and scattered lines.  On 20000 blocks of 24^3,
// FP64, 0.73 ms per launch (0.97 with a pass per axis, field and barrier pair
// through LDS); 5000 such blocks, FP32, 140 us (178 before).  FP32 takes all
// fields at a time and is held to 4 waves per SIMD (3 at bs 32: two fields and
// 4 waves spill, 131 against 94 us on 1500 blocks); FP64 keeps its registers
// (2 waves: held to 4 it spills ~70 and slows down).
template <typename T, int BS>
__global__ __launch_bounds__(NT_GEN) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? (BS == 32 ? 3 : 4) : 1)))
void nlface_kernel(const Tab* __restrict__ tab,
                                                        const int32_t* __restrict__ cf, int64_t n,
                                                        const T* __restrict__ in, Layout Lin,
                                                        T* __restrict__ hb, int* queue) {
  constexpr int S = BS / 2 + 3;   // tangential coarse positions -2, 0, ..., bs+2
  constexpr int PER = (S * S + NT_GEN - 1) / NT_GEN;
  constexpr int B2 = BS * BS;
  constexpr int NFINE = (3 * B2 + NT_GEN - 1) / NT_GEN;
  constexpr int NF = sizeof(T) == 4 ? 4 : 2;  // fields at a time
  // columns of the last pass are halved where that fills the threads better
  constexpr int RUNS = NF * 3 * BS > NT_GEN || 2 * NF * 3 * BS <= NT_GEN ? 2 : 1;
  __shared__ Tab st;
  __shared__ T pa[NF * 3 * S * S];
  __shared__ T pb[NF * 3 * S * BS];
  __shared__ int qitem;
  const T w0 = T(DDW0), w1 = T(DDW1);
  auto odd = [&](T a0, T a1, T a2, T a3) {
    return fma(w0, a3, fma(w1, a2, fma(w1, a1, w0 * a0)));
  };
  const int64_t fs = Lin.fstride;
  const int tid = threadIdx.x;
  const bool dyn = queue != nullptr;
  int qh = blockIdx.x & 7, qpend = 0;
  const int qchunk = (int)((n + 7) / 8);
  if (dyn && tid == 0) qitem = queue_take(queue, qh, qchunk, (int)n, atomicAdd(queue + qh * QSTRIDE, 1));
  int64_t wnext = blockIdx.x;
  for (;;) {
    __syncthreads();
    const int64_t wk = dyn ? (int64_t)__builtin_amdgcn_readfirstlane(qitem) : wnext;
    if (wk >= n) break;
    wnext += gridDim.x;
    const int32_t ib = cf[2 * wk], f = cf[2 * wk + 1];
    load_tab(tab + ib, st);
    __syncthreads();
    if (dyn && tid == 0) qpend = atomicAdd(queue + qh * QSTRIDE, 1);
    const int slot = st.meta[0];
    const int axis = f >> 1, side = f & 1;
    const int ua = axis == 0 ? 1 : 0, ub = axis == 2 ? 1 : 2;  // tangential axes t0, t1
    const int r = (axis == 0 ? 2 * side : 1) + 3 * (axis == 1 ? 2 * side : 1) +
                  9 * (axis == 2 ? 2 * side : 1);
    T* hbf = hb + ((int64_t)slot * 6 + f) * 12 * B2;
    if (st.kind[r] > 0) {
      // finer neighbour: every halo point is a point of a finer leaf; all
      // loads of this thread's points first, then the stores
      T v[NFINE][4];
#pragma unroll
      for (int k = 0; k < NFINE; ++k) {
        const int p = tid + k * NT_GEN;
        if (p < 3 * B2) {
          const int d = p / B2, qq = p - d * B2;
          int li[3];
          li[axis] = side ? BS + d : -1 - d;
          li[ua] = qq % BS;
          li[ub] = qq / BS;
          const int64_t o = point_offset(st, BS, Lin, li[0], li[1], li[2]);
#pragma unroll
          for (int c = 0; c < 4; ++c) v[k][c] = in[o + c * fs];
        }
      }
#pragma unroll
      for (int k = 0; k < NFINE; ++k) {
        const int p = tid + k * NT_GEN;
        if (p < 3 * B2) {
#pragma unroll
          for (int c = 0; c < 4; ++c) hbf[(int64_t)(c * 3) * B2 + p] = v[k][c];
        }
      }
      if (dyn && tid == 0) qitem = queue_take(queue, qh, qchunk, (int)n, qpend);
      continue;
    }
    // coarser neighbour.  Normal ghost positions g_d = bs + d (side 1) or
    // -1 - d (side 0); the even positions their stencils use run from n0 in
    // steps of 2: side 1 [bs-2, bs+4] (4 points), side 0 [-6, 2] (5 points)
    const int n0 = side ? BS - 2 : -6;
    T v[PER][4][5];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int qq = tid + k * NT_GEN;
      if (qq < S * S) {
        int li[3];
        li[ua] = 2 * (qq % S) - 2;
        li[ub] = 2 * (qq / S) - 2;
#pragma unroll
        for (int m = 0; m < 5; ++m) {
          if (m == 4 && side) break;
          li[axis] = n0 + 2 * m;
          const int64_t o = point_offset(st, BS, Lin, li[0], li[1], li[2]);
#pragma unroll
          for (int c = 0; c < 4; ++c) v[k][c][m] = in[o + c * fs];
        }
      }
    }
#pragma unroll
    for (int c0 = 0; c0 < 4; c0 += NF) {
      // along the normal: pa[c][d][t1'][t0']
#pragma unroll
      for (int k = 0; k < PER; ++k) {
        const int qq = tid + k * NT_GEN;
        if (qq < S * S) {
#pragma unroll
          for (int c = 0; c < NF; ++c) {
            const T* s = v[k][c0 + c];
            T* o = pa + c * 3 * S * S + qq;
            const T low = odd(s[0], s[1], s[2], s[3]);
            o[0] = side ? s[1] : odd(s[1], s[2], s[3], s[4]);
            o[S * S] = side ? low : s[2];
            o[2 * S * S] = side ? s[2] : low;
          }
        }
      }
      lds_barrier();
      // along t0 in pairs (even, odd): pb[c][d][t1'][t0], t0 in [0, bs)
      for (int p = tid; p < NF * 3 * S * (BS / 2); p += NT_GEN) {
        const int t = p % (BS / 2), row = p / (BS / 2);
        const T* s = pa + row * S + t;
        pb[row * BS + 2 * t] = s[1];
        pb[row * BS + 2 * t + 1] = odd(s[0], s[1], s[2], s[3]);
      }
      lds_barrier();
      // along t1, one thread per column or half a column: out[c][d][t1][t0]
      for (int p = tid; p < RUNS * NF * 3 * BS; p += NT_GEN) {
        const int t0 = p % BS, rest = p / BS, run = rest / (NF * 3), cd = rest - run * (NF * 3);
        const int u0 = run * (BS / 2 / RUNS);
        const T* s = pb + (cd * S + u0) * BS + t0;
        T* o = hbf + (c0 * 3 + cd) * B2 + 2 * u0 * BS + t0;
        T a0 = s[0], a1 = s[BS], a2 = s[2 * BS];
#pragma unroll
        for (int u = 0; u < BS / 2 / RUNS; ++u) {
          const T a3 = s[(u + 3) * BS];
          o[2 * u * BS] = a1;
          o[(2 * u + 1) * BS] = odd(a0, a1, a2, a3);
          a0 = a1;
          a1 = a2;
          a2 = a3;
        }
      }
    }
    if (dyn && tid == 0) qitem = queue_take(queue, qh, qchunk, (int)n, qpend);
  }
}

// --------------------------------------------------------------------------
// reductions (FP64 accumulation, fixed order -> deterministic)
// --------------------------------------------------------------------------
// per block: max over interior points of |u|^2 -> part[ib]; the block edge
// is a template constant, so that the index arithmetic needs no division
template <typename T, int bs>
__global__ __launch_bounds__(NT_GEN) void maxu_kernel(const Tab* __restrict__ tab, int64_t nb,
                                                      const T* __restrict__ U, Layout L,
                                                      double* __restrict__ part) {
  __shared__ double red[NT_GEN / 64];
  constexpr int n3 = bs * bs * bs;
  for (int64_t ib = blockIdx.x; ib < nb; ib += gridDim.x) {
    const T* b = U + (int64_t)tab[ib].meta[0] * L.bstride;
    double m = 0.0;
#pragma unroll 4
    for (int q = threadIdx.x; q < n3; q += NT_GEN) {
      const int i = q % bs, j = (q / bs) % bs, k = q / (bs * bs);
      const int64_t o = ((int64_t)(k + L.ng) * L.P + (j + L.ng)) * L.P + (i + L.ng);
      const double u = b[o], v = b[o + L.fstride], w = b[o + 2 * L.fstride];
      m = fmax(m, speed2(u, v, w));
    }
    m = wave_max(m);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
      double r = red[0];
      for (int w = 1; w < NT_GEN / 64; ++w) r = fmax(r, red[w]);
      part[ib] = r;
    }
  }
}

// CFL step from the maxima.  With t, the time first advances by the step that
// *dt_out still holds: between two steps of one call one launch instead of two
// (349 blocks of 16^2, five steps: 219.5 -> 214.0 us).
__global__ __launch_bounds__(NT_GEN) void dt_finalize(const double* __restrict__ part, int64_t nb,
                                                      wacm_params p, double hmin,
                                                      double* dt_out, double* t) {
  __shared__ double red[NT_GEN / 64];
  double m = 0.0;
#pragma unroll 8
  for (int64_t q = threadIdx.x; q < nb; q += blockDim.x) m = fmax(m, part[q]);
  m = wave_max(m);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    double r = red[0];
    for (int w = 1; w < NT_GEN / 64; ++w) r = fmax(r, red[w]);
    const double umax = sqrt(r);
    const double ueig = umax + sqrt(umax * umax + p.c0 * p.c0);
    double dt = p.cfl * hmin / ueig;
    if (p.mask) dt = fmin(dt, p.cfl_eta * p.c_eta);
    if (p.sponge) dt = fmin(dt, p.cfl_eta * p.c_sp);
    if (p.nu > 0) dt = fmin(dt, p.cfl_nu * hmin * hmin / p.nu);
    if (t) *t = *t + *dt_out;
    *dt_out = dt;
  }
}

__global__ void advance_time(double* t, const double* dt) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *t = *t + *dt;
}

// diagnostics partials per block: [max|u|^2, max|u|, max|v|, max|w|, max|p|,
// sum chi(u-us) x3 (times h^3/C_eta), sum |u|^2 (times h^3/2), number of
// NaN or Inf values]; the maxima ignore NaN, the count sees it
// MASK: that of the parameters (the plate's factors take LDS and the masks take
// registers that the kernel without one would miss: 12034 blocks of 16^3, FP32,
// 330 us with them for 273 us).
constexpr int NDIAG = 10;
template <typename T, int bs, int MASK>
__global__ __launch_bounds__(NT_GEN) void diag_kernel(const Tab* __restrict__ tab, int64_t nb,
                                                      const T* __restrict__ U, Layout L,
                                                      const T* __restrict__ dus, double Ldom,
                                                      wacm_params p, double t,
                                                      double* __restrict__ part) {
  __shared__ double red[NDIAG][NT_GEN];
  constexpr bool PLATE = MASK == WACM_MASK_PLATE;
  __shared__ typename std::conditional<PLATE, PlateTab<bs>, NoTab>::type ptab;
  constexpr int n3 = bs * bs * bs;
  const MaskTime mt = MASK ? mask_time(p, t) : MaskTime{1.0, 0.0, 0.0};
  for (int64_t ib = blockIdx.x; ib < nb; ib += gridDim.x) {
    const int32_t* m = tab[ib].meta;
    const int slot = m[0], J = m[1];
    const double h = Ldom / (double(int64_t(1) << J) * bs);
    const T* b = U + (int64_t)slot * L.bstride;
    const bool masked = MASK && (pen_reach(p, Ldom, bs, m, mt.ca, mt.sa) & 1) != 0;
    if constexpr (PLATE) {
      if (masked) {  // uniform; the last block's reduction has ended
        plate_tab_fill<bs>(p, mt, m, h, ptab);
        __syncthreads();
      }
    }
    double acc[NDIAG] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    for (int q = threadIdx.x; q < n3; q += NT_GEN) {
      const int i = q % bs, j = (q / bs) % bs, k = q / (bs * bs);
      const int64_t o = ((int64_t)(k + L.ng) * L.P + (j + L.ng)) * L.P + (i + L.ng);
      T v[4];
      for (int c = 0; c < 4; ++c) v[c] = b[o + c * L.fstride];
      // the mask while the loads are in flight
      double chi = 0.0, us[3] = {0.0, 0.0, 0.0};
      if (masked) {
        const double xg = (double)(m[2] * bs + i) * h, yg = (double)(m[3] * bs + j) * h,
                     zg = (double)(m[4] * bs + k) * h;
        if constexpr (PLATE) {
          chi = plate_tab_chi<bs>(p, ptab, i, j, k);
          us[0] = mt.ad * (zg - p.x_le[2]);
          us[2] = -mt.ad * (xg - p.x_le[0]);
        } else {
          chi = sphere_chi<false>(p, xg, yg, zg);
        }
        if (dus)
          for (int d = 0; d < 3; ++d) us[d] += (double)dus[((int64_t)slot * 3 + d) * n3 + q];
      }
      const double u[4] = {(double)v[0], (double)v[1], (double)v[2], (double)v[3]};
      for (int c = 0; c < 4; ++c) acc[9] += isfinite(u[c]) ? 0.0 : 1.0;
      const double m2 = u[0] * u[0] + u[1] * u[1] + u[2] * u[2];
      acc[0] = fmax(acc[0], m2);
      for (int c = 0; c < 4; ++c) acc[1 + c] = fmax(acc[1 + c], fabs(u[c]));
      if (masked) {
        for (int d = 0; d < 3; ++d) acc[5 + d] += chi * (u[d] - us[d]);
      } else if (MASK) {
        // chi is 0; 0 times a value that is not finite is not
        for (int d = 0; d < 3; ++d) acc[5 + d] += 0.0 * u[d];
      }
      acc[8] += m2;
    }
    __syncthreads();
    for (int c = 0; c < NDIAG; ++c) red[c][threadIdx.x] = acc[c];
    __syncthreads();
    for (int s = NT_GEN / 2; s > 0; s >>= 1) {
      if ((int)threadIdx.x < s) {
        for (int c = 0; c < 5; ++c)
          red[c][threadIdx.x] = fmax(red[c][threadIdx.x], red[c][threadIdx.x + s]);
        for (int c = 5; c < NDIAG; ++c) red[c][threadIdx.x] += red[c][threadIdx.x + s];
      }
      __syncthreads();
    }
    if (threadIdx.x == 0) {
      const double vol = h * h * h;
      for (int c = 0; c < 5; ++c) part[ib * NDIAG + c] = red[c][0];
      for (int c = 5; c < 8; ++c)
        part[ib * NDIAG + c] = p.mask ? red[c][0] * vol / p.c_eta : 0.0;
      part[ib * NDIAG + 8] = 0.5 * red[8][0] * vol;
      part[ib * NDIAG + 9] = red[9][0];
    }
  }
}

__global__ __launch_bounds__(NT_GEN) void diag_finalize(const double* __restrict__ part,
                                                        int64_t nb, double* __restrict__ out) {
  __shared__ double red[NDIAG][NT_GEN];
  double acc[NDIAG] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
  for (int64_t q = threadIdx.x; q < nb; q += blockDim.x) {
    for (int c = 0; c < 5; ++c) acc[c] = fmax(acc[c], part[q * NDIAG + c]);
    for (int c = 5; c < NDIAG; ++c) acc[c] += part[q * NDIAG + c];
  }
  for (int c = 0; c < NDIAG; ++c) red[c][threadIdx.x] = acc[c];
  __syncthreads();
  for (int s = NT_GEN / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) {
      for (int c = 0; c < 5; ++c)
        red[c][threadIdx.x] = fmax(red[c][threadIdx.x], red[c][threadIdx.x + s]);
      for (int c = 5; c < NDIAG; ++c) red[c][threadIdx.x] += red[c][threadIdx.x + s];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    out[0] = sqrt(red[0][0]);
    for (int c = 1; c < NDIAG; ++c) out[c] = red[c][0];
  }
}

// --------------------------------------------------------------------------
// wavelet details and coarsening flags (Sec. 3.1, 3.3-3.5)
// --------------------------------------------------------------------------
// max over blocks of the per-block field maxima part[4 ib + c] -> norm[c]
// (1 where the field vanishes); used by the two-dimensional thresholding
__global__ __launch_bounds__(NT_GEN) void norm_finalize(const double* __restrict__ part,
                                                        int64_t nb, double* __restrict__ norm) {
  __shared__ double red[4][NT_GEN / 64];
  double m[4] = {0, 0, 0, 0};
  for (int64_t q = threadIdx.x; q < nb; q += blockDim.x)
    for (int c = 0; c < 4; ++c) m[c] = fmax(m[c], part[q * 4 + c]);
  for (int c = 0; c < 4; ++c) {
    const double v = wave_max(m[c]);
    if ((threadIdx.x & 63) == 0) red[c][threadIdx.x >> 6] = v;
  }
  __syncthreads();
  if (threadIdx.x < 4) {
    double r = red[threadIdx.x][0];
    for (int w = 1; w < NT_GEN / 64; ++w) r = fmax(r, red[threadIdx.x][w]);
    norm[threadIdx.x] = r > 0.0 ? r : 1.0;
  }
}

// The x and y passes of the tensor DD4 prediction, marching through the planes
// of a lattice: 4 fields together, NT = BS^2 threads, one per (i, j) column.  A
// plane's raw lattice values ([field][row][S], S points per row, SY rows) go to
// LDS, then its x pass (raw -> X, BS points per row), then each thread's y pass
// from X.  Raw values and X are double-buffered, so that a step does the x pass
// of plane m, stores plane m + 1 and loads plane m + 2 before one LDS barrier.
// Every X is formed once; threads take the even rows first, so that a wave's
// rows mostly have one parity.  A point's even lattice neighbour at or below is
// lattice index H + i / 2 (H points of halo below).
template <typename T, int BS, int S, int H>
struct PredictPlanes {
  static constexpr int NT = BS * BS, S2 = S * S, NX = S * BS;
  static constexpr int PR = (4 * S2 + NT - 1) / NT, PX = (4 * NX + NT - 1) / NT;
  T (*raw)[4 * S2];
  T (*xp)[4 * NX];
  int tid, i, j;   // this thread's column
  int lo[PR];      // element offset of its raw values in their plane, or -1
  int xs[PX];      // lattice index its x-pass values start from, or -1
  T rv[PR];
  __device__ PredictPlanes(T (*r)[4 * S2], T (*x)[4 * NX], int P, int fs, int org, int step)
      : raw(r), xp(x), tid(threadIdx.x) {
    i = tid % BS;
    const int jr = tid / BS;
    j = jr < BS / 2 ? 2 * jr : 2 * (jr - BS / 2) + 1;
#pragma unroll
    for (int q = 0; q < PR; ++q) {
      const int e = tid + q * NT, c = e / S2, k = e - c * S2;
      lo[q] = e < 4 * S2 ? c * fs + org + step * ((k / S) * P + k % S) : -1;
    }
#pragma unroll
    for (int q = 0; q < PX; ++q) {
      const int e = tid + q * NT, c = e / NX, k = e - c * NX;
      xs[q] = e < 4 * NX ? c * S2 + (k / BS) * S + H + (k % BS) / 2 : -1;
    }
  }
  __device__ void load(const T* plane) {
#pragma unroll
    for (int q = 0; q < PR; ++q) rv[q] = lo[q] >= 0 ? plane[lo[q]] : T(0);
  }
  __device__ void store(int m) {
#pragma unroll
    for (int q = 0; q < PR; ++q)
      if (lo[q] >= 0) raw[m & 1][tid + q * NT] = rv[q];
  }
  __device__ void xpass(int m) {
    const T w0 = T(DDW0), w1 = T(DDW1);
#pragma unroll
    for (int q = 0; q < PX; ++q)
      if (xs[q] >= 0) {
        const T* r = raw[m & 1] + xs[q];
        const T a = r[-1], b = r[0], c = r[1], d = r[2];
        // NX and NT are even: every value of a thread has its column's parity
        xp[m & 1][tid + q * NT] = (i & 1) ? w0 * a + w1 * b + w1 * c + w0 * d : b;
      }
  }
  // P along x and y of plane m at this thread's column, field c
  __device__ T ypass(int m, int c) const {
    const T w0 = T(DDW0), w1 = T(DDW1);
    const T* x = xp[m & 1] + c * NX + (H + j / 2) * BS + i;
    if (!(j & 1)) return x[0];
    return w0 * x[-BS] + w1 * x[0] + w1 * x[BS] + w0 * x[2 * BS];
  }
};

// Wavelet details (Sec. 3.1) of one block: d = u - P R u at every interior
// point with an odd index, P R u the tensor-product DD4 prediction from the
// block's even lattice (ghost-synchronised pool), evaluated separably while
// marching in z over the coarse planes k' = -2, 0, ..., bs + 2: x and y passes
// through LDS (PredictPlanes), the last 4 coarse planes of the thread's column
// in registers, z pass and comparison for the fine planes k' (even) and k' - 3
// (odd), whose points are loaded a plane ahead.  One workgroup per block.
// Bound: reading the block; it was the latency of each plane's own loads before
// its barrier (4005 blocks of 24^3, FP64: 1059 -> 580 us).  Per block and field
// the maxima of |u_c| and |d_c| over the interior (part[8 ib + c], part[8 ib +
// 4 + c]), and the mask range (0 without a mask, and for a block where the mask
// vanishes at time t); thr_finalize turns them into the normalised detail
// maximum and the coarsening flag (Sec. 3.3-3.5).
template <typename T, int BS>
__global__ __launch_bounds__(BS* BS) void detail_kernel(const Tab* __restrict__ tab, int64_t nb,
                                                        const T* __restrict__ U, Layout L,
                                                        double Ldom, wacm_params p, double t,
                                                        double* __restrict__ part,
                                                        double* __restrict__ mrange) {
  constexpr int S = BS / 2 + 3;  // even positions -2, 0, ..., bs+2
  using PP = PredictPlanes<T, BS, S, 1>;
  constexpr int NT = PP::NT;
  __shared__ T raw[2][4 * PP::S2], xp[2][4 * PP::NX];
  __shared__ double red[10][NT / 64];
  __shared__ PlateTab<BS> ptab;
  const T w0 = T(DDW0), w1 = T(DDW1);
  const int P = L.P, ng = L.ng, P2 = P * P, fs = (int)L.fstride;
  const int64_t ib = blockIdx.x;
  if (ib >= nb) return;  // whole workgroup
  const int32_t* m = tab[ib].meta;
  const T* b = U + (int64_t)m[0] * L.bstride;
  PP pp(raw, xp, P, fs, (ng - 2) * P + (ng - 2), 2);
  const int tid = pp.tid, i = pp.i, j = pp.j;
  const int col = (j + ng) * P + (i + ng);
  auto plane = [&](int mm) { return b + (2 * mm - 2 + ng) * P2; };
  T ue[4], uo[4];
  auto load_fine = [&](int mm) {  // the fine planes that coarse plane mm completes
    const int kc = 2 * mm - 2, ko = kc - 3;
    if (kc >= 0 && kc < BS)
#pragma unroll
      for (int c = 0; c < 4; ++c) ue[c] = b[c * fs + col + (kc + ng) * P2];
    if (ko >= 0 && ko < BS)
#pragma unroll
      for (int c = 0; c < 4; ++c) uo[c] = b[c * fs + col + (ko + ng) * P2];
  };
  pp.load(plane(0));
  double cmin = 1e300, cmax = -1e300;
  if (p.mask) {
    const MaskTime mt = mask_time(p, t);
    if (!(pen_reach(p, Ldom, BS, m, mt.ca, mt.sa) & 1)) {
      cmin = cmax = 0.0;  // the mask is exactly 0 on the whole block
    } else {
      const double h = Ldom / (double(int64_t(1) << m[1]) * BS);
      const bool plate = p.mask == WACM_MASK_PLATE;
      if (plate) {
        plate_tab_fill<BS>(p, mt, m, h, ptab);
        __syncthreads();
      }
      for (int k = 0; k < BS; ++k) {
        const double chi = plate ? plate_tab_chi<BS>(p, ptab, i, j, k)
                                 : sphere_chi(p, (double)(m[2] * BS + i) * h,
                                              (double)(m[3] * BS + j) * h,
                                              (double)(m[4] * BS + k) * h);
        cmin = fmin(cmin, chi);
        cmax = fmax(cmax, chi);
      }
    }
  }
  pp.store(0);
  pp.load(plane(1));
  load_fine(0);
  T dmc[4] = {T(0), T(0), T(0), T(0)}, umc[4] = {T(0), T(0), T(0), T(0)};
  T y0[4], y1[4], y2[4], y3[4];  // Y of the coarse planes mm, mm-1, mm-2, mm-3
#pragma unroll
  for (int c = 0; c < 4; ++c) y0[c] = y1[c] = y2[c] = y3[c] = T(0);
  const bool oddij = ((i | j) & 1) != 0;
  lds_barrier();
#pragma unroll 1
  for (int mm = 0; mm < S; ++mm) {
    const int kc = 2 * mm - 2;  // coarse plane
    const int ko = kc - 3;      // odd fine plane whose prediction this plane completes
    const bool he = kc >= 0 && kc < BS, ho = ko >= 0 && ko < BS;
    pp.xpass(mm);
    if (mm + 1 < S) pp.store(mm + 1);
    T fe[4], fo[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      fe[c] = ue[c];
      fo[c] = uo[c];
    }
    if (mm + 2 < S) pp.load(plane(mm + 2));
    if (mm + 1 < S) load_fine(mm + 1);
    lds_barrier();
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      y3[c] = y2[c];
      y2[c] = y1[c];
      y1[c] = y0[c];
      y0[c] = pp.ypass(mm, c);
    }
    // z pass: the even fine plane kc and the odd fine plane kc - 3 (taps
    // kc-6, kc-4, kc-2, kc = coarse planes mm-3 .. mm)
    if (he) {
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        umc[c] = fmax(umc[c], fabs(fe[c]));
        if (oddij) dmc[c] = fmax(dmc[c], fabs(fe[c] - y0[c]));
      }
    }
    if (ho) {
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const T pr = w0 * y3[c] + w1 * y2[c] + w1 * y1[c] + w0 * y0[c];
        umc[c] = fmax(umc[c], fabs(fo[c]));
        dmc[c] = fmax(dmc[c], fabs(fo[c] - pr));
      }
    }
  }
  double v[10];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    v[c] = (double)wave_max(umc[c]);
    v[4 + c] = (double)wave_max(dmc[c]);
  }
  v[8] = wave_min(cmin);
  v[9] = wave_max(cmax);
  if ((tid & 63) == 0)
#pragma unroll
    for (int q = 0; q < 10; ++q) red[q][tid >> 6] = v[q];
  __syncthreads();
  if (tid < 10) {
    double r = red[tid][0];
    for (int w = 1; w < NT / 64; ++w) r = tid == 8 ? fmin(r, red[tid][w]) : fmax(r, red[tid][w]);
    red[tid][0] = r;
  }
  __syncthreads();
  if (tid < 8) part[ib * 8 + tid] = red[tid][0];
  if (tid == 0) mrange[ib] = p.mask ? red[9][0] - red[8][0] : 0.0;
}

// One workgroup: the field norms (max |u_c| over all blocks, 1 where a field
// vanishes) into norm, then per block the normalised detail maximum
// max_c max|d_c| / norm_c (equal to the maximum of the normalised details:
// scaling by a positive factor keeps the order) and the coarsening flag:
// 1 iff J > jmin and either dealiasing at J = jmax or the maximum is below
// eps with a constant mask.
__global__ __launch_bounds__(1024) void thr_finalize(const Tab* __restrict__ tab, int64_t nb,
                                                     const double* __restrict__ part,
                                                     const double* __restrict__ mrange,
                                                     double eps, int dealias, int jmin, int jmax,
                                                     double* __restrict__ norm,
                                                     double* __restrict__ dmax,
                                                     int8_t* __restrict__ flags) {
  __shared__ double red[4][1024 / 64];
  __shared__ double inv[4];
  const int tid = threadIdx.x;
  double mx[4] = {0, 0, 0, 0};
#pragma unroll 4
  for (int64_t q = tid; q < nb; q += blockDim.x)
#pragma unroll
    for (int c = 0; c < 4; ++c) mx[c] = fmax(mx[c], part[q * 8 + c]);
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const double v = wave_max(mx[c]);
    if ((tid & 63) == 0) red[c][tid >> 6] = v;
  }
  __syncthreads();
  if (tid < 4) {
    double r = red[tid][0];
    for (int w = 1; w < (int)blockDim.x / 64; ++w) r = fmax(r, red[tid][w]);
    const double nrm = r > 0.0 ? r : 1.0;
    norm[tid] = nrm;
    inv[tid] = 1.0 / nrm;
  }
  __syncthreads();
  for (int64_t q = tid; q < nb; q += blockDim.x) {
    double dm = 0.0;
#pragma unroll
    for (int c = 0; c < 4; ++c) dm = fmax(dm, part[q * 8 + 4 + c] * inv[c]);
    dmax[q] = dm;
    const int J = tab[q].meta[1];
    int f = 0;
    if (J > jmin) {
      if (dealias && J == jmax)
        f = 1;
      else if (dm < eps && mrange[q] == 0.0)
        f = 1;
    }
    flags[q] = (int8_t)f;
  }
}

// Wavelet filtering of a block at its own level: removing its details (Sec.
// 3.1) sets every interior point with an odd local index to P R u, the
// tensor-product DD4 prediction from the block's even lattice (ghost layers
// included); the even points are kept.  Only blocks of level `level` are
// filtered (every block if level < 0).  Same separable, z-marching passes as
// detail_kernel.  In place: the passes read only points whose three local
// indices are even, and the writes change only points with an odd index
// (all-even points are rewritten with their own value).
template <typename T, int BS>
__global__ __launch_bounds__(NT_GEN) void filter_kernel(const Tab* __restrict__ tab, int64_t nb,
                                                        T* U, Layout L, int level) {
  constexpr int S = BS / 2 + 3;  // even positions -2, 0, ..., bs+2
  constexpr int B2 = BS * BS;
  constexpr int NX = S * BS;                             // x-pass values per field and plane
  constexpr int KX = (4 * NX + NT_GEN - 1) / NT_GEN;     // x-pass values per thread
  constexpr int KQ = (B2 + NT_GEN - 1) / NT_GEN;         // (i, j) columns per thread
  __shared__ T xp[4 * NX];  // X(i, j', k') of the current coarse plane, 4 fields
  const T w0 = T(DDW0), w1 = T(DDW1);
  const int tid = threadIdx.x;
  const int P = L.P, ng = L.ng;
  for (int64_t ib = blockIdx.x; ib < nb; ib += gridDim.x) {
    const int32_t* m = tab[ib].meta;
    const int slot = m[0], J = m[1];
    if (level >= 0 && J != level) continue;  // uniform over the workgroup
    T* b = U + (int64_t)slot * L.bstride;
    auto ix = [&](int c, int i, int j, int k) -> int64_t {
      return c * L.fstride + ((int64_t)(k + ng) * P + (j + ng)) * P + (i + ng);
    };
    // Y(i, j, k') of this thread's columns for the last 4 coarse planes
    // (oldest first), all 4 fields, in registers
    T ring[KQ][4][4] = {};
    for (int mm = 0; mm < S; ++mm) {
      const int kc = 2 * mm - 2;  // coarse plane
      __syncthreads();            // xp is free again
      // x pass on the coarse rows j' = 2 jj - 2 of plane kc, 4 fields
#pragma unroll 2
      for (int kx = 0; kx < KX; ++kx) {
        const int it = tid + kx * NT_GEN;
        if (it < 4 * NX) {
          const int c = it / NX, q = it - c * NX;
          const int jj = q / BS, i = q - jj * BS, jc = 2 * jj - 2;
          T v;
          if ((i & 1) == 0)
            v = b[ix(c, i, jc, kc)];
          else
            v = w0 * b[ix(c, i - 3, jc, kc)] + w1 * b[ix(c, i - 1, jc, kc)] +
                w1 * b[ix(c, i + 1, jc, kc)] + w0 * b[ix(c, i + 3, jc, kc)];
          xp[it] = v;
        }
      }
      __syncthreads();
      // y pass into the ring, z pass: the even fine plane kc (the whole plane
      // is stored, so that its rows are written as whole lines: at points
      // with i and j even Y is the point itself, copied through both passes
      // without arithmetic) and the odd fine plane kc - 3
#pragma unroll
      for (int kq = 0; kq < KQ; ++kq) {
        const int q = tid + kq * NT_GEN;
        if (q < B2) {
          const int j = q / BS, i = q - j * BS;
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            const T* xc = xp + c * NX;
            T y;
            if ((j & 1) == 0) {
              y = xc[(j / 2 + 1) * BS + i];
            } else {
              const int jj = (j - 3) / 2 + 1;  // coarse row of j - 3
              y = w0 * xc[jj * BS + i] + w1 * xc[(jj + 1) * BS + i] + w1 * xc[(jj + 2) * BS + i] +
                  w0 * xc[(jj + 3) * BS + i];
            }
            if (kc >= 0 && kc < BS) b[ix(c, i, j, kc)] = y;
            const int ko = kc - 3;
            if (ko >= 0 && ko < BS)
              b[ix(c, i, j, ko)] = w0 * ring[kq][c][1] + w1 * ring[kq][c][2] +
                                   w1 * ring[kq][c][3] + w0 * y;
            ring[kq][c][0] = ring[kq][c][1];
            ring[kq][c][1] = ring[kq][c][2];
            ring[kq][c][2] = ring[kq][c][3];
            ring[kq][c][3] = y;
          }
        }
      }
    }
  }
}

// --------------------------------------------------------------------------
// refinement (prediction into 8 children) and coarsening (decimation)
// --------------------------------------------------------------------------
// Refinement (Sec. 3.1 prediction, Sec. 3.5): child octant oct of a
// ghost-synchronised parent.  Child point (i, j, k) is the parent's fine-grid
// point Q = off + (i, j, k), off = octant offset (0 or bs per axis); even Q
// copy the parent point Q/2, odd Q use the DD4 taps (Q-3)/2 .. (Q+3)/2 (the
// parent's ghost layers included).  Separable and z-marching as in
// detail_kernel, 4 fields together, one workgroup per child: x and y passes of
// each parent plane through LDS, a ring of 4 planes per column in registers, z
// pass for the child planes the ring completes.  Bound: the child's writes
// (5216 children of 16^3, FP64: 635 -> 470 us; with one field at a time each
// plane waited for its loads behind 3 barriers, and rows were written in part).
template <typename T, int BS>
__global__ __launch_bounds__(BS* BS) void prolong_kernel(const int32_t* __restrict__ list,
                                                         int64_t n, T* U, Layout L) {
  constexpr int S = BS / 2 + 4;  // parent points off/2 - 2 .. off/2 + bs/2 + 1
  using PP = PredictPlanes<T, BS, S, 2>;
  __shared__ T raw[2][4 * PP::S2], xp[2][4 * PP::NX];
  const T w0 = T(DDW0), w1 = T(DDW1);
  const int P = L.P, ng = L.ng, P2 = P * P, fs = (int)L.fstride;
  for (int64_t w = blockIdx.x; w < n; w += gridDim.x) {
    const int32_t ps = list[3 * w], cs = list[3 * w + 1], oct = list[3 * w + 2];
    const int h0 = (oct & 1) * (BS / 2) - 2, h1 = ((oct >> 1) & 1) * (BS / 2) - 2,
              h2 = ((oct >> 2) & 1) * (BS / 2) - 2;  // first parent index per axis
    const T* __restrict__ par = U + (int64_t)ps * L.bstride;
    T* __restrict__ ch = U + (int64_t)cs * L.bstride;
    PP pp(raw, xp, P, fs, (h1 + ng) * P + (h0 + ng), 1);
    const int col = (pp.j + ng) * P + (pp.i + ng);
    // the x-ghost columns of each row are cleared too, so that whole cache
    // lines are written (a child's ghost layers carry no values yet)
    const int gx = pp.i < ng ? -ng : (pp.i >= BS - ng ? ng : 0);
    auto plane = [&](int mm) { return par + (h2 + mm + ng) * P2; };
    pp.load(plane(0));
    T y0[4], y1[4], y2[4], y3[4];  // parent planes mm, mm-1, mm-2, mm-3
#pragma unroll
    for (int c = 0; c < 4; ++c) y0[c] = y1[c] = y2[c] = y3[c] = T(0);
    lds_barrier();  // the last child's planes are no longer read
    pp.store(0);
    pp.load(plane(1));
    lds_barrier();
#pragma unroll 1
    for (int mm = 0; mm < S; ++mm) {
      pp.xpass(mm);
      if (mm + 1 < S) pp.store(mm + 1);
      if (mm + 2 < S) pp.load(plane(mm + 2));
      lds_barrier();
      // z pass: child plane k even uses plane mm = 2 + k/2; k odd uses planes
      // 1 + (k-1)/2 .. 4 + (k-1)/2, complete when mm = 4 + (k-1)/2
      const int ke = 2 * (mm - 2), ko = 2 * (mm - 4) + 1;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        y3[c] = y2[c];
        y2[c] = y1[c];
        y1[c] = y0[c];
        y0[c] = pp.ypass(mm, c);
      }
      if (ke >= 0 && ke < BS)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          ch[c * fs + col + (ke + ng) * P2] = y0[c];
          if (gx) ch[c * fs + col + gx + (ke + ng) * P2] = T(0);
        }
      if (ko >= 0 && ko < BS)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          ch[c * fs + col + (ko + ng) * P2] = w0 * y3[c] + w1 * y2[c] + w1 * y1[c] + w0 * y0[c];
          if (gx) ch[c * fs + col + gx + (ko + ng) * P2] = T(0);
        }
    }
  }
}

template <typename T>
__global__ __launch_bounds__(NT_GEN) void decimate_kernel(const int32_t* __restrict__ list,
                                                          int64_t n, T* __restrict__ U, Layout L,
                                                          int bs) {
  const int n3 = bs * bs * bs;
  for (int64_t w = blockIdx.x; w < n; w += gridDim.x) {
    const int32_t* e = list + 10 * w;
    T* par = U + (int64_t)e[0] * L.bstride;
    for (int q = threadIdx.x; q < n3; q += blockDim.x) {
      const int i = q % bs, j = (q / bs) % bs, k = q / (bs * bs);
      const int ci = 2 * i >= bs, cj = 2 * j >= bs, ck = 2 * k >= bs;
      const T* ch = U + (int64_t)e[1 + ci + 2 * cj + 4 * ck] * L.bstride;
      const int64_t os = ((int64_t)(2 * k - ck * bs + L.ng) * L.P + (2 * j - cj * bs + L.ng)) *
                             L.P +
                         (2 * i - ci * bs + L.ng);
      const int64_t od = ((int64_t)(k + L.ng) * L.P + (j + L.ng)) * L.P + (i + L.ng);
      for (int c = 0; c < 4; ++c) par[od + c * L.fstride] = ch[os + c * L.fstride];
    }
  }
}

// --------------------------------------------------------------------------
// blocks without penalization
// --------------------------------------------------------------------------
// Two kernels: pen_flags marks each active block (1: far, 0: not), one
// thread per block; pen_compact, one workgroup of 1024 threads, writes
// list = the far blocks (active order), then the others, and cnt = {far
// count, other count}: each thread takes a contiguous run of flags, counts,
// and places its blocks after a workgroup prefix sum of the counts, so that
// each part keeps the active (Morton) order.  With t_dev given, the plate is
// classified for the pitch angles of the window [t, t + dt] of one step;
// else for every angle.
__global__ __launch_bounds__(NT_GEN) void pen_flags(const Tab* __restrict__ tab, int64_t nb,
                                                    wacm_params p, double L, int bs,
                                                    const double* __restrict__ t_dev,
                                                    const double* __restrict__ dt_dev,
                                                    int8_t* __restrict__ flag) {
  const int64_t b = (int64_t)blockIdx.x * NT_GEN + threadIdx.x;
  if (b >= nb) return;
  PitchWindow win{1.0, 0.0, 0.0, false};
  if (t_dev) win = pitch_window(p, *t_dev, *t_dev + *dt_dev);
  flag[b] = pen_far(p, L, bs, tab[b].meta, win) ? 1 : 0;
}

__global__ __launch_bounds__(1024) void pen_compact(const int8_t* __restrict__ flag, int64_t nb,
                                                    int32_t* __restrict__ list,
                                                    int32_t* __restrict__ cnt) {
  __shared__ int32_t wsum[2][16], woff[2][16], tot;
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int64_t per = (nb + 1023) / 1024;
  const int64_t b0 = t * per < nb ? t * per : nb, b1 = b0 + per < nb ? b0 + per : nb;
  int32_t nf = 0;
  for (int64_t b = b0; b < b1; ++b) nf += flag[b];
  const int32_t nn = (int32_t)(b1 - b0) - nf;
  // inclusive scans within the wave, then over the 16 waves' totals
  int32_t sf = nf, sn = nn;
  for (int o = 1; o < 64; o <<= 1) {
    const int32_t xf = __shfl_up(sf, o), xn = __shfl_up(sn, o);
    if (lane >= o) {
      sf += xf;
      sn += xn;
    }
  }
  if (lane == 63) {
    wsum[0][wv] = sf;
    wsum[1][wv] = sn;
  }
  __syncthreads();
  if (t == 0) {
    int32_t af = 0, an = 0;
    for (int w = 0; w < 16; ++w) {
      woff[0][w] = af;
      woff[1][w] = an;
      af += wsum[0][w];
      an += wsum[1][w];
    }
    tot = af;
    cnt[0] = af;
    cnt[1] = an;
  }
  __syncthreads();
  int32_t of = woff[0][wv] + sf - nf, on = tot + woff[1][wv] + sn - nn;
  for (int64_t b = b0; b < b1; ++b) {
    if (flag[b])
      list[of++] = (int32_t)b;
    else
      list[on++] = (int32_t)b;
  }
}

// the two lists of blocks with and without penalization, in list/cnt
static hipError_t pen_classify(const wacm_grid* g, const wacm_params* p, const double* t_dev,
                               const double* dt_dev, int32_t* list, int32_t* cnt,
                               int8_t* flag, hipStream_t st) {
  const unsigned nwg = (unsigned)((g->nb + NT_GEN - 1) / NT_GEN);
  if (nwg > 0) {
    pen_flags<<<nwg, NT_GEN, 0, st>>>(g->d_tab, g->nb, *p, g->d.L, g->d.bs, t_dev, dt_dev, flag);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  pen_compact<<<1, 1024, 0, st>>>(flag, g->nb, list, cnt);
  return hipGetLastError();
}

// --------------------------------------------------------------------------
// launchers
// --------------------------------------------------------------------------
// Records an event pair around the launches in its scope when profiling is on.
class ProfScope {
 public:
  ProfScope(const wacm_grid* g, int cls, hipStream_t st) : g_(g), st_(st) {
    if (!g_->prof.on) return;
    Profiler& p = g_->prof;
    if (p.recs.size() >= 4096) (void)profile_flush(g_);
    hipEvent_t e[2];
    for (int i = 0; i < 2; ++i) {
      if (!p.spare.empty()) {
        e[i] = p.spare.back();
        p.spare.pop_back();
      } else if (hipEventCreate(&e[i]) != hipSuccess) {
        e[i] = nullptr;
      }
    }
    if (!e[0] || !e[1]) return;
    rec_ = {cls, e[0], e[1]};
    active_ = hipEventRecord(e[0], st_) == hipSuccess;
  }
  ~ProfScope() {
    if (!active_) return;
    if (hipEventRecord(rec_.b, st_) == hipSuccess) g_->prof.recs.push_back(rec_);
  }

 private:
  const wacm_grid* g_;
  hipStream_t st_;
  Profiler::Rec rec_{};
  bool active_ = false;
};

hipError_t profile_flush(const wacm_grid* g) {
  Profiler& p = g->prof;
  hipError_t err = hipSuccess;
  for (const auto& r : p.recs) {
    float ms = 0.f;
    hipError_t e = hipEventSynchronize(r.b);
    if (e == hipSuccess) e = hipEventElapsedTime(&ms, r.a, r.b);
    if (e == hipSuccess) {
      p.ms[r.cls] += ms;
      p.n[r.cls] += 1;
    } else {
      err = e;
    }
    p.spare.push_back(r.a);
    p.spare.push_back(r.b);
  }
  p.recs.clear();
  return err;
}

static Layout pool_layout(const wacm_grid* g) {
  Layout L;
  L.P = g->P;
  L.ng = g->d.ng;
  L.fstride = (int64_t)g->P * g->P * g->P;
  L.bstride = 4 * L.fstride;
  return L;
}
static Layout compact_layout(const wacm_grid* g) {
  Layout L;
  L.P = g->d.bs;
  L.ng = 0;
  L.fstride = (int64_t)g->d.bs * g->d.bs * g->d.bs;
  L.bstride = 4 * L.fstride;
  return L;
}

// the stage inputs between stages: compact, x-split
static Layout split_layout(const wacm_grid* g) {
  Layout L = compact_layout(g);
  L.xs = 1;
  return L;
}

static unsigned grid_for(int64_t n, int per_cu) {
  int64_t cap = (int64_t)num_cus() * per_cu;
  return (unsigned)(n < cap ? (n > 0 ? n : 1) : cap);
}

// The face-halo kernel follows the stage kernel's XCD mapping: with work
// counters (q) it takes its faces from a second set of them.
template <typename T>
static hipError_t nlface_launch(const wacm_grid* g, const T* in, const Layout& Lin, T* hb,
                                int* q, hipStream_t st) {
  const unsigned grid = grid_for(g->n_cface, 8);
  if (q) {
    queue_clear<<<1, 8 * QSTRIDE, 0, st>>>(q);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  switch (g->d.bs) {
    case 16:
      nlface_kernel<T, 16><<<grid, NT_GEN, 0, st>>>(g->d_tab, g->d_cface, g->n_cface, in, Lin, hb, q);
      break;
    case 24:
      nlface_kernel<T, 24><<<grid, NT_GEN, 0, st>>>(g->d_tab, g->d_cface, g->n_cface, in, Lin, hb, q);
      break;
    case 32:
      nlface_kernel<T, 32><<<grid, NT_GEN, 0, st>>>(g->d_tab, g->d_cface, g->n_cface, in, Lin, hb, q);
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// work buffer: acc, ping, pong (compact, bs^3 per field) and the coarse-face
// halo buffer (6 faces x 4 fields x 3 x bs^2 per slot), 256-byte aligned parts
struct WorkParts {
  size_t acc, ping, pong, uc, hb, total;
};
static WorkParts work_parts(const wacm_grid* g) {
  const size_t es = g->d.dtype == WACM_F64 ? 8 : 4;
  const size_t cap = (size_t)g->d.capacity;
  const size_t b3 = (size_t)g->d.bs * g->d.bs * g->d.bs, b2 = (size_t)g->d.bs * g->d.bs;
  auto up = [](size_t v) { return (v + 255) / 256 * 256; };
  WorkParts w;
  w.acc = 0;
  w.ping = up(cap * 4 * b3 * es);
  w.pong = w.ping + up(cap * 4 * b3 * es);
  w.uc = w.pong + up(cap * 4 * b3 * es);
  w.hb = w.uc + up(cap * 4 * b3 * es);
  w.total = w.hb + up(cap * 6 * 4 * 3 * b2 * es);
  return w;
}

size_t work_bytes(const wacm_grid* g) { return work_parts(g).total; }

// Many workgroups of few regions each: faces, edges and corners differ 16-fold
// in work, and what a fixed share of them leaves uneven costs 18% (8 workgroups
// per CU: 486 us and 370 us in place of the figures above).
template <typename T, int BS>
static void sync_coarser_launch(const wacm_grid* g, T* U, hipStream_t st) {
  sync_coarser_kernel<T, BS><<<grid_for(g->n_cregion, 64), NT_GEN, 0, st>>>(
      g->d_tab, g->d_cregion, g->n_cregion, U, pool_layout(g));
}

// Full ghost fill: point-wise for same-level and finer regions, and the
// separable region kernel for regions in a coarser leaf.
template <typename T>
static hipError_t sync_t(const wacm_grid* g, T* U, hipStream_t st) {
  if (g->nb == 0) return hipSuccess;
  const bool split = g->d.ng <= SC_MAXG && g->n_cregion > 0;
  sync_kernel<T><<<grid_for(g->nb, 8), NT_GEN, 0, st>>>(g->d_tab, g->nb, U, pool_layout(g),
                                                        g->d.bs, split ? 1 : 0, nullptr);
  if (split) {
    switch (g->d.bs) {
      case 16:
        sync_coarser_launch<T, 16>(g, U, st);
        break;
      case 24:
        sync_coarser_launch<T, 24>(g, U, st);
        break;
      case 32:
        sync_coarser_launch<T, 32>(g, U, st);
        break;
      default:
        return hipErrorInvalidValue;
    }
  }
  return hipGetLastError();
}

template <typename T>
static hipError_t sync_lattice_t(const wacm_grid* g, T* U, hipStream_t st) {
  if (g->nb == 0) return hipSuccess;
  const unsigned grid = grid_for(g->nb, 8);
  const Layout L = pool_layout(g);
  switch (g->d.bs) {
    case 16:
      sync_lattice_kernel<T, 16><<<grid, NT_GEN, 0, st>>>(g->d_tab, g->nb, U, L);
      break;
    case 24:
      sync_lattice_kernel<T, 24><<<grid, NT_GEN, 0, st>>>(g->d_tab, g->nb, U, L);
      break;
    case 32:
      sync_lattice_kernel<T, 32><<<grid, NT_GEN, 0, st>>>(g->d_tab, g->nb, U, L);
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_sync_lattice(const wacm_grid* g, void* U, hipStream_t st) {
  return g->d.dtype == WACM_F64 ? sync_lattice_t(g, (double*)U, st)
                                : sync_lattice_t(g, (float*)U, st);
}

// The CDF 4/0 phase of a lifted stage's sync: the read boxes of regions in a
// finer leaf (what the face-star lifted values read there from a block's
// padded array) and every region in a coarser leaf (whole, by the region
// kernel); the stage and the lifted values read same-level values in place,
// and the lifted phase writes the finer face halos.
template <typename T>
static hipError_t sync_lifted_stage_t(const wacm_grid* g, T* U, const int32_t* box,
                                      hipStream_t st) {
  if (g->nb == 0) return hipSuccess;
  if (g->d.ng > SC_MAXG || !box) return sync_t(g, U, st);
  // one level only: where a region lies in a finer leaf, that leaf sees the block
  // as a coarser one
  if (g->n_cregion == 0) return hipSuccess;
  sync_kernel<T><<<grid_for(g->nb, 8), NT_GEN, 0, st>>>(g->d_tab, g->nb, U, pool_layout(g),
                                                        g->d.bs, 1, box);
  switch (g->d.bs) {
    case 16:
      sync_coarser_launch<T, 16>(g, U, st);
      break;
    case 24:
      sync_coarser_launch<T, 24>(g, U, st);
      break;
    case 32:
      sync_coarser_launch<T, 32>(g, U, st);
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_sync_lifted_stage(const wacm_grid* g, void* U, const int32_t* box,
                                    hipStream_t st) {
  return g->d.dtype == WACM_F64 ? sync_lifted_stage_t(g, (double*)U, box, st)
                                : sync_lifted_stage_t(g, (float*)U, box, st);
}

hipError_t launch_sync(const wacm_grid* g, void* U, hipStream_t st) {
  return g->d.dtype == WACM_F64 ? sync_t(g, (double*)U, st) : sync_t(g, (float*)U, st);
}

// The second set of work counters, for the face-halo kernel.
template <typename T>
static int* face_queue(const StageArgs<T>& a) {
  return a.queue ? a.queue + 8 * QSTRIDE : nullptr;
}

// Room for a call's own work counters in its work buffer: the halo of a face
// next to a leaf of the same level is read in place and never stored.  -1: none.
static int64_t spare_face(const wacm_grid* g) {
  for (const Tab& t : g->h_tab)
    for (int f = 0; f < 6; ++f)
      if (t.kind[FACE_REGION[f]] == 0) return (int64_t)t.meta[0] * 6 + f;
  return -1;
}

template <typename T>
static StageArgs<T> base_args(const wacm_grid* g, const wacm_params* p) {
  StageArgs<T> a{};
  a.tab = g->d_tab;
  a.nb = g->nb;
  a.L = g->d.L;
  a.xcd_map = g->sched.xcd_map < 0 ? 1 : g->sched.xcd_map;
  a.queue = g->sched.xcd_map == 2 ? g->d_queue : nullptr;
  a.nt = g->sched.nontemporal;
  a.kscale = 1.0;
  a.p = *p;
  return a;
}

// One RK stage s (1..4) of the fused kernel for the lifted-wavelet step:
// input, U^n and output in the padded pool layout, the accumulator compact
// (bs^3 values per field, from the start of its padded-size register); same-level
// halos from the neighbours' interiors, the halos of faces next to another
// level from the input's own ghost layers (filled before each stage), no
// face-halo buffer.  Tiles of 8 rows; early epilogue loads for FP32.
template <typename T>
static hipError_t stage_owng_t(const wacm_grid* g, const wacm_params* p, int s,
                               const double* t_dev, const double* dt_dev, const T* in, T* un,
                               T* out, T* acc, const T* dus, hipStream_t st) {
  if (g->nb == 0) return hipSuccess;
  StageArgs<T> a = base_args<T>(g, p);
  const Layout L = pool_layout(g);
  a.in = in;
  a.Lin = L;
  a.un = un;
  a.Lun = L;
  a.out = out;
  a.Lout = L;
  // the accumulator is never synchronised: compact, [c][z][y][x]
  a.acc = acc;
  a.Lacc.P = g->d.bs;
  a.Lacc.ng = 0;
  a.Lacc.fstride = (int64_t)g->d.bs * g->d.bs * g->d.bs;
  a.Lacc.bstride = 4 * a.Lacc.fstride;
  a.Lacc.xs = 0;
  a.dus = dus;
  a.t_dev = t_dev;
  a.dt_dev = dt_dev;
  return stage_run<T>(10 + s, g->d.bs, a, g->sched, st);
}

hipError_t launch_stage_owng(const wacm_grid* g, const wacm_params* p, int s,
                             const double* t_dev, const double* dt_dev, const void* in, void* un,
                             void* out, void* acc, const void* dus, hipStream_t st) {
  return g->d.dtype == WACM_F64
             ? stage_owng_t(g, p, s, t_dev, dt_dev, (const double*)in, (double*)un,
                            (double*)out, (double*)acc, (const double*)dus, st)
             : stage_owng_t(g, p, s, t_dev, dt_dev, (const float*)in, (float*)un, (float*)out,
                            (float*)acc, (const float*)dus, st);
}

template <typename T>
static hipError_t rhs_t(const wacm_grid* g, const wacm_params* p, double t, const T* U, T* dU,
                        const T* dus, hipStream_t st) {
  if (g->nb == 0) return hipSuccess;
  StageArgs<T> a = base_args<T>(g, p);
  a.in = U;
  a.Lin = pool_layout(g);
  a.out = dU;
  a.Lout = pool_layout(g);
  a.un = dU;
  a.Lun = pool_layout(g);
  a.acc = dU;
  a.Lacc = pool_layout(g);
  a.dus = dus;
  a.t_host = t;
  return stage_run<T>(0, g->d.bs, a, rhs_schedule(g->sched), st);
}

hipError_t launch_rhs(const wacm_grid* g, const wacm_params* p, double t, const void* U,
                      void* dU, const void* dus, hipStream_t st) {
  return g->d.dtype == WACM_F64
             ? rhs_t(g, p, t, (const double*)U, (double*)dU, (const double*)dus, st)
             : rhs_t(g, p, t, (const float*)U, (float*)dU, (const float*)dus, st);
}

template <typename T>
static hipError_t dt_t(const wacm_grid* g, const wacm_params* p, const T* U, double* dt_dev,
                       hipStream_t st) {
  if (g->nb == 0) return hipSuccess;
  const unsigned grid = grid_for(g->nb, 8);
  switch (g->d.bs) {
    case 16:
      maxu_kernel<T, 16><<<grid, NT_GEN, 0, st>>>(g->d_tab, g->nb, U, pool_layout(g), g->d_part);
      break;
    case 24:
      maxu_kernel<T, 24><<<grid, NT_GEN, 0, st>>>(g->d_tab, g->nb, U, pool_layout(g), g->d_part);
      break;
    case 32:
      maxu_kernel<T, 32><<<grid, NT_GEN, 0, st>>>(g->d_tab, g->nb, U, pool_layout(g), g->d_part);
      break;
    default:
      return hipErrorInvalidValue;
  }
  const double hmin = g->d.L / (double(int64_t(1) << g->jfine) * g->d.bs);
  dt_finalize<<<1, NT_GEN, 0, st>>>(g->d_part, g->nb, *p, hmin, dt_dev, nullptr);
  return hipGetLastError();
}

hipError_t launch_dt(const wacm_grid* g, const wacm_params* p, const void* U, double* dt_dev,
                     hipStream_t st) {
  return g->d.dtype == WACM_F64 ? dt_t(g, p, (const double*)U, dt_dev, st)
                                : dt_t(g, p, (const float*)U, dt_dev, st);
}

// nsteps classical RK4 steps.  With the CFL rule, the first step's dt comes
// from a reduction over U; every later step's from the maximum the previous
// step's last stage formed while writing U (the same value, bit for bit).
// Between the steps of one call the state stays in the x-split register uc:
// only the first step reads the pool and only the last one writes it.
// Whether to split the blocks of a penalized stage (schedule pen_split: 0
// never, 2 always, 1 when it pays).  Two launches per stage and their tails
// cost more than the unpenalized kernel saves on small grids: the split
// needs at least 2048 active blocks, and, for a static mask or sponge, at
// least 512 blocks without penalization (counted here from the host copy of
// the tables).  A pitching plate's per-step lists leave only the blocks near
// the plate penalized, so its grids need only the size.
static bool pen_split_pays(const wacm_grid* g, const wacm_params* p) {
  if (g->sched.pen_split != 1) return g->sched.pen_split == 2;
  if (g->nb < 2048) return false;
  if (p->mask == WACM_MASK_PLATE) return true;
  const PitchWindow any{1.0, 0.0, 0.0, false};
  int64_t nfar = 0;
  for (int64_t b = 0; b < g->nb && nfar < 512; ++b)
    nfar += pen_far(*p, g->d.L, g->d.bs, g->h_tab[b].meta, any) ? 1 : 0;
  return nfar >= 512;
}

// A stage input of one RK4 step recomputed from U^n, for the adjoint: s = 1
// Y2 = U^n + dt/2 rhs(U^n), 2 Y3 = U^n + dt/2 rhs(Y2), 3 Y4 = U^n + dt
// rhs(Y3); `in` is the input's predecessor (U^n in the pool layout for s = 1,
// else x-split), out x-split, hb the face-halo buffer.
template <typename T>
static hipError_t stage_input_t(const wacm_grid* g, const wacm_params* p, int s, double t,
                                double dt, const T* un, const T* in, T* out, T* hb, const T* dus,
                                hipStream_t st) {
  StageArgs<T> a = base_args<T>(g, p);
  a.in = in;
  a.Lin = s == 1 ? pool_layout(g) : split_layout(g);
  a.hb = hb;
  a.un = const_cast<T*>(un);
  a.Lun = pool_layout(g);
  a.out = out;
  a.Lout = split_layout(g);
  a.dus = dus;
  a.t_host = t;
  a.dt_host = dt;
  a.kscale = s == 2 ? 0.5 : 1.0;
  if (g->n_cface > 0)
    if (hipError_t e = nlface_launch<T>(g, in, a.Lin, hb, face_queue(a), st); e != hipSuccess)
      return e;
  return stage_run<T>(s == 1 ? 1 : 3, g->d.bs, a,
                      stage_schedule(g->sched, sizeof(T) == 8, g->d.bs, g->nb, false), st);
}

hipError_t launch_stage_input(const wacm_grid* g, const wacm_params* p, int s, double t,
                              double dt, const void* un, const void* in, void* out, void* hb,
                              const void* dus, hipStream_t st) {
  return g->d.dtype == WACM_F64
             ? stage_input_t(g, p, s, t, dt, (const double*)un, (const double*)in, (double*)out,
                             (double*)hb, (const double*)dus, st)
             : stage_input_t(g, p, s, t, dt, (const float*)un, (const float*)in, (float*)out,
                             (float*)hb, (const float*)dus, st);
}

hipError_t launch_nlface(const wacm_grid* g, const void* in, const Layout& Lin, void* hb,
                         hipStream_t st) {
  if (g->n_cface == 0) return hipSuccess;
  int* q = g->sched.xcd_map == 2 ? g->d_queue + 8 * QSTRIDE : nullptr;
  return g->d.dtype == WACM_F64
             ? nlface_launch<double>(g, (const double*)in, Lin, (double*)hb, q, st)
             : nlface_launch<float>(g, (const float*)in, Lin, (float*)hb, q, st);
}

template <typename T>
static hipError_t rk4_t(const wacm_grid* g, const wacm_params* p, double* t_dev, double* dt_dev,
                        T* U, void* work, const T* dus, int dt_mode, int64_t nsteps,
                        hipStream_t st) {
  if (g->nb == 0) return hipSuccess;
  hipError_t e;
  const WorkParts wp = work_parts(g);
  char* w = (char*)work;
  T* acc = (T*)(w + wp.acc);
  T* ping = (T*)(w + wp.ping);
  T* pong = (T*)(w + wp.pong);
  T* uc = (T*)(w + wp.uc);
  T* hb = (T*)(w + wp.hb);
  StageArgs<T> a = base_args<T>(g, p);
  a.acc = acc;
  a.Lacc = compact_layout(g);
  a.hb = hb;
  a.dus = dus;
  a.t_dev = t_dev;
  a.dt_dev = dt_dev;
  const Layout Lp = pool_layout(g), Ls = split_layout(g);
  T* ins[4] = {U, ping, pong, ping};
  T* outs[4] = {ping, pong, ping, U};
  Layout lins[4] = {Lp, Ls, Ls, Ls};
  const bool f64 = sizeof(T) == 8;
  const int64_t face = large_grid(f64, g->d.bs, g->nb) ? spare_face(g) : -1;
  const wacm_schedule sched = stage_schedule(g->sched, f64, g->d.bs, g->nb, face >= 0);
  if (sched.xcd_map == XCD_OWN_COUNTERS) {
    // (not the grid's: fixed steps without penalization may overlap in time)
    a.queue = reinterpret_cast<int*>(hb + face * 12 * g->d.bs * g->d.bs);
    a.xcd_map = 2;
  }
  const double hmin = g->d.L / (double(int64_t(1) << g->jfine) * g->d.bs);
  int64_t nmax = 0;  // velocity maxima the last stage of the previous step left
  // blocks without penalization first (the adaptation lists are free
  // during a step: capacity entries of the list, then the 2 counts); a
  // pitching plate is classified per step, for the angles of that step
  const bool split = (p->mask || p->sponge || dus) && pen_split_pays(g, p);
  const bool split_step = split && p->mask == WACM_MASK_PLATE;
  int32_t* const plist = g->d_list;
  int32_t* const pcnt = g->d_list + g->d.capacity;
  int8_t* const pflag = reinterpret_cast<int8_t*>(g->d_list + g->d.capacity + 2);
  if (split) {
    a.blist = plist;
    a.bcnt = pcnt;
  }
  if (split && !split_step &&
      (e = pen_classify(g, p, nullptr, nullptr, plist, pcnt, pflag, st)) != hipSuccess)
    return e;
  for (int64_t k = 0; k < nsteps; ++k) {
    if (dt_mode == WACM_DT_CFL) {
      ProfScope ps(g, 0, st);
      if (k == 0) {
        if ((e = dt_t<T>(g, p, U, dt_dev, st)) != hipSuccess) return e;
      } else {
        dt_finalize<<<1, NT_GEN, 0, st>>>(g->d_part, nmax, *p, hmin, dt_dev, t_dev);
        if ((e = hipGetLastError()) != hipSuccess) return e;
      }
    }
    // U^n of this step and U^{n+1}: the pool at the ends of the call, uc between
    T* un = k == 0 ? U : uc;
    const Layout Lun = k == 0 ? Lp : Ls;
    T* unext = k + 1 == nsteps ? U : uc;
    const Layout Lnext = k + 1 == nsteps ? Lp : Ls;
    ins[0] = un;
    lins[0] = Lun;
    for (int s = 0; s < 4; ++s) {
      a.in = ins[s];
      a.Lin = lins[s];
      a.out = s == 3 ? unext : outs[s];
      a.Lout = s == 3 ? Lnext : Ls;
      a.un = s == 3 ? unext : un;
      a.Lun = s == 3 ? Lnext : Lun;
      a.umax_part = (s == 3 && dt_mode == WACM_DT_CFL && k + 1 < nsteps) ? g->d_part : nullptr;
      a.nmax = a.umax_part ? &nmax : nullptr;
      if (g->n_cface > 0) {
        ProfScope ps(g, 1, st);
        if ((e = nlface_launch<T>(g, a.in, a.Lin, hb, face_queue(a), st)) != hipSuccess) return e;
      }
      ProfScope ps(g, 2, st);
      if (s == 0 && split_step &&
          (e = pen_classify(g, p, t_dev, dt_dev, plist, pcnt, pflag, st)) != hipSuccess)
        return e;
      e = stage_run<T>(s + 1, g->d.bs, a, sched, st);
      if (e != hipSuccess) return e;
    }
    if (dt_mode == WACM_DT_CFL && k + 1 < nsteps) continue;  // by the next step's dt_finalize
    ProfScope ps(g, 3, st);
    advance_time<<<1, 64, 0, st>>>(t_dev, dt_dev);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_rk4(const wacm_grid* g, const wacm_params* p, double* t_dev, double* dt_dev,
                      void* U, void* work, const void* dus, int dt_mode, int64_t nsteps,
                      hipStream_t st) {
  return g->d.dtype == WACM_F64 ? rk4_t(g, p, t_dev, dt_dev, (double*)U, work,
                                        (const double*)dus, dt_mode, nsteps, st)
                                : rk4_t(g, p, t_dev, dt_dev, (float*)U, work, (const float*)dus,
                                        dt_mode, nsteps, st);
}

template <typename T, int BS>
static void diag_launch(const wacm_grid* g, const wacm_params* p, double t, const T* U,
                        const T* dus, hipStream_t st) {
  auto run = [&](auto kernel) {
    kernel<<<grid_for(g->nb, 8), NT_GEN, 0, st>>>(g->d_tab, g->nb, U, pool_layout(g), dus, g->d.L,
                                                  *p, t, g->d_part);
  };
  if (p->mask == WACM_MASK_PLATE)
    run(diag_kernel<T, BS, WACM_MASK_PLATE>);
  else if (p->mask)
    run(diag_kernel<T, BS, WACM_MASK_SPHERE>);
  else
    run(diag_kernel<T, BS, WACM_MASK_NONE>);
}

template <typename T>
static hipError_t diag_t(const wacm_grid* g, const wacm_params* p, double t, const T* U,
                         const T* dus, double* out, hipStream_t st) {
  if (g->nb == 0) return hipSuccess;
  switch (g->d.bs) {
    case 16:
      diag_launch<T, 16>(g, p, t, U, dus, st);
      break;
    case 24:
      diag_launch<T, 24>(g, p, t, U, dus, st);
      break;
    case 32:
      diag_launch<T, 32>(g, p, t, U, dus, st);
      break;
    default:
      return hipErrorInvalidValue;
  }
  diag_finalize<<<1, NT_GEN, 0, st>>>(g->d_part, g->nb, out);
  return hipGetLastError();
}

hipError_t launch_diag(const wacm_grid* g, const wacm_params* p, double t, const void* U,
                       const void* dus, double* out, hipStream_t st) {
  return g->d.dtype == WACM_F64
             ? diag_t(g, p, t, (const double*)U, (const double*)dus, out, st)
             : diag_t(g, p, t, (const float*)U, (const float*)dus, out, st);
}

template <typename T>
static hipError_t thr_t(const wacm_grid* g, const wacm_params* p, double t, const T* U,
                        double eps, int dealias, double* dmax, double* mrange, int8_t* flags,
                        hipStream_t st) {
  if (g->nb == 0) return hipSuccess;
  const Layout L = pool_layout(g);
  switch (g->d.bs) {
#define WACM_DETAIL(BSV)                                                                    \
  case BSV:                                                                                 \
    detail_kernel<T, BSV><<<(unsigned)g->nb, BSV * BSV, 0, st>>>(g->d_tab, g->nb, U, L,    \
                                                                  g->d.L, *p, t, g->d_part, \
                                                                  mrange);                  \
    break;
    WACM_DETAIL(16)
    WACM_DETAIL(24)
    WACM_DETAIL(32)
#undef WACM_DETAIL
    default:
      return hipErrorInvalidValue;
  }
  if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  thr_finalize<<<1, 1024, 0, st>>>(g->d_tab, g->nb, g->d_part, mrange, eps, dealias, g->d.jmin,
                                   g->d.jmax, g->d_norm, dmax, flags);
  return hipGetLastError();
}

hipError_t launch_threshold(const wacm_grid* g, const wacm_params* p, double t, const void* U,
                            double eps, int dealias, double* dmax, double* mrange,
                            int8_t* flags, hipStream_t st) {
  return g->d.dtype == WACM_F64
             ? thr_t(g, p, t, (const double*)U, eps, dealias, dmax, mrange, flags, st)
             : thr_t(g, p, t, (const float*)U, eps, dealias, dmax, mrange, flags, st);
}

template <typename T>
static hipError_t filter_t(const wacm_grid* g, T* U, int level, hipStream_t st) {
  if (g->nb == 0) return hipSuccess;
  const unsigned grid = grid_for(g->nb, 8);
  const Layout L = pool_layout(g);
  switch (g->d.bs) {
    case 16:
      filter_kernel<T, 16><<<grid, NT_GEN, 0, st>>>(g->d_tab, g->nb, U, L, level);
      break;
    case 24:
      filter_kernel<T, 24><<<grid, NT_GEN, 0, st>>>(g->d_tab, g->nb, U, L, level);
      break;
    case 32:
      filter_kernel<T, 32><<<grid, NT_GEN, 0, st>>>(g->d_tab, g->nb, U, L, level);
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_filter(const wacm_grid* g, void* U, int level, hipStream_t st) {
  return g->d.dtype == WACM_F64 ? filter_t(g, (double*)U, level, st)
                                : filter_t(g, (float*)U, level, st);
}

template <typename T>
static hipError_t prolong_t(const wacm_grid* g, T* U, int64_t n, hipStream_t st) {
  const unsigned grid = grid_for(n, 8);
  switch (g->d.bs) {
    case 16:
      prolong_kernel<T, 16><<<grid, 256, 0, st>>>(g->d_list, n, U, pool_layout(g));
      break;
    case 24:
      prolong_kernel<T, 24><<<grid, 576, 0, st>>>(g->d_list, n, U, pool_layout(g));
      break;
    case 32:
      prolong_kernel<T, 32><<<grid, 1024, 0, st>>>(g->d_list, n, U, pool_layout(g));
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_prolong(const wacm_grid* g, void* U, int64_t n, hipStream_t st) {
  if (n == 0) return hipSuccess;
  return g->d.dtype == WACM_F64 ? prolong_t(g, (double*)U, n, st)
                                : prolong_t(g, (float*)U, n, st);
}

// reductions shared with the two-dimensional path (kernels2d.hip)
hipError_t finalize_dt(const double* part, int64_t n, const wacm_params& p, double hmin,
                       double* dt_dev, double* t_dev, hipStream_t st) {
  dt_finalize<<<1, NT_GEN, 0, st>>>(part, n, p, hmin, dt_dev, t_dev);
  return hipGetLastError();
}
hipError_t finalize_diag(const double* part, int64_t n, double* out, hipStream_t st) {
  diag_finalize<<<1, NT_GEN, 0, st>>>(part, n, out);
  return hipGetLastError();
}
hipError_t finalize_norm(const double* part, int64_t n, double* norm, hipStream_t st) {
  norm_finalize<<<1, NT_GEN, 0, st>>>(part, n, norm);
  return hipGetLastError();
}
hipError_t add_dt_to_time(double* t_dev, const double* dt_dev, hipStream_t st) {
  advance_time<<<1, 64, 0, st>>>(t_dev, dt_dev);
  return hipGetLastError();
}

hipError_t launch_decimate(const wacm_grid* g, void* U, int64_t n, hipStream_t st) {
  if (n == 0) return hipSuccess;
  if (g->d.dtype == WACM_F64)
    decimate_kernel<double><<<grid_for(n, 8), NT_GEN, 0, st>>>(g->d_list, n, (double*)U,
                                                              pool_layout(g), g->d.bs);
  else
    decimate_kernel<float><<<grid_for(n, 8), NT_GEN, 0, st>>>(g->d_list, n, (float*)U,
                                                             pool_layout(g), g->d.bs);
  return hipGetLastError();
}

}  // namespace wacm
