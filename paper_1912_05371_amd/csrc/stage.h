// Device pieces shared by the kernels that march through a block's planes
// with a depth-3 halo: the fused rhs + RK stage and its adjoint.
#pragma once

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

}  // namespace wacm
