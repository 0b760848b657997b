// The fused rhs + RK stage kernel (Sec. 2.2-2.3) and its launchers.  Included by
// one source per element type, so that the instantiations compile in parallel.
#pragma once

#include <algorithm>

#include "resolve.h"
#include "schedule.h"
#include "stage.h"
#include "wacm_internal.h"

namespace wacm {

// MODE 0: dU = rhs(U) with U's own ghost layers.  MODE s = 1..4: classical
// RK4 stage s with registers U^n, W and the stage inputs Y_s:
//   s1: out = Y2 = U^n + dt/2 k1                    (input = U^n)
//   s2: out = Y3 = U^n + dt/2 k2,  W = (U^n + Y2)/3 + dt/3 k2
//   s3: out = Y4 = U^n + dt k3
//   s4: U^{n+1} = W + Y4/3 + dt/6 k4
// Since dt k1 = 2 (Y2 - U^n) and dt k3 = Y4 - U^n, the update
// U^n + dt/6 (k1 + 2 k2 + 2 k3 + k4) equals W + Y4/3 + dt/6 k4 with
// W = 2/3 U^n + dt/6 k1 + dt/3 k2: only stage 2 writes a second register and
// stages 3 and 4 read one besides their input (same values up to rounding of
// U^n's size).
// PEN: penalization/sponge terms present.  PREF: load the epilogue operands
// (U^n, acc) before the barrier instead of after the rhs.  Work items are
// tiles of TY rows of a block's (x,y) columns (TY = BS: the whole block), one
// persistent workgroup per item at a time, one thread per column marching in
// z: z-neighbours in a register queue, the x/y cross of the current plane in a
// double-buffered LDS slab, the next plane's loads issued before the barrier.
// Rows between tiles of one block are read from the block itself.
// Occupancy: FP64 tiles are held to 2 waves per SIMD, FP32 tiles to 3; a
// whole bs-16 block (4 waves) to 2 per SIMD, which keeps two workgroups per
// CU for the penalized FP64 variant at the cost of a few spills (measured
// faster than one workgroup per CU without spills).
// MODEX = MODE (0 rhs only, 1..4 RK stage) or 10 + MODE: the RK stage with
// every register in the padded pool layout, same-level halos read from the
// neighbours' interiors and the others from the input's own synchronised
// ghost layers (the lifted-wavelet step).
template <typename T, int BS, int TY, int MODEX, bool PEN, bool PREF, int NZ>
__global__ __launch_bounds__(BS* TY) __attribute__((amdgpu_waves_per_eu(TY == BS ? (BS == 16 ? 2 : 1) : (sizeof(T) == 8 ? 2 : 3))))
void stage_kernel(StageArgs<T> a) {
  constexpr int H = 3, W = BS + 2 * H, WY = TY + 2 * H, NT = BS * TY;
  constexpr int NTY = BS / TY, NH = 6 * TY + 6 * BS;
  constexpr int NPB = NTY * NZ, ZR = BS / NZ;  // items per block, planes per item
  static_assert(ZR >= 4 && (NZ == 1 || ZR % 2 == 0), "runs of planes");
  static_assert(NH <= NT || TY == BS, "halo points per plane exceed the threads");
  constexpr int MODE = MODEX % 10;
  constexpr bool OWNG = MODEX >= 10;
  constexpr int HALO = OWNG ? HALO_MIX : (MODE == 0 ? HALO_OWN : HALO_NB);
  // the stage registers between stages are x-split; U^n is the pool or, from
  // the second step of a multi-step call on, an x-split register too
  const bool xin = !OWNG && (MODE >= 2 || (MODE == 1 && a.Lin.xs != 0));
  const bool xun = MODE >= 2 && a.Lun.xs != 0;
  constexpr bool XOUT = !OWNG && MODE >= 1 && MODE <= 3;
  __shared__ T slab[2][4][W * WY];
  __shared__ FaceDesc<T> fds[6];
  __shared__ int32_t meta[6];
  __shared__ typename std::conditional<PEN, PlateTab<BS>, NoTab>::type ptab;
  __shared__ double red[NT / 64];
  __shared__ int qitem;
  const int tid = threadIdx.x;
  const int x = tid % BS, yl = tid / BS;
  const T a1 = T(TW1), a2 = T(TW2), a3 = T(TW3);
  const T c2a = T(D2A), c2b = T(D2B), c2c = T(D2C);
  auto lap1 = [&](T m2, T m1, T c0, T p1, T p2) {
    return fma(c2a, p2, fma(c2b, p1, fma(c2c, c0, fma(c2b, m1, c2a * m2))));
  };
  double tc = a.t_host, dt = 0.0;
  if (MODE != 0) {
    if (a.t_dev) tc = *a.t_dev;
    dt = a.dt_dev ? *a.dt_dev : a.dt_host;
  }
  const T nu = T(a.p.nu), c0sq = T(a.p.c0 * a.p.c0), cg = T(a.p.c_gamma);
  const T fA = T(MODE == 4 ? dt / 6.0 : dt / 3.0);  // k weight of W (s2) and of U^{n+1} (s4)
  // the stage time and what of the mask depends on it alone
  const double ts = tc + (MODE == 2 || MODE == 3 ? 0.5 * dt : (MODE == 4 ? dt : 0.0));
  const MaskTime mt = PEN && a.p.mask ? mask_time(a.p, ts) : MaskTime{1.0, 0.0, 0.0};
  const T fB = T(MODE == 3 ? a.kscale * dt : 0.5 * dt);
  const int fin = (int)a.Lin.fstride, Pi = a.Lin.P;
  const int cidx = (yl + H) * W + (x + H);
  // this thread's halo point of every plane (threads < NH): x-faces of the
  // tile's rows, then the 3 rows below and above the tile
  const bool hthr = tid < NH;
  int hkind = 0, hd = 0, hs = 0, hli = 0;  // hkind: 0..3 face x-,x+,below,above
  if (hthr) {
    if (tid < 6 * TY) {
      hkind = tid / (3 * TY);
      const int rem = tid - hkind * 3 * TY;
      hd = rem / TY;
      hs = rem - hd * TY;
      const int hx = hkind == 0 ? -1 - hd : BS + hd;
      hli = (hs + H) * W + (hx + H);
    } else {
      const int q = tid - 6 * TY;
      hkind = 2 + q / (3 * BS);
      const int rem = q - (hkind - 2) * 3 * BS;
      hd = rem / BS;
      hs = rem - hd * BS;
      const int hyl = hkind == 2 ? -1 - hd : TY + hd;
      hli = (hyl + H) * W + (hs + H);
    }
  }
  // plane steps of this thread's column
  const int zs = xin ? xsplit_zstride(BS, x) : Pi * Pi;
  const int azs = a.Lacc.P * a.Lacc.P, afs = (int)a.Lacc.fstride;
  const int uzs = xun ? xsplit_zstride(BS, x) : a.Lun.P * a.Lun.P, ufs = (int)a.Lun.fstride;
  const int ozs = XOUT ? xsplit_zstride(BS, x) : a.Lout.P * a.Lout.P;
  const int ofs = (int)a.Lout.fstride;

  // work items: static (round-robin or contiguous per XCD) or from the
  // per-XCD queues, whose next item thread 0 requests while the current one
  // is processed and publishes in qitem before the loop's first barrier
  int64_t nblk = a.nb, boff = 0;
  if (a.blist) {
    boff = a.bsel ? a.bcnt[0] : 0;
    nblk = a.bcnt[a.bsel];
  }
  const int64_t nitems = nblk * NPB;
  const bool dyn = a.queue != nullptr;
  BlockIter it(nitems, a.xcd_map);
  int qh = blockIdx.x & 7, qpend = 0;
  const int qchunk = (int)((nitems + 7) / 8);
  if (dyn && tid == 0) qitem = queue_take(a.queue, qh, qchunk, (int)nitems,
                                          atomicAdd(a.queue + qh * QSTRIDE, 1));
  for (;;) {
    lds_barrier();
    const int64_t item = dyn ? (int64_t)__builtin_amdgcn_readfirstlane(qitem) : it.ib;
    if (item >= (dyn ? nitems : it.end)) break;
    if (!dyn) it.ib += it.step;
    const int64_t il = item / NPB;
    const int64_t ibk = a.blist ? a.blist[boff + il] : il;
    const int tile = (int)(item - il * NPB);
    const int y0 = tile / NZ * TY;
    const int z0 = NZ == 1 ? 0 : __builtin_amdgcn_readfirstlane(tile % NZ * ZR);
    const int y = y0 + yl;
    if (tid < 6) fds[tid] = face_desc<T, BS, HALO>(a.tab[ibk], a.in, a.Lin, a.hb, tid, xin);
    if (tid < 5) meta[tid] = a.tab[ibk].meta[tid];
    lds_barrier();
    if (dyn && tid == 0) qpend = atomicAdd(a.queue + qh * QSTRIDE, 1);
    // offsets of this thread's column in the input, accumulator and U^n
    const int col = xin ? xsplit_offset(BS, x, y, 0)
                        : (a.Lin.ng * Pi + (y + a.Lin.ng)) * Pi + (x + a.Lin.ng);
    const int acol = (a.Lacc.ng * a.Lacc.P + (y + a.Lacc.ng)) * a.Lacc.P + (x + a.Lacc.ng);
    const int ucol = xun ? xsplit_offset(BS, x, y, 0)
                         : (a.Lun.ng * a.Lun.P + (y + a.Lun.ng)) * a.Lun.P + (x + a.Lun.ng);
    const int ocol = XOUT ? xsplit_offset(BS, x, y, 0)
                          : (a.Lout.ng * a.Lout.P + (y + a.Lout.ng)) * a.Lout.P + (x + a.Lout.ng);
    // uniform over the workgroup: scalar registers
    const int slot = __builtin_amdgcn_readfirstlane(meta[0]);
    const int J = __builtin_amdgcn_readfirstlane(meta[1]);
    const double hdd = a.L / (double(int64_t(1) << J) * BS);
    const T ih = T(1.0 / hdd), ih2 = T(1.0 / (hdd * hdd));
    const T* __restrict__ inb = a.in + (int64_t)slot * a.Lin.bstride + col;
    T* accb = a.acc + (int64_t)slot * a.Lacc.bstride + acol;
    T* unb = a.un + (int64_t)slot * a.Lun.bstride + ucol;
    T* outb = a.out + (int64_t)slot * a.Lout.bstride + ocol;
    // field c of this thread's column at depth d below (f = 4) or above
    // (f = 5) the block; the descriptor is re-read from LDS at each use
    auto zface = [&](int f, int d, int c) -> T {
      const FaceDesc<T>& fz = fds[f];
      if (xin && fz.mode == 1) return fz.ptr[c * fin + col + (f == 4 ? BS - 1 - d : d) * zs];
      return fz.ptr[c * fz.fs + d * fz.sd + x * fz.s0 + y * fz.s1];
    };
    // this thread's halo point as an affine map in z: hp[c hfs + z hzs]
    const T* hp = nullptr;
    int hfs = 0, hzs = 0;
    if (hthr) {
      if (hkind < 2) {
        const FaceDesc<T>& fh = fds[hkind];
        hp = fh.ptr + hd * fh.sd + (y0 + hs) * fh.s0;
        hfs = fh.fs;
        hzs = fh.s1;
      } else {
        const int hy = hkind == 2 ? y0 - 1 - hd : y0 + TY + hd;
        if (hy < 0 || hy >= BS) {
          const FaceDesc<T>& fh = fds[hy < 0 ? 2 : 3];
          if (xin && fh.mode == 1) {
            hp = fh.ptr + xsplit_offset(BS, hs, hy < 0 ? BS + hy : hy - BS, 0);
            hfs = fin;
            hzs = xsplit_zstride(BS, hs);
          } else {
            hp = fh.ptr + (hy < 0 ? -1 - hy : hy - BS) * fh.sd + hs * fh.s0;
            hfs = fh.fs;
            hzs = fh.s1;
          }
        } else if (xin) {
          hp = a.in + (int64_t)slot * a.Lin.bstride + xsplit_offset(BS, hs, hy, 0);
          hfs = fin;
          hzs = xsplit_zstride(BS, hs);
        } else {
          hp = a.in + (int64_t)slot * a.Lin.bstride +
               (a.Lin.ng * Pi + (hy + a.Lin.ng)) * Pi + (hs + a.Lin.ng);
          hfs = fin;
          hzs = Pi * Pi;
        }
      }
    }

    double m2 = 0.0;  // stage 4: max |u|^2 of this thread's new points
    // mask, solid velocity and sponge of this thread's point of the next
    // plane, evaluated at the end of the previous plane where fewer values
    // are live (the extra solid velocity loaded with the rhs's terms instead:
    // 134 registers spilled instead of 49, FP64 16^3)
    T pchi = T(0), psp = T(0), pus[3] = {T(0), T(0), T(0)}, pdu[3];
    int reach = 0;  // whether the mask (1) and the sponge (2) reach this block
    bool masked = false, sponged = false;
    auto pen_at = [&](int zz) {
      if (!reach) return;
      const double xg = (double)(meta[2] * BS + x) * hdd, yg = (double)(meta[3] * BS + y) * hdd,
                   zg = (double)(meta[4] * BS + zz) * hdd;
      if constexpr (PEN) {
        if (masked && a.p.mask == WACM_MASK_PLATE) {
          pchi = T(plate_tab_chi<BS>(a.p, ptab, x, y, zz));
          // (products kept apart from the difference they enter)
          pus[0] = opaque(T(mt.ad * (zg - a.p.x_le[2])));
          pus[2] = opaque(T(-mt.ad * (xg - a.p.x_le[0])));
        } else if (masked) {
          pchi = T(sphere_chi(a.p, xg, yg, zg));
        }
        if (masked && a.dus) {
          const T* du = a.dus + (int64_t)slot * 3 * BS * BS * BS + (zz * BS + y) * BS + x;
          pdu[0] = du[0];
          pdu[1] = du[BS * BS * BS];
          pdu[2] = du[2 * BS * BS * BS];
        }
      }
      if (sponged) psp = T(sponge_eval(a.p, a.L, xg, yg, zg));
    };
    T q[4][7];
#pragma unroll
    for (int mm = 0; mm < 7; ++mm) {
      // a run has at least 4 planes: z0 + 3 lies in the block
      const int z = z0 + mm - 3;
#pragma unroll
      for (int c = 0; c < 4; ++c)
        q[c][mm] = mm < 3 && z < 0 ? zface(4, -1 - z, c) : inb[c * fin + z * zs];
    }
    if constexpr (PEN) {
      // one thread of the last wave tests the block while the loads above are
      // in flight
      if (tid == NT - 1) meta[5] = pen_reach(a.p, a.L, BS, meta, mt.ca, mt.sa);
    }
    // the first plane into its slab (z0 is even: slab 0)
#pragma unroll
    for (int c = 0; c < 4; ++c) slab[0][c][cidx] = q[c][3];
    if (hthr) {
#pragma unroll
      for (int c = 0; c < 4; ++c) slab[0][c][hli] = hp[c * hfs + z0 * hzs];
    }
    if constexpr (PEN) {
      lds_barrier();
      reach = __builtin_amdgcn_readfirstlane(meta[5]);
      masked = (reach & 1) != 0;
      sponged = (reach & 2) != 0;
      if (masked && a.p.mask == WACM_MASK_PLATE) {
        plate_tab_fill<BS>(a.p, mt, meta, hdd, ptab, z0, ZR);
        lds_barrier();
      }
      pen_at(z0);
    }

    for (int k = 0; k < ZR; ++k) {
      const int z = z0 + k;
      T(*sb)[W * WY] = slab[z & 1];
      // loads for the next plane: column value at z+4 and this thread's halo point
      T nq[4], hnx[4];
      if (k + 1 < ZR) {
        const int zz = z + 4;
#pragma unroll
        for (int c = 0; c < 4; ++c)
          nq[c] = zz < BS ? inb[c * fin + zz * zs] : zface(5, zz - BS, c);
        if (hthr) {
#pragma unroll
          for (int c = 0; c < 4; ++c) hnx[c] = hp[c * hfs + (z + 1) * hzs];
        }
      }
      // epilogue operands of this point, loaded early if PREF
      T unv[4], acv[4];
      if (PREF) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          if (MODE == 2 || MODE == 3) unv[c] = ntload(unb + c * ufs + z * uzs, a.nt);
          if (MODE == 4) acv[c] = ntload(accb + c * afs + z * azs, a.nt);
        }
      }
      lds_barrier();

      // rhs, accumulated field by field, in explicit fused multiply-adds: the
      // compiler would contract the variants of this kernel differently, and
      // every schedule has to give the same bits.  The Laplacian is summed one
      // axis after the other: with the six equal distances first (20 FP64
      // operations fewer per point, 2% of a step of 20000 blocks of 24^3) its
      // partial sums are three times as large, and the rhs of a flow that
      // viscosity dominates is 1.7 times as far from its 64-bit value.
      const T u = q[0][3], v = q[1][3], w = q[2][3], pr = q[3][3];
      T r[4], div = T(0);
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const T* s = sb[c];
        const T dx = fma(a3, s[cidx + 3] - s[cidx - 3],
                         fma(a1, s[cidx + 1] - s[cidx - 1], a2 * (s[cidx + 2] - s[cidx - 2])));
        const T dy = fma(a3, s[cidx + 3 * W] - s[cidx - 3 * W],
                         fma(a1, s[cidx + W] - s[cidx - W],
                             a2 * (s[cidx + 2 * W] - s[cidx - 2 * W])));
        const T dz =
            fma(a3, q[c][6] - q[c][0], fma(a1, q[c][4] - q[c][2], a2 * (q[c][5] - q[c][1])));
        if (c < 3) {
          const T lap = (lap1(s[cidx - 2], s[cidx - 1], s[cidx], s[cidx + 1], s[cidx + 2]) +
                         lap1(s[cidx - 2 * W], s[cidx - W], s[cidx], s[cidx + W],
                              s[cidx + 2 * W])) +
                        lap1(q[c][1], q[c][2], q[c][3], q[c][4], q[c][5]);
          const T conv = fma(w, dz * ih, fma(u, dx * ih, v * (dy * ih)));
          r[c] = fma(lap * ih2, nu, -conv);
          div = fma(c == 0 ? dx : (c == 1 ? dy : dz), ih, div);
        } else {
          r[0] = fma(-dx, ih, r[0]);
          r[1] = fma(-dy, ih, r[1]);
          r[2] = fma(-dz, ih, r[2]);
        }
      }
      r[3] = fma(-c0sq, div, -cg * pr);
      if (PEN) {
        const wacm_params& p = a.p;
        T chi = pchi, sp = psp, us[3] = {pus[0], pus[1], pus[2]};
        if (masked && a.dus) {
#pragma unroll
          for (int d = 0; d < 3; ++d) us[d] += pdu[d];
        }
        const T iceta = masked ? T(1.0 / p.c_eta) : T(0), icsp = sponged ? T(1.0 / p.c_sp) : T(0);
        const T val[4] = {u, v, w, pr};
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          if (masked) r[c] = fma(-chi * iceta, val[c] - us[c], r[c]);
          if (sponged) r[c] = fma(-sp * icsp, val[c] - T(p.u_inf[c]), r[c]);
        }
        if (sponged) r[3] = fma(-sp * icsp, pr - T(p.p_inf), r[3]);
      }

      if (!PREF) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          if (MODE == 2 || MODE == 3) unv[c] = ntload(unb + c * ufs + z * uzs, a.nt);
          if (MODE == 4) acv[c] = ntload(accb + c * afs + z * azs, a.nt);
        }
      }
      if (MODE == 0) {
#pragma unroll
        for (int c = 0; c < 4; ++c) outb[c * ofs + z * ozs] = r[c];
      } else if (MODE == 4) {
        const T val[4] = {u, v, w, pr};
        T nv[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          nv[c] = fma(fA, r[c], fma(val[c], T(1.0 / 3.0), acv[c]));
          ntstore(nv[c], unb + c * ufs + z * uzs, a.nt);
        }
        // The x-ghost columns of the row are cleared too, so that every cache
        // line of the padded row is written whole: rows of partly written lines
        // store far slower.  Ghost layers carry no state between steps.
        const int gx = a.Lun.ng;
        if (!xun && (x < gx || x >= BS - gx)) {
          const int off = x < gx ? -gx : gx;
#pragma unroll
          for (int c = 0; c < 4; ++c) ntstore(T(0), unb + c * ufs + z * uzs + off, a.nt);
        }
        if (a.umax_part) m2 = fmax(m2, speed2(double(nv[0]), double(nv[1]), double(nv[2])));
      } else {
        const T val[4] = {u, v, w, pr};
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const T u0 = MODE == 1 ? val[c] : unv[c];
          // (U^n + Y2)/3 = 2/3 U^n + dt/6 k1, from the input Y2 = U^n + dt/2 k1
          if (MODE == 2)
            ntstore(fma(u0 + val[c], T(1.0 / 3.0), fA * r[c]), accb + c * afs + z * azs, a.nt);
          outb[c * ofs + z * ozs] = fma(fB, r[c], u0);
        }
        // a padded output's rows are written whole as in stage 4 (the next
        // stage's fill rewrites every ghost point that is read)
        const int gx = a.Lout.ng;
        if (OWNG && (x < gx || x >= BS - gx)) {
          const int off = x < gx ? -gx : gx;
#pragma unroll
          for (int c = 0; c < 4; ++c) outb[c * ofs + z * ozs + off] = T(0);
        }
      }
      if (k + 1 < ZR) {
        // plane z+1 into the other slab: it was last read before this
        // plane's barrier, which every thread has passed
        T(*nb_)[W * WY] = slab[(z + 1) & 1];
#pragma unroll
        for (int c = 0; c < 4; ++c) nb_[c][cidx] = q[c][4];
        if (hthr) {
#pragma unroll
          for (int c = 0; c < 4; ++c) nb_[c][hli] = hnx[c];
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) {
#pragma unroll
          for (int mm = 0; mm < 6; ++mm) q[c][mm] = q[c][mm + 1];
          q[c][6] = nq[c];
        }
        if (PEN) pen_at(z + 1);
      }
    }
    if (MODE == 4 && a.umax_part) {
      // the work item's maximum, reduced in the workgroup; red is free again
      // by the next item's writes (several barriers later)
      m2 = wave_max(m2);
      if ((tid & 63) == 0) red[tid >> 6] = m2;
      lds_barrier();
      if (tid == 0) {
        double mx = red[0];
#pragma unroll
        for (int w = 1; w < NT / 64; ++w) mx = fmax(mx, red[w]);
        a.umax_part[boff * NPB + item] = mx;
      }
    }
    if (dyn && tid == 0) qitem = queue_take(a.queue, qh, qchunk, (int)nitems, qpend);
  }
}

// resident workgroups per CU of a kernel (queried once per instantiation)
template <typename K>
static int resident_per_cu(K kernel, int threads) {
  int n = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, kernel, threads, 0) != hipSuccess || n < 1)
    n = 1;
  return n;
}

template <typename T, int BS, int TY, int MODE, bool PEN, bool PREF, int NZ>
static hipError_t stage_launch_z(const StageArgs<T>& a, int64_t slots, hipStream_t st) {
  const int64_t items = a.nb * (BS / TY) * NZ;
  const int64_t grid = std::max<int64_t>(1, std::min(slots, items));
  if (a.nmax) *a.nmax = items;
  if (a.queue) {
    queue_clear<<<1, 8 * QSTRIDE, 0, st>>>(a.queue);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  stage_kernel<T, BS, TY, MODE, PEN, PREF, NZ><<<(unsigned)grid, BS * TY, 0, st>>>(a);
  return hipGetLastError();
}

// EARLY, RUNS: epilogue operands loaded before the plane's barrier, in whole
// columns and in runs of planes.  The rhs and the first stage have none: one
// kernel for both.
template <typename T, int BS, int TY, int MODE, bool PEN, bool EARLY, bool RUNS>
static hipError_t stage_launch_t(const StageArgs<T>& a, int wg_per_cu, hipStream_t st) {
  constexpr bool E = EARLY && MODE % 10 >= 2, R = RUNS && MODE % 10 >= 2;
  static const int resident =
      resident_per_cu(stage_kernel<T, BS, TY, MODE, PEN, E, 1>, BS * TY);
  const int cus = num_cus(), per_cu = wg_per_cu > 0 ? wg_per_cu : resident;
  const int64_t slots = (int64_t)per_cu * cus;
  // the lists of blocks with and without penalization are counted on the
  // device only; the split is for large grids
  const int nz = a.blist ? 1 : plane_runs(a.nb * (BS / TY), per_cu, cus, BS);
  if (nz == 4) return stage_launch_z<T, BS, TY, MODE, PEN, R, 4>(a, slots, st);
  if (nz == 2) return stage_launch_z<T, BS, TY, MODE, PEN, R, 2>(a, slots, st);
  return stage_launch_z<T, BS, TY, MODE, PEN, E, 1>(a, slots, st);
}

template <typename T, int BS, int TY, int MODE, bool PEN>
static hipError_t stage_launch_e(const StageArgs<T>& a, const wacm_schedule& s, hipStream_t st) {
  constexpr bool f64 = sizeof(T) == 8;
  const int w = s.wg_per_cu;
  if (!early_loads(s, f64, 1)) return stage_launch_t<T, BS, TY, MODE, PEN, false, false>(a, w, st);
  if constexpr (f64 && TY == 8)  // early_loads tells whole columns from runs for its FP64 tiles
    if (!early_loads(s, f64, 2)) return stage_launch_t<T, BS, TY, MODE, PEN, true, false>(a, w, st);
  return stage_launch_t<T, BS, TY, MODE, PEN, true, true>(a, w, st);
}

// tile_rows 0: whole-block work items; 8: tiles of 8 rows (bs >= 24, where the
// halo of a tile plane fits in one point per thread; smaller blocks use whole
// blocks)
template <typename T, int BS, int MODE, bool PEN>
static hipError_t stage_launch_p(const StageArgs<T>& a, const wacm_schedule& s, hipStream_t st) {
  if constexpr (BS >= 24) {
    if (s.tile_rows == 8) return stage_launch_e<T, BS, 8, MODE, PEN>(a, s, st);
  }
  return stage_launch_e<T, BS, BS, MODE, PEN>(a, s, st);
}

template <typename T, int BS, int MODE>
static hipError_t stage_launch(const StageArgs<T>& a, const wacm_schedule& s, hipStream_t st) {
  const bool pen = a.p.mask || a.p.sponge || a.dus;
  if (pen && a.blist) {
    // the blocks where the penalization vanishes take the unpenalized
    // variant, the others the penalized one
    StageArgs<T> f = a, n = a;
    f.bsel = 0;
    n.bsel = 1;
    hipError_t e = stage_launch_p<T, BS, MODE, false>(f, s, st);
    return e != hipSuccess ? e : stage_launch_p<T, BS, MODE, true>(n, s, st);
  }
  return pen ? stage_launch_p<T, BS, MODE, true>(a, s, st)
             : stage_launch_p<T, BS, MODE, false>(a, s, st);
}

template <typename T, int MODE>
static hipError_t stage_dispatch(int bs, const StageArgs<T>& a, const wacm_schedule& s,
                                 hipStream_t st) {
  switch (bs) {
    case 16:
      return stage_launch<T, 16, MODE>(a, s, st);
    case 24:
      return stage_launch<T, 24, MODE>(a, s, st);
    case 32:
      return stage_launch<T, 32, MODE>(a, s, st);
    default:
      return hipErrorInvalidValue;
  }
}

template <typename T, int BS, int S>
static hipError_t stage_owng_bs(const StageArgs<T>& a, int wg_per_cu, hipStream_t st) {
  constexpr bool early = sizeof(T) == 4;
  return a.p.mask || a.p.sponge || a.dus
             ? stage_launch_t<T, BS, 8, 10 + S, true, early, early>(a, wg_per_cu, st)
             : stage_launch_t<T, BS, 8, 10 + S, false, early, early>(a, wg_per_cu, st);
}

template <typename T, int BS>
static hipError_t stage_owng_mode(int s, const StageArgs<T>& a, int w, hipStream_t st) {
  switch (s) {
    case 1: return stage_owng_bs<T, BS, 1>(a, w, st);
    case 2: return stage_owng_bs<T, BS, 2>(a, w, st);
    case 3: return stage_owng_bs<T, BS, 3>(a, w, st);
    case 4: return stage_owng_bs<T, BS, 4>(a, w, st);
    default: return hipErrorInvalidValue;
  }
}

template <typename T>
static hipError_t stage_run_t(int mode, int bs, const StageArgs<T>& a, const wacm_schedule& s,
                              hipStream_t st) {
  switch (mode) {
    case 0: return stage_dispatch<T, 0>(bs, a, s, st);
    case 1: return stage_dispatch<T, 1>(bs, a, s, st);
    case 2: return stage_dispatch<T, 2>(bs, a, s, st);
    case 3: return stage_dispatch<T, 3>(bs, a, s, st);
    case 4: return stage_dispatch<T, 4>(bs, a, s, st);
    default:
      return bs == 24   ? stage_owng_mode<T, 24>(mode - 10, a, s.wg_per_cu, st)
             : bs == 32 ? stage_owng_mode<T, 32>(mode - 10, a, s.wg_per_cu, st)
                        : hipErrorInvalidValue;
  }
}

}  // namespace wacm
