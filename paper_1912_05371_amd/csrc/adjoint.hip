// Discrete adjoint of the hot path on a frozen grid with a fixed time step:
// transposes of the ghost synchronisation (Sec. 4.2 / 3.1), of the linearised
// penalized ACM right-hand side (Sec. 2.2-2.3) and of one classical RK4 step,
// plus the gradient of the x-component of the penalization force (Sec. 2.2).
// Parameters: theta = (amp, freq, phase) of the plate pitch and a static
// extra solid velocity dus.  Every reduction runs in a fixed order, so the
// results are bitwise reproducible.
#include <algorithm>
#include <tuple>

#include "resolve.h"
#include "stage.h"
#include "wacm_internal.h"

namespace wacm {

// --------------------------------------------------------------------------
// transpose of the ghost fill: CSR gather plan built on the host
// --------------------------------------------------------------------------
void free_adj_plans(wacm_grid* g) {
  g->plan[0] = AdjPlan{};
  g->plan[1] = AdjPlan{};
}

// Face-star plan, for the RK4 step's adjoint.  Same-level faces need no plan
// (adj_stage_kernel reads the neighbours in place).  For each face next to
// another level adj_face_kernel leaves in its slot of the face buffer, per
// field, what the ghost values of that face return: next to a finer leaf one
// value per ghost point, due to the coincident fine point; next to a coarser
// one a value per point of the lattice box the prediction reads.  Rows are
// the interior points that receive such values (field 0 element offset in the
// compact layout), entries the positions in the face buffer, in order, so the
// sums are fixed.  Kept on the host until the grid changes.
constexpr int adj_face_stride(int bs) { return 3 * bs * bs; }  // per field and face

static void build_face_plan(const wacm_grid* g, AdjPlan& pl) {
  const int bs = g->d.bs, S = bs / 2 + 3, F = adj_face_stride(bs);
  Layout L;
  L.P = bs;
  L.ng = 0;
  L.fstride = (int64_t)bs * bs * bs;
  L.bstride = 4 * L.fstride;
  std::vector<std::pair<int64_t, int64_t>> ent;  // (receiving point, buffer position)
  ent.reserve((size_t)g->n_cface * F);
  int64_t k = 0;  // position in the list of faces next to another level (coarse_faces)
  for (const Tab& t : g->h_tab)
    for (int f = 0; f < 6; ++f) {
      const int kind = t.kind[FACE_REGION[f]];
      if (kind == 0) continue;
      const int axis = f >> 1, side = f & 1, ua = axis == 0 ? 1 : 0, ub = axis == 2 ? 1 : 2;
      const int n0 = kind > 0 ? (side ? bs : -1) : (side ? bs - 2 : -6);
      const int dn = kind > 0 ? (side ? 1 : -1) : 2;
      const int nn = kind > 0 ? 3 : (side ? 4 : 5), nt = kind > 0 ? bs : S;
      for (int p = 0; p < nn * nt * nt; ++p) {
        const int q = p % (nt * nt);
        int li[3];
        li[axis] = n0 + dn * (p / (nt * nt));
        li[ua] = kind > 0 ? q % nt : 2 * (q % nt) - 2;
        li[ub] = kind > 0 ? q / nt : 2 * (q / nt) - 2;
        ent.emplace_back(point_offset(t, bs, L, li[0], li[1], li[2]), 4 * F * k + p);
      }
      ++k;
    }
  std::sort(ent.begin(), ent.end());
  pl.h_src.reserve(ent.size());
  for (size_t e = 0; e < ent.size(); ++e) {
    if (e == 0 || ent[e].first != ent[e - 1].first) {
      pl.h_dst.push_back(ent[e].first);
      pl.h_ptr.push_back((int64_t)e);
    }
    pl.h_src.push_back(ent[e].second);
  }
  pl.h_ptr.push_back((int64_t)ent.size());
  pl.nrows = (int64_t)pl.h_dst.size();
  pl.nnz = (int64_t)pl.h_src.size();
}

// Full plan (all ng layers), for wacm_sync_ghosts_adj: every ghost point of
// every active block, with the interior points its value was taken from:
// rows are the source interior points, entries the ghost points that read
// them with their prediction weights, sorted so the gather is deterministic.
// Host part only (kept until the grid changes); upload_adj_plan copies it
// into the caller's buffer.
int build_adj_plan(wacm_grid* g, int face_only, std::string& err) {
  AdjPlan& pl = g->plan[face_only ? 1 : 0];
  if (pl.built || !pl.h_ptr.empty()) return WACM_OK;
  (void)err;
  AdjPlan np;
  if (face_only) {
    build_face_plan(g, np);
    pl = std::move(np);
    return WACM_OK;
  }
  const int bs = g->d.bs, ng = g->d.ng, P = g->P;
  Layout L;
  L.P = P;
  L.ng = ng;
  L.fstride = (int64_t)P * P * P;
  L.bstride = 4 * L.fstride;
  const int npts = P * P * P - bs * bs * bs;
  std::vector<std::tuple<int64_t, int64_t, double>> ent;
  std::vector<int64_t> ghosts;
  ghosts.reserve((size_t)g->nb * npts);
  ent.reserve((size_t)g->nb * npts * 2);
  for (int64_t ib = 0; ib < g->nb; ++ib) {
    const Tab& t = g->h_tab[ib];
    const int64_t base = (int64_t)t.meta[0] * L.bstride;
    for (int p = 0; p < npts; ++p) {
      int i, j, k;
      shell_point(p, bs, ng, P, 0, i, j, k);
      const int64_t go = base + ((int64_t)(k + ng) * P + (j + ng)) * P + (i + ng);
      ghosts.push_back(go);
      ghost_taps<double>(t, bs, L, i, j, k,
                         [&](int64_t off, double w) { ent.emplace_back(off, go, w); });
    }
  }
  std::sort(ent.begin(), ent.end());
  np.h_src.reserve(ent.size());
  np.h_w.reserve(ent.size());
  for (size_t e = 0; e < ent.size(); ++e) {
    if (e == 0 || std::get<0>(ent[e]) != std::get<0>(ent[e - 1])) {
      np.h_dst.push_back(std::get<0>(ent[e]));
      np.h_ptr.push_back((int64_t)e);
    }
    np.h_src.push_back(std::get<1>(ent[e]));
    np.h_w.push_back(std::get<2>(ent[e]));
  }
  np.h_ptr.push_back((int64_t)ent.size());
  np.h_ghost.swap(ghosts);
  np.nrows = (int64_t)np.h_dst.size();
  np.nnz = (int64_t)np.h_src.size();
  np.nghost = (int64_t)np.h_ghost.size();
  pl = std::move(np);
  return WACM_OK;
}

static size_t up256(size_t v) { return (v + 255) / 256 * 256; }

// device bytes of a plan: dst, ptr, src, w, ghost, each 256-byte aligned (the
// face-star plan has no weights and no ghost list)
size_t adj_plan_bytes(const AdjPlan& p) {
  return up256(8 * p.h_dst.size()) + up256(8 * p.h_ptr.size()) + up256(8 * p.h_src.size()) +
         up256(8 * p.h_w.size()) + up256(8 * p.h_ghost.size());
}

int upload_adj_plan(wacm_grid* g, int face_only, void* ws, size_t bytes, std::string& err) {
  AdjPlan& pl = g->plan[face_only ? 1 : 0];
  if (int rc = build_adj_plan(g, face_only, err)) return rc;
  if (bytes < adj_plan_bytes(pl)) {
    err = "adjoint plan buffer smaller than wacm_adj_plan_bytes()";
    return WACM_E_INVAL;
  }
  char* w = (char*)ws;
  hipError_t e = hipSuccess;
  auto put = [&](auto** d, const auto& v) {
    using E = typename std::remove_reference<decltype(v)>::type::value_type;
    *d = reinterpret_cast<E*>(w);
    if (e == hipSuccess && !v.empty())
      e = hipMemcpy(w, v.data(), sizeof(E) * v.size(), hipMemcpyHostToDevice);
    w += up256(sizeof(E) * v.size());
  };
  put(&pl.d_dst, pl.h_dst);
  put(&pl.d_ptr, pl.h_ptr);
  put(&pl.d_src, pl.h_src);
  put(&pl.d_w, pl.h_w);
  put(&pl.d_ghost, pl.h_ghost);
  if (e != hipSuccess) {
    pl.built = 0;
    err = std::string("adjoint plan upload: ") + hipGetErrorString(e);
    return WACM_E_HIP;
  }
  pl.built = 1;
  return WACM_OK;
}

template <typename T>
__global__ __launch_bounds__(NT_GEN) void sync_adj_gather(const int64_t* __restrict__ dst,
                                                          const int64_t* __restrict__ ptr,
                                                          const int64_t* __restrict__ src,
                                                          const double* __restrict__ w,
                                                          int64_t nrows, T* __restrict__ U,
                                                          int64_t fs) {
  for (int64_t r = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; r < nrows;
       r += (int64_t)gridDim.x * blockDim.x) {
    double acc[4] = {0, 0, 0, 0};
    for (int64_t e = ptr[r]; e < ptr[r + 1]; ++e) {
      const double we = w[e];
#pragma unroll
      for (int c = 0; c < 4; ++c) acc[c] += we * (double)U[src[e] + c * fs];
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) U[dst[r] + c * fs] += T(acc[c]);
  }
}

template <typename T>
__global__ __launch_bounds__(NT_GEN) void zero_points(const int64_t* __restrict__ idx, int64_t n,
                                                      T* __restrict__ U, int64_t fs) {
  for (int64_t r = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; r < n;
       r += (int64_t)gridDim.x * blockDim.x) {
#pragma unroll
    for (int c = 0; c < 4; ++c) U[idx[r] + c * fs] = T(0);
  }
}

// --------------------------------------------------------------------------
// transpose of the linearised rhs, gather form within each block
// --------------------------------------------------------------------------
// For a point j of the block (interior, or face star of depth 3), with v the
// rhs adjoint (zero outside the interior) and u the synchronised state:
//   Ubar_c += sum_d D1_d[v_c u_d] + nu sum_d D2_d[v_c] + C0^2 D1_c[v_p]
//             - [j interior] (sum_c' v_c' D1_c u_c' + chi/C_eta v_c + sponge)
//   Ubar_p += sum_d D1_d[v_d] - [j interior] (C_gamma + sponge) v_p
// (D1, D2 the forward stencils applied to fields that vanish outside the
// interior: the transpose of the antisymmetric D1 moves its sign into the
// convective and gradient terms).
template <typename T>
struct AdjArgs {
  const Tab* tab;
  int64_t nb;
  const T* U;
  const T* V;
  T* Ub;
  Layout L;
  int bs;
  double Ldom;
  double t;
  wacm_params p;
  const T* dus;    // [slot][3][bs^3] or null
  double* dusbar;  // [slot][3][bs^3] or null (accumulated, FP64)
  double* part;    // per-block theta partials [nb][3]
  double weight;   // force adjoint weight
};

template <typename T>
__global__ __launch_bounds__(NT_GEN) void rhs_adj_kernel(AdjArgs<T> a) {
  __shared__ double red[3][NT_GEN];
  const int bs = a.bs, ng = a.L.ng, P = a.L.P;
  const int64_t fs = a.L.fstride;
  const int n3 = bs * bs * bs, nf = 18 * bs * bs;
  const double tw[3] = {TW1, TW2, TW3};
  const double w2[5] = {D2A, D2B, D2C, D2B, D2A};
  const wacm_params& p = a.p;
  for (int64_t ib = blockIdx.x; ib < a.nb; ib += gridDim.x) {
    const int32_t* m = a.tab[ib].meta;
    const int slot = m[0], J = m[1];
    const double h = a.Ldom / (double(int64_t(1) << J) * bs);
    const T ih = T(1.0 / h), ih2 = T(1.0 / (h * h));
    const int64_t base = (int64_t)slot * a.L.bstride;
    const T* U = a.U + base;
    const T* V = a.V + base;
    T* B = a.Ub + base;
    auto idx = [&](int i, int j, int k) -> int64_t {
      return ((int64_t)(k + ng) * P + (j + ng)) * P + (i + ng);
    };
    auto inside = [&](int i, int j, int k) {
      return i >= 0 && i < bs && j >= 0 && j < bs && k >= 0 && k < bs;
    };
    const PlateAdjTime pm = plate_adj_time(p, a.t);
    double th[3] = {0, 0, 0};
    for (int pt = threadIdx.x; pt < n3 + nf; pt += blockDim.x) {
      int q[3];
      if (pt < n3) {
        q[0] = pt % bs;
        q[1] = (pt / bs) % bs;
        q[2] = pt / (bs * bs);
      } else {
        shell_point(pt - n3, bs, ng, P, 1, q[0], q[1], q[2]);
      }
      const bool in = pt < n3;
      T acc[4] = {T(0), T(0), T(0), T(0)};
      for (int d = 0; d < 3; ++d) {
        for (int mm = 1; mm <= 3; ++mm) {
          int qp[3] = {q[0], q[1], q[2]}, qm[3] = {q[0], q[1], q[2]};
          qp[d] += mm;
          qm[d] -= mm;
          const bool ip = inside(qp[0], qp[1], qp[2]), im = inside(qm[0], qm[1], qm[2]);
          T vp[4] = {T(0), T(0), T(0), T(0)}, vm[4] = {T(0), T(0), T(0), T(0)};
          T up = T(0), um = T(0);
          if (ip) {
            const int64_t o = idx(qp[0], qp[1], qp[2]);
            for (int c = 0; c < 4; ++c) vp[c] = V[o + c * fs];
            up = U[o + d * fs];
          }
          if (im) {
            const int64_t o = idx(qm[0], qm[1], qm[2]);
            for (int c = 0; c < 4; ++c) vm[c] = V[o + c * fs];
            um = U[o + d * fs];
          }
          const T am = T(tw[mm - 1]) * ih;
          for (int c = 0; c < 3; ++c) acc[c] += am * (vp[c] * up - vm[c] * um);
          acc[d] += T(p.c0 * p.c0) * am * (vp[3] - vm[3]);
          acc[3] += am * (vp[d] - vm[d]);
        }
        for (int o = -2; o <= 2; ++o) {
          int qo[3] = {q[0], q[1], q[2]};
          qo[d] += o;
          if (!inside(qo[0], qo[1], qo[2])) continue;
          const int64_t oo = idx(qo[0], qo[1], qo[2]);
          const T wgt = T(p.nu * w2[o + 2]) * ih2;
          for (int c = 0; c < 3; ++c) acc[c] += wgt * V[oo + c * fs];
        }
      }
      const int64_t oj = idx(q[0], q[1], q[2]);
      if (in) {
        T v[4], u[4];
        for (int c = 0; c < 4; ++c) {
          v[c] = V[oj + c * fs];
          u[c] = U[oj + c * fs];
        }
        // pointwise: - sum_c' v_c' D1_c u_c'
        for (int c = 0; c < 3; ++c) {
          const int64_t st = c == 0 ? 1 : (c == 1 ? P : (int64_t)P * P);
          for (int c2 = 0; c2 < 3; ++c2) {
            const T* f = U + c2 * fs;
            const T d1 = (T(TW1) * (f[oj + st] - f[oj - st]) +
                          T(TW2) * (f[oj + 2 * st] - f[oj - 2 * st]) +
                          T(TW3) * (f[oj + 3 * st] - f[oj - 3 * st])) *
                         ih;
            acc[c] -= v[c2] * d1;
          }
        }
        acc[3] -= T(p.c_gamma) * v[3];
        const double xg = (double)(m[2] * bs + q[0]) * h, yg = (double)(m[3] * bs + q[1]) * h,
                     zg = (double)(m[4] * bs + q[2]) * h;
        if (p.sponge) {
          const T sp = T(sponge_eval(p, a.Ldom, xg, yg, zg) / p.c_sp);
          for (int c = 0; c < 4; ++c) acc[c] -= sp * v[c];
        }
        if (p.mask) {
          const int qi = (q[2] * bs + q[1]) * bs + q[0];
          double chi, dchi = 0.0, us[3], dsd[3] = {0, 0, 0};
          if (p.mask == WACM_MASK_PLATE)
            plate_adj_point(p, pm, xg, yg, zg, chi, dchi, us, dsd);
          else
            mask_eval(p, a.t, xg, yg, zg, chi, us);
          double gal = 0.0, gad = 0.0;
          for (int c = 0; c < 3; ++c) {
            acc[c] -= T(chi / p.c_eta) * v[c];
            if (a.dusbar)
              a.dusbar[((int64_t)slot * 3 + c) * n3 + qi] += chi / p.c_eta * (double)v[c];
            const double e = a.dus ? (double)a.dus[((int64_t)slot * 3 + c) * n3 + qi] : 0.0;
            gal += -dchi / p.c_eta * ((double)u[c] - us[c] - e) * (double)v[c];
            gad += chi / p.c_eta * dsd[c] * (double)v[c];
          }
          for (int k2 = 0; k2 < 3; ++k2) th[k2] += gal * pm.dal[k2] + gad * pm.dad[k2];
        }
      }
      for (int c = 0; c < 4; ++c) B[oj + c * fs] += acc[c];
    }
    __syncthreads();
    for (int k2 = 0; k2 < 3; ++k2) red[k2][threadIdx.x] = th[k2];
    __syncthreads();
    for (int s = NT_GEN / 2; s > 0; s >>= 1) {
      if ((int)threadIdx.x < s)
        for (int k2 = 0; k2 < 3; ++k2) red[k2][threadIdx.x] += red[k2][threadIdx.x + s];
      __syncthreads();
    }
    if (threadIdx.x == 0)
      for (int k2 = 0; k2 < 3; ++k2) a.part[ib * 3 + k2] = red[k2][0];
  }
}

// Gradient of weight * F_x (the x-force, Sec. 2.2 midpoint rule) at time t.
// PLATE: the factor tables are the plate's; a sphere's kernel does without their
// LDS (904 blocks of 32^3, FP64: 516 us with it, 440 without).
template <typename T, int bs, bool PLATE>
__global__ __launch_bounds__(NT_GEN) void force_adj_kernel(AdjArgs<T> a) {
  __shared__ double red[3][NT_GEN];
  __shared__ typename std::conditional<PLATE, PlateAdjTab<bs>, NoTab>::type ptab;
  const int ng = a.L.ng, P = a.L.P;
  constexpr int n3 = bs * bs * bs;
  const wacm_params& p = a.p;
  const PlateAdjTime pm = plate_adj_time(p, a.t);
  for (int64_t ib = blockIdx.x; ib < a.nb; ib += gridDim.x) {
    const int32_t* m = a.tab[ib].meta;
    const int slot = m[0], J = m[1];
    const double h = a.Ldom / (double(int64_t(1) << J) * bs);
    const double vol = h * h * h;
    const int64_t base = (int64_t)slot * a.L.bstride;
    double th[3] = {0, 0, 0};
    const bool masked = (pen_reach(p, a.Ldom, bs, m, pm.ca, pm.sa) & 1) != 0;
    if constexpr (PLATE) {
      if (masked) {  // uniform; the last block's reduction has ended
        plate_adj_tab_fill<bs>(p, pm, m, h, 0, bs, ptab);
        __syncthreads();
      }
    }
    for (int qi = threadIdx.x; qi < n3; qi += NT_GEN) {
      const int i = qi % bs, j = (qi / bs) % bs, k = qi / (bs * bs);
      const int64_t o = base + ((int64_t)(k + ng) * P + (j + ng)) * P + (i + ng);
      if (!masked) {
        // every term is 0; 0 times a value that is not finite is not
        for (int k2 = 0; k2 < 3; ++k2) th[k2] += 0.0 * (double)a.U[o];
        continue;
      }
      const T u0 = a.U[o], b0 = a.Ub[o];  // in flight while the mask is evaluated
      const double xg = (double)(m[2] * bs + i) * h, yg = (double)(m[3] * bs + j) * h,
                   zg = (double)(m[4] * bs + k) * h;
      double chi, dchi = 0.0, us[3] = {0, 0, 0}, dsd[3] = {0, 0, 0};
      if constexpr (PLATE)
        plate_adj_tab_point<bs>(p, pm, ptab, i, j, k, xg, zg, chi, dchi, us, dsd);
      else
        chi = sphere_chi<false>(p, xg, yg, zg);
      const double cw = a.weight * chi * vol / p.c_eta;
      a.Ub[o] = b0 + T(cw);
      if (a.dusbar) a.dusbar[((int64_t)slot * 3) * n3 + qi] -= cw;
      const double e = a.dus ? (double)a.dus[((int64_t)slot * 3) * n3 + qi] : 0.0;
      const double gal = a.weight * dchi * ((double)u0 - us[0] - e) * vol / p.c_eta;
      const double gad = -cw * dsd[0];
      for (int k2 = 0; k2 < 3; ++k2) th[k2] += gal * pm.dal[k2] + gad * pm.dad[k2];
    }
    __syncthreads();
    for (int k2 = 0; k2 < 3; ++k2) red[k2][threadIdx.x] = th[k2];
    __syncthreads();
    for (int s = NT_GEN / 2; s > 0; s >>= 1) {
      if ((int)threadIdx.x < s)
        for (int k2 = 0; k2 < 3; ++k2) red[k2][threadIdx.x] += red[k2][threadIdx.x + s];
      __syncthreads();
    }
    if (threadIdx.x == 0)
      for (int k2 = 0; k2 < 3; ++k2) a.part[ib * 3 + k2] = red[k2][0];
  }
}

// dtheta += sum over blocks of the partials (fixed order)
__global__ __launch_bounds__(NT_GEN) void theta_finalize(const double* __restrict__ part,
                                                         int64_t nb, double* __restrict__ dtheta) {
  __shared__ double red[3][NT_GEN];
  double s[3] = {0, 0, 0};
  for (int64_t q = threadIdx.x; q < nb; q += blockDim.x)
    for (int k = 0; k < 3; ++k) s[k] += part[q * 3 + k];
  for (int k = 0; k < 3; ++k) red[k][threadIdx.x] = s[k];
  __syncthreads();
  for (int st = NT_GEN / 2; st > 0; st >>= 1) {
    if ((int)threadIdx.x < st)
      for (int k = 0; k < 3; ++k) red[k][threadIdx.x] += red[k][threadIdx.x + st];
    __syncthreads();
  }
  if (threadIdx.x == 0)
    for (int k = 0; k < 3; ++k) dtheta[k] += red[k][0];
}

// --------------------------------------------------------------------------
// one RK stage of the adjoint step
// --------------------------------------------------------------------------
// B = S^T J_rhs(U)^T kb, with kb the rhs adjoint of the stage, U its
// synchronised input and S^T the transpose of the ghost fill.  The stencils of
// the rhs transpose are the forward ones applied to kb and to the products
// kb_c u_d; next to a same-level block the ghost values it returns to that
// block are what these stencils give when kb and u are read across the face,
// so same-level faces need no ghost layers at all.  Next to another level kb
// counts as 0 outside the block; what the block returns across such a face is
// formed by adj_face_kernel and added by adj_gather_kernel.
template <typename T>
struct AdjStage {
  const Tab* tab;
  int64_t nb;
  const T* u;  // stage input: the pool, or x-split
  Layout Lu;
  const T* hb;  // its face halos next to other levels [slot][6][4][3][bs][bs]
  const T* v;   // rhs adjoint kb = vs v
  Layout Lv;
  T vs;
  const T* lam;  // adjoint of the step's output (pool layout)
  Layout Lp;
  const T* sum;  // running sum B_4 + ... (compact)
  T* sout;       // the sum, or at the last stage lam with the sum added
  Layout Lso;
  T* kn;  // next rhs adjoint = lamw lam + kw B (compact), null at the last stage
  Layout Lc;
  T lamw, kw;
  double Ldom, t;
  wacm_params p;
  const T* dus;    // [slot][3][bs^3] or null
  double* dusbar;  // [slot][3][bs^3] or null (accumulated, FP64)
  double* bad;     // per work item: 0, or NaN if kb is not finite somewhere
  double* part;    // theta partials, 3 per work item of adj_pen_kernel
};

// Element offset (field 0) of a block's interior point in a register.
__device__ __forceinline__ int64_t point_in(const Layout& L, int bs, int slot, int i, int j,
                                            int k) {
  return (int64_t)slot * L.bstride +
         (L.xs ? (int64_t)xsplit_offset(bs, i, j, k)
               : ((int64_t)(k + L.ng) * L.P + (j + L.ng)) * L.P + (i + L.ng));
}

// Bound: memory (24 values per point).  Same scheme as the forward stage
// kernel: work items are tiles of TY rows of a block (TY = BS = 16: the whole
// block), one thread per column marching in z, the planes of kb (4 fields) and
// u (3) in a double-buffered LDS slab, their z neighbours in registers, one
// LDS barrier per plane, the next plane's loads and the point's other operands
// issued before it, without branches (a conditional load, or a product with
// what was loaded, would wait there).  The pointwise mask and sponge terms are
// adj_pen_kernel's.  FIRST, LAST: position of the stage in the reverse sweep.
// The sum is of the B_s alone, lam joins it at the last stage: with lam in it
// from the start, FP32 rounded lam once per kernel and stage, and the gradient of
// 5 steps was 1.05 times as far from its 64-bit value as with one rounding per
// stage.  1632 blocks of 16^3, FP32: 245 us; the rhs transpose in gather form
// from the padded pool, the zeroing, the transposed ghost fill and three
// combinations that it stands for took 2.7 ms.
template <typename T, int BS, int TY, bool FIRST, bool LAST>
__global__ __launch_bounds__(BS* TY) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 8 ? 2 : 3)))
void adj_stage_kernel(AdjStage<T> a) {
  constexpr int H = 3, W = BS + 2 * H, WY = TY + 2 * H, NT = BS * TY, NTY = BS / TY;
  constexpr int NH = 6 * TY + 6 * BS, B3 = BS * BS * BS;
  static_assert(NH <= NT, "one halo point per thread and plane");
  __shared__ T slab[2][7][W * WY];  // kb_u, kb_v, kb_w, kb_p, u, v, w
  __shared__ FaceDesc<T> fu[6], fv[6];
  __shared__ int32_t meta[8];  // slot, level; 2 + f: kb is 0 beyond face f
  __shared__ T red[NT / 64];
  const int tid = threadIdx.x, x = tid % BS, yl = tid / BS;
  const T am[3] = {T(TW1), T(TW2), T(TW3)};
  const T c0sq = T(a.p.c0 * a.p.c0), cg = T(a.p.c_gamma), vs = a.vs;
  const bool xin = a.Lu.xs != 0;
  const int cidx = (yl + H) * W + (x + H);
  // this thread's halo point of every plane: x faces of the tile's rows, then
  // the 3 rows below and above the tile
  const bool hthr = tid < NH;
  int hkind = 0, hd = 0, hs = 0, hli = 0;
  if (tid < 6 * TY) {
    hkind = tid / (3 * TY);
    const int rem = tid - hkind * 3 * TY;
    hd = rem / TY;
    hs = rem - hd * TY;
    hli = (hs + H) * W + ((hkind == 0 ? -1 - hd : BS + hd) + H);
  } else if (hthr) {
    const int q = tid - 6 * TY;
    hkind = 2 + q / (3 * BS);
    const int rem = q - (hkind - 2) * 3 * BS;
    hd = rem / BS;
    hs = rem - hd * BS;
    hli = ((hkind == 2 ? -1 - hd : TY + hd) + H) * W + (hs + H);
  }
  const int ufs = (int)a.Lu.fstride, vfs = (int)a.Lv.fstride;
  const int vzs = a.Lv.P * a.Lv.P, pzs = a.Lp.P * a.Lp.P;
  const int sozs = a.Lso.P * a.Lso.P;
  const int64_t nitems = a.nb * NTY;
  BlockIter it(nitems, 1);
  for (; it.ib < it.end; it.ib += it.step) {
    const int64_t item = it.ib, ibk = item / NTY;
    const int y0 = (int)(item - ibk * NTY) * TY, y = y0 + yl;
    lds_barrier();
    if (tid < 6) {
      const Tab& tb = a.tab[ibk];
      fu[tid] = face_desc<T, BS, HALO_NB>(tb, a.u, a.Lu, a.hb, tid, xin);
      const int r = tid == 0 ? 12 : (tid == 1 ? 14 : (tid == 2 ? 10 : (tid == 3 ? 16 : (tid == 4 ? 4 : 22))));
      const bool none = tb.kind[r] != 0;  // (reads there stay inside the block)
      FaceDesc<T> f = face_desc<T, BS, HALO_NB>(tb, a.v, a.Lv, a.v, tid, false);
      if (none) {
        f.ptr = a.v + point_in(a.Lv, BS, tb.meta[0], 0, 0, 0);
        f.fs = vfs;
        f.sd = f.s0 = f.s1 = 0;
      }
      fv[tid] = f;
      meta[2 + tid] = none ? 1 : 0;
      if (tid < 2) meta[tid] = tb.meta[tid];
    }
    lds_barrier();
    const int slot = __builtin_amdgcn_readfirstlane(meta[0]);
    const int J = __builtin_amdgcn_readfirstlane(meta[1]);
    const bool zlo = __builtin_amdgcn_readfirstlane(meta[6]) != 0;
    const bool zhi = __builtin_amdgcn_readfirstlane(meta[7]) != 0;
    const double h = a.Ldom / (double(int64_t(1) << J) * BS);
    const T ih = T(1.0 / h), ih2 = T(1.0 / (h * h));
    // weights of rhs_adj_kernel, rounded as there: an FP32 weight's rounding
    // is an error of every point alike, which the gradients would add up
    const T ah[3] = {am[0] * ih, am[1] * ih, am[2] * ih};
    const T w2[3] = {T(a.p.nu * D2C) * ih2, T(a.p.nu * D2B) * ih2, T(a.p.nu * D2A) * ih2};
    // uniform block origins; this thread's column offsets and plane steps
    const T* ub = a.u + (int64_t)slot * a.Lu.bstride;
    const T* vb = a.v + (int64_t)slot * a.Lv.bstride;
    const T* lb = a.lam + (int64_t)slot * a.Lp.bstride;
    const T* sib = a.sum + (int64_t)slot * a.Lc.bstride;
    T* sob = a.sout + (int64_t)slot * a.Lso.bstride;
    T* kob = a.kn + (int64_t)slot * a.Lc.bstride;
    const int ucol = xin ? xsplit_offset(BS, x, y, 0)
                         : (a.Lu.ng * a.Lu.P + (y + a.Lu.ng)) * a.Lu.P + (x + a.Lu.ng);
    const int uzs = xin ? xsplit_zstride(BS, x) : a.Lu.P * a.Lu.P;
    const int pcol = (a.Lp.ng * a.Lp.P + (y + a.Lp.ng)) * a.Lp.P + (x + a.Lp.ng);
    const int ccol = y * BS + x;
    const int vcol = a.Lv.ng ? pcol : ccol;
    const int socol = LAST ? pcol : ccol;
    // values of this thread's column at depth d below (f = 4) or above (f = 5)
    auto zu = [&](int f, int d, int c) -> T {
      const FaceDesc<T>& fz = fu[f];
      if (fz.mode == 1) return fz.ptr[c * ufs + ucol + (f == 4 ? BS - 1 - d : d) * uzs];
      return fz.ptr[c * fz.fs + d * fz.sd + x * fz.s0 + y * fz.s1];
    };
    auto zv = [&](int f, int d, int c) -> T {
      const FaceDesc<T>& fz = fv[f];
      return fz.ptr[c * fz.fs + d * fz.sd + x * fz.s0 + y * fz.s1];
    };
    // this thread's halo point as an affine map in z: ptr[c fs + z zs]; kb's
    // value there is hz times the one loaded, or 0
    const T *hu = a.u, *hv = a.v;
    int hufs = 0, huzs = 0, hvfs = 0, hvzs = 0;
    bool hnone = false;
    if (hthr) {
      const int hy = hkind < 2 ? y0 + hs : (hkind == 2 ? y0 - 1 - hd : y0 + TY + hd);
      if (hkind < 2 || hy < 0 || hy >= BS) {
        const int f = hkind < 2 ? hkind : (hy < 0 ? 2 : 3);
        const int d = hkind < 2 ? hd : (hy < 0 ? -1 - hy : hy - BS), s = hkind < 2 ? hy : hs;
        const FaceDesc<T>& f1 = fu[f];
        if (f1.mode == 1) {
          hu = f1.ptr + xsplit_offset(BS, hs, hy < 0 ? BS + hy : hy - BS, 0);
          hufs = ufs;
          huzs = xsplit_zstride(BS, hs);
        } else {
          hu = f1.ptr + d * f1.sd + s * f1.s0;
          hufs = f1.fs;
          huzs = f1.s1;
        }
        const FaceDesc<T>& f2 = fv[f];
        hv = f2.ptr + d * f2.sd + s * f2.s0;
        hvfs = f2.fs;
        hvzs = f2.s1;
        hnone = meta[2 + f] != 0;
      } else {  // a row of the block's other tiles
        hu = a.u + point_in(a.Lu, BS, slot, hs, hy, 0);
        hufs = ufs;
        huzs = xin ? xsplit_zstride(BS, hs) : a.Lu.P * a.Lu.P;
        hv = a.v + point_in(a.Lv, BS, slot, hs, hy, 0);
        hvfs = vfs;
        hvzs = vzs;
      }
    }
    T q[7][7];  // column values at z - 3 .. z + 3: kb (4), u (3)
#pragma unroll
    for (int mm = 0; mm < 7; ++mm) {
      const int z = mm - 3;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const T w = z < 0 ? zv(4, -1 - z, c) : vb[vcol + c * vfs + z * vzs];
        q[c][mm] = z < 0 && zlo ? T(0) : vs * w;
      }
#pragma unroll
      for (int c = 0; c < 3; ++c)
        q[4 + c][mm] = z < 0 ? zu(4, -1 - z, c) : ub[ucol + c * ufs + z * uzs];
    }
#pragma unroll
    for (int c = 0; c < 7; ++c) slab[0][c][cidx] = q[c][3];
    if (hthr) {
#pragma unroll
      for (int c = 0; c < 4; ++c) slab[0][c][hli] = hnone ? T(0) : vs * hv[c * hvfs];
#pragma unroll
      for (int c = 0; c < 3; ++c) slab[0][4 + c][hli] = hu[c * hufs];
    }
    T bad = T(0);  // not 0 if a value of kb is not finite
#pragma unroll 1
    for (int z = 0; z < BS; ++z) {
      T(*sb)[W * WY] = slab[z & 1];
      T nq[7], hn[7], lv[4], sv[4];
      if (z + 1 < BS) {
        if (z + 4 < BS) {
#pragma unroll
          for (int c = 0; c < 4; ++c) nq[c] = vb[vcol + c * vfs + (z + 4) * vzs];
#pragma unroll
          for (int c = 0; c < 3; ++c) nq[4 + c] = ub[ucol + c * ufs + (z + 4) * uzs];
        } else {
#pragma unroll
          for (int c = 0; c < 4; ++c) nq[c] = zv(5, z + 4 - BS, c);
#pragma unroll
          for (int c = 0; c < 3; ++c) nq[4 + c] = zu(5, z + 4 - BS, c);
        }
        if (hthr) {
#pragma unroll
          for (int c = 0; c < 4; ++c) hn[c] = hv[c * hvfs + (z + 1) * hvzs];
#pragma unroll
          for (int c = 0; c < 3; ++c) hn[4 + c] = hu[c * hufs + (z + 1) * huzs];
        }
      }
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        if (!FIRST) sv[c] = sib[ccol + z * BS * BS + c * B3];
        lv[c] = lb[pcol + z * pzs + c * (int)a.Lp.fstride];
      }
      lds_barrier();
      const T v[4] = {q[0][3], q[1][3], q[2][3], q[3][3]};
      T acc[4] = {T(0), T(0), T(0), T(0)};
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        const int st = d == 0 ? 1 : W;
        auto at = [&](int c, int o) -> T { return d == 2 ? q[c][3 + o] : sb[c][cidx + o * st]; };
        T up[3], um[3];  // u_d at +m, -m
#pragma unroll
        for (int m = 0; m < 3; ++m) {
          up[m] = at(4 + d, m + 1);
          um[m] = at(4 + d, -1 - m);
        }
        T dv = T(0);  // D1_d kb_d
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          T pr = w2[0] * v[c], du = T(0);
#pragma unroll
          for (int m = 0; m < 3; ++m) {
            const T vp = at(c, m + 1), vm = at(c, -1 - m);
            pr += ah[m] * (vp * up[m] - vm * um[m]);
            if (m < 2) pr += w2[m + 1] * (vp + vm);
            if (c == d) dv += ah[m] * (vp - vm);
            du += am[m] * (c == d ? up[m] - um[m] : at(4 + c, m + 1) - at(4 + c, -1 - m));
          }
          acc[c] += pr;
          acc[d] -= v[c] * (ih * du);
        }
        T dp = T(0);
#pragma unroll
        for (int m = 0; m < 3; ++m) dp += (c0sq * ah[m]) * (at(3, m + 1) - at(3, -1 - m));
        acc[d] += dp;
        acc[3] += dv;
      }
      acc[3] -= cg * v[3];
      bad += T(0) * (v[0] + v[1] + v[2]);
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const T sum = FIRST ? acc[c] : sv[c] + acc[c];
        sob[socol + z * sozs + c * (int)a.Lso.fstride] = LAST ? lv[c] + sum : sum;
        if (!LAST) kob[ccol + z * BS * BS + c * B3] = fma(a.kw, acc[c], a.lamw * lv[c]);
      }
      if (z + 1 < BS) {
        T(*nb_)[W * WY] = slab[(z + 1) & 1];
#pragma unroll
        for (int c = 0; c < 7; ++c) nb_[c][cidx] = q[c][4];
        if (hthr) {
#pragma unroll
          for (int c = 0; c < 7; ++c) nb_[c][hli] = c < 4 ? (hnone ? T(0) : vs * hn[c]) : hn[c];
        }
        const bool none = zhi && z + 4 >= BS;
#pragma unroll
        for (int c = 0; c < 7; ++c) {
#pragma unroll
          for (int mm = 0; mm < 6; ++mm) q[c][mm] = q[c][mm + 1];
          q[c][6] = c < 4 ? (none ? T(0) : vs * nq[c]) : nq[c];
        }
      }
    }
    if (a.p.mask) {
      // where the mask is 0 its terms are 0 times kb: not 0 if kb is not finite
      for (int o = 32; o > 0; o >>= 1) bad += __shfl_xor(bad, o, 64);
      if ((tid & 63) == 0) red[tid >> 6] = bad;
      lds_barrier();
      if (tid == 0) {
        T s = red[0];
        for (int w = 1; w < NT / 64; ++w) s += red[w];
        a.bad[item] = (double)s;
      }
    }
  }
}

// The pointwise terms of the mask and the sponge, in the blocks they reach:
// B_c -= chi/C_eta kb_c + sponge kb_c added to the running sum and, weighted,
// to the next rhs adjoint; the gradients with respect to dus and theta.  Bound
// by the latency of its loads (21 per point), so a block's planes are dealt to
// BS / 4 workgroups; a slab needs the plate's factors of its own planes only.
// Points where every term is 0 are passed over.  NTY: work items of the stage
// kernel per block.  100 us per stage on the plate's 1632 blocks, FP32 (inside
// the stage kernel the same terms made it three times as slow).
constexpr int ADJ_PZ = 4;  // planes per work item
template <typename T, int BS, int NTY>
__global__ __launch_bounds__(NT_GEN) void adj_pen_kernel(AdjStage<T> a) {
  constexpr int B3 = BS * BS * BS, NZ = BS / ADJ_PZ, NQ = ADJ_PZ * BS * BS;
  __shared__ PlateAdjTab<BS> ptab;
  __shared__ double red[3][NT_GEN / 64];
  const wacm_params& p = a.p;
  const PlateAdjTime pm = plate_adj_time(p, a.t);
  for (int64_t w = blockIdx.x; w < a.nb * NZ; w += gridDim.x) {
    const int64_t ib = w / NZ;
    const int z0 = (int)(w - ib * NZ) * ADJ_PZ;
    const int32_t* m = a.tab[ib].meta;
    const int slot = m[0];
    const int reach = pen_reach(p, a.Ldom, BS, m, pm.ca, pm.sa);  // uniform
    const bool masked = (reach & 1) != 0, sponged = (reach & 2) != 0;
    double poison = 0.0;
    if (p.mask)
      for (int t = 0; t < NTY; ++t) poison += a.bad[ib * NTY + t];
    const bool bad = !isfinite(poison);
    double th[3] = {poison, poison, poison};
    if (threadIdx.x != 0) th[0] = th[1] = th[2] = 0.0;
    T* __restrict__ sob = a.sout;
    T* __restrict__ ko = a.kn + (int64_t)slot * a.Lc.bstride;
    double* __restrict__ db = a.dusbar + (int64_t)slot * 3 * B3;
    const T* __restrict__ du = a.dus + (int64_t)slot * 3 * B3;
    if (reach || bad) {
      const double h = a.Ldom / (double(int64_t(1) << m[1]) * BS);
      const bool plate = masked && p.mask == WACM_MASK_PLATE;
      __syncthreads();  // the last item's factors and partials are free
      if (plate) plate_adj_tab_fill<BS>(p, pm, m, h, z0, z0 + ADJ_PZ, ptab);
      __syncthreads();
      for (int qq = threadIdx.x; qq < NQ; qq += NT_GEN) {
        const int q = z0 * BS * BS + qq;
        const int i = q % BS, j = (q / BS) % BS, k = q / (BS * BS);
        const double xg = (double)(m[2] * BS + i) * h, yg = (double)(m[3] * BS + j) * h,
                     zg = (double)(m[4] * BS + k) * h;
        const T sp = sponged ? T(sponge_eval(p, a.Ldom, xg, yg, zg) / p.c_sp) : T(0);
        double chi = 0.0, dchi = 0.0, us[3] = {0, 0, 0}, dsd[3] = {0, 0, 0};
        if (plate)
          plate_adj_tab_point<BS>(p, pm, ptab, i, j, k, xg, zg, chi, dchi, us, dsd);
        else if (masked)
          chi = sphere_chi(p, xg, yg, zg);
        // 0 times a value that is not finite is not 0
        if (sp == T(0) && chi == 0.0 && dchi == 0.0 && !bad) continue;
        const int64_t ov = point_in(a.Lv, BS, slot, i, j, k);
        const int64_t ou = point_in(a.Lu, BS, slot, i, j, k);
        T* so = sob + point_in(a.Lso, BS, slot, i, j, k);
        T v[4], u[3], e[3], s0[4], k0[4], acc[4];
        double d0[3];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          v[c] = a.vs * a.v[ov + c * a.Lv.fstride];
          s0[c] = so[c * a.Lso.fstride];
          k0[c] = a.kn ? ko[q + c * B3] : T(0);
          acc[c] = -sp * v[c];
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          u[c] = a.u[ou + c * a.Lu.fstride];
          e[c] = a.dus ? du[c * B3 + q] : T(0);
          d0[c] = a.dusbar ? db[c * B3 + q] : 0.0;
        }
        if (p.mask) {
          const double ce = chi / p.c_eta, de = dchi / p.c_eta;
          double gal = 0.0, gad = 0.0;
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            acc[c] -= T(ce) * v[c];
            if (a.dusbar) db[c * B3 + q] = d0[c] + ce * (double)v[c];
            gal += -de * ((double)u[c] - us[c] - (double)e[c]) * (double)v[c];
            gad += ce * dsd[c] * (double)v[c];
          }
          for (int k2 = 0; k2 < 3; ++k2) th[k2] += gal * pm.dal[k2] + gad * pm.dad[k2];
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          so[c * a.Lso.fstride] = s0[c] + acc[c];
          if (a.kn) ko[q + c * B3] = fma(a.kw, acc[c], k0[c]);
        }
      }
    }
    if (p.mask) {
      if (masked || bad) {
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          for (int o = 32; o > 0; o >>= 1) th[k] += __shfl_xor(th[k], o, 64);
          if ((threadIdx.x & 63) == 0) red[k][threadIdx.x >> 6] = th[k];
        }
        __syncthreads();
      }
      if (threadIdx.x < 3) {
        double s = 0.0;
        if (masked || bad)
          for (int t = 0; t < NT_GEN / 64; ++t) s += red[threadIdx.x][t];
        a.part[w * 3 + threadIdx.x] = s;
      }
    }
  }
}

// What a block returns across its faces next to another level: the rhs
// transpose at the 3 ghost layers of the face, which only the 3 interior
// layers next to it reach, along the normal.  Next to a coarser leaf the
// transpose of the prediction takes these values to the lattice box the
// forward fill reads, one axis at a time (t1, t0, normal) through LDS, in
// FP64; next to a finer leaf they go to the coincident fine points as they
// are.  One work item per face of the list, results in its slot of fb.
template <typename T, int BS>
__global__ __launch_bounds__(NT_GEN) void adj_face_kernel(const Tab* __restrict__ tab,
                                                          const int32_t* __restrict__ cf,
                                                          int64_t n, AdjStage<T> a,
                                                          double* __restrict__ fb) {
  constexpr int B2 = BS * BS, S = BS / 2 + 3, F = adj_face_stride(BS);
  constexpr int PER = (B2 + NT_GEN - 1) / NT_GEN;
  __shared__ double gb[3 * B2];      // ghost values of one field [d][t1][t0]
  __shared__ double pb[3 * S * BS];  // after t1
  __shared__ double pa[3 * S * S];   // after t0
  constexpr double W4[4] = {DDW0, DDW1, DDW1, DDW0};
  const int tid = threadIdx.x;
  const T am[3] = {T(TW1), T(TW2), T(TW3)};
  const T w2[3] = {T(a.p.nu * D2C), T(a.p.nu * D2B), T(a.p.nu * D2A)};
  const T c0sq = T(a.p.c0 * a.p.c0);
  for (int64_t wk = blockIdx.x; wk < n; wk += gridDim.x) {
    const Tab& tb = tab[cf[2 * wk]];
    const int f = cf[2 * wk + 1], axis = f >> 1, side = f & 1;
    const int ua = axis == 0 ? 1 : 0, ub = axis == 2 ? 1 : 2;
    const int r = (axis == 0 ? 2 * side : 1) + 3 * (axis == 1 ? 2 * side : 1) +
                  9 * (axis == 2 ? 2 * side : 1);
    const bool fine = tb.kind[r] > 0;
    const int slot = tb.meta[0];
    const double h = a.Ldom / (double(int64_t(1) << tb.meta[1]) * BS);
    const T ih = T(1.0 / h), ih2 = T(1.0 / (h * h)), sg = side ? T(-1) : T(1);
    // the 3 interior layers of this thread's columns: kb and the normal velocity
    T v[PER][4][3], un[PER][3];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int qq = tid + k * NT_GEN;
      if (qq < B2) {
        int li[3];
        li[ua] = qq % BS;
        li[ub] = qq / BS;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
          li[axis] = side ? BS - 1 - d : d;
          const int64_t ov = point_in(a.Lv, BS, slot, li[0], li[1], li[2]);
#pragma unroll
          for (int c = 0; c < 4; ++c) v[k][c][d] = a.vs * a.v[ov + c * a.Lv.fstride];
          un[k][d] = a.u[point_in(a.Lu, BS, slot, li[0], li[1], li[2]) + axis * a.Lu.fstride];
        }
      }
    }
    double* out = fb + wk * 4 * F;
    const int n0 = side ? BS - 2 : -6, NN = side ? 4 : 5;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
#pragma unroll
      for (int k = 0; k < PER; ++k) {
        const int qq = tid + k * NT_GEN;
        if (qq < B2) {
#pragma unroll
          for (int d = 0; d < 3; ++d) {
            // ghost depth d, interior layer e: distance e + d + 1
            T s = T(0);
#pragma unroll
            for (int e = 0; e + d < 3; ++e) {
              const int m = e + d;  // distance m + 1
              const T w = am[m] * ih * sg;
              if (c < 3) {
                s += w * (v[k][c][e] * un[k][e]);
                if (c == axis) s += (c0sq * w) * v[k][3][e];
                if (m < 2) s += (w2[m + 1] * ih2) * v[k][c][e];
              } else {
                s += w * (axis == 0 ? v[k][0][e] : (axis == 1 ? v[k][1][e] : v[k][2][e]));
              }
            }
            if (fine)
              out[c * F + d * B2 + qq] = (double)s;
            else
              gb[d * B2 + qq] = (double)s;
          }
        }
      }
      if (fine) continue;
      __syncthreads();
      // transposed t1 pass: lattice row s takes t1 = 2 (s - 1) with weight 1
      // and the odd t1 = 2 (s - e) + 1 with weight W4[e]
      for (int p = tid; p < 3 * S * BS; p += NT_GEN) {
        const int t0 = p % BS, rest = p / BS, s = rest % S, d = rest / S;
        const double* g = gb + d * B2 + t0;
        double val = s >= 1 && s <= BS / 2 ? g[2 * (s - 1) * BS] : 0.0;
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (s - e >= 0 && s - e < BS / 2) val += W4[e] * g[(2 * (s - e) + 1) * BS];
        pb[p] = val;
      }
      __syncthreads();
      for (int p = tid; p < 3 * S * S; p += NT_GEN) {
        const int s = p % S, rest = p / S;  // rest = d S + s1
        const double* g = pb + rest * BS;
        double val = s >= 1 && s <= BS / 2 ? g[2 * (s - 1)] : 0.0;
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (s - e >= 0 && s - e < BS / 2) val += W4[e] * g[2 * (s - e) + 1];
        pa[p] = val;
      }
      __syncthreads();
      // normal: lattice layer m takes the ghost layers whose prediction reads it
      for (int p = tid; p < NN * S * S; p += NT_GEN) {
        const int m = p / (S * S), qq = p - m * S * S;
        double val = 0.0;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
          const int g = side ? BS + d : -1 - d;
          if ((g & 1) == 0) {
            if ((g - n0) / 2 == m) val += pa[d * S * S + qq];
          } else {
            const int e = m - (g - 3 - n0) / 2;
            if (e >= 0 && e < 4) val += W4[e] * pa[d * S * S + qq];
          }
        }
        out[c * F + p] = val;
      }
      __syncthreads();
    }
  }
}

// Adds what the faces next to other levels return: per receiving point the
// sum of its entries of the face buffer, to the running sum and, weighted, to
// the next rhs adjoint.  Rows address the compact layout.
template <typename T>
__global__ __launch_bounds__(NT_GEN) void adj_gather_kernel(const int64_t* __restrict__ dst,
                                                            const int64_t* __restrict__ ptr,
                                                            const int64_t* __restrict__ src,
                                                            int64_t nrows, int bs,
                                                            const double* __restrict__ fb,
                                                            AdjStage<T> a) {
  const int F = adj_face_stride(bs);
  for (int64_t r = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; r < nrows;
       r += (int64_t)gridDim.x * blockDim.x) {
    double acc[4] = {0, 0, 0, 0};
    for (int64_t e = ptr[r]; e < ptr[r + 1]; ++e) {
      const double* b = fb + src[e];
#pragma unroll
      for (int c = 0; c < 4; ++c) acc[c] += b[c * F];
    }
    const int64_t o = dst[r];
    const int slot = (int)(o / a.Lc.bstride), q = (int)(o - slot * a.Lc.bstride);
    T* so = a.sout + point_in(a.Lso, bs, slot, q % bs, (q / bs) % bs, q / (bs * bs));
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      so[c * a.Lso.fstride] += T(acc[c]);
      if (a.kn) a.kn[o + c * a.Lc.fstride] += a.kw * T(acc[c]);
    }
  }
}

// --------------------------------------------------------------------------
// launchers
// --------------------------------------------------------------------------
static Layout pool_L(const wacm_grid* g) {
  Layout L;
  L.P = g->P;
  L.ng = g->d.ng;
  L.fstride = (int64_t)g->P * g->P * g->P;
  L.bstride = 4 * L.fstride;
  return L;
}

static unsigned grid_n(int64_t n, int64_t cap = 2048) {
  return (unsigned)std::max<int64_t>(1, std::min<int64_t>(n, cap));
}

size_t adj_work_bytes(const wacm_grid* g) {
  const size_t es = g->d.dtype == WACM_F64 ? 8 : 4;
  const size_t reg = (size_t)g->d.capacity * 4 * g->P * g->P * g->P * es;
  return 8 * ((reg + 255) / 256 * 256);
}

template <typename T>
static hipError_t sync_adj_t(const wacm_grid* g, T* Ub, hipStream_t st) {
  const AdjPlan& pl = g->plan[0];
  const int64_t fs = (int64_t)g->P * g->P * g->P;
  if (pl.nrows > 0)
    sync_adj_gather<T><<<grid_n((pl.nrows + NT_GEN - 1) / NT_GEN), NT_GEN, 0, st>>>(
        pl.d_dst, pl.d_ptr, pl.d_src, pl.d_w, pl.nrows, Ub, fs);
  if (pl.nghost > 0)
    zero_points<T><<<grid_n((pl.nghost + NT_GEN - 1) / NT_GEN), NT_GEN, 0, st>>>(
        pl.d_ghost, pl.nghost, Ub, fs);
  return hipGetLastError();
}

hipError_t launch_sync_adj(const wacm_grid* g, void* Ub, hipStream_t st) {
  return g->d.dtype == WACM_F64 ? sync_adj_t(g, (double*)Ub, st) : sync_adj_t(g, (float*)Ub, st);
}

template <typename T>
static AdjArgs<T> adj_args(const wacm_grid* g, const wacm_params* p, double t, const T* U,
                           const T* V, T* Ub, double* dusbar, const T* dus) {
  AdjArgs<T> a{};
  a.tab = g->d_tab;
  a.nb = g->nb;
  a.U = U;
  a.V = V;
  a.Ub = Ub;
  a.L = pool_L(g);
  a.bs = g->d.bs;
  a.Ldom = g->d.L;
  a.t = t;
  a.p = *p;
  a.dus = dus;
  a.dusbar = dusbar;
  a.part = g->d_part;
  return a;
}

template <typename T>
static hipError_t rhs_adj_t(const wacm_grid* g, const wacm_params* p, double t, const T* U,
                            const T* V, T* Ub, double* dtheta, double* dusbar, const T* dus,
                            hipStream_t st) {
  if (g->nb == 0) return hipSuccess;
  AdjArgs<T> a = adj_args<T>(g, p, t, U, V, Ub, dusbar, dus);
  rhs_adj_kernel<T><<<grid_n(g->nb), NT_GEN, 0, st>>>(a);
  theta_finalize<<<1, NT_GEN, 0, st>>>(g->d_part, g->nb, dtheta);
  return hipGetLastError();
}

hipError_t launch_rhs_adj(const wacm_grid* g, const wacm_params* p, double t, const void* U,
                          const void* V, void* Ub, double* dtheta, double* dusbar,
                          const void* dus, hipStream_t st) {
  return g->d.dtype == WACM_F64
             ? rhs_adj_t(g, p, t, (const double*)U, (const double*)V, (double*)Ub, dtheta,
                         dusbar, (const double*)dus, st)
             : rhs_adj_t(g, p, t, (const float*)U, (const float*)V, (float*)Ub, dtheta, dusbar,
                         (const float*)dus, st);
}

template <typename T, int BS>
static void force_adj_launch(const wacm_grid* g, const AdjArgs<T>& a, hipStream_t st) {
  if (a.p.mask == WACM_MASK_PLATE)
    force_adj_kernel<T, BS, true><<<grid_n(g->nb), NT_GEN, 0, st>>>(a);
  else
    force_adj_kernel<T, BS, false><<<grid_n(g->nb), NT_GEN, 0, st>>>(a);
}

template <typename T>
static hipError_t force_adj_t(const wacm_grid* g, const wacm_params* p, double t, double weight,
                              const T* U, T* Ub, double* dtheta, double* dusbar, const T* dus,
                              hipStream_t st) {
  if (g->nb == 0 || !p->mask) return hipSuccess;
  AdjArgs<T> a = adj_args<T>(g, p, t, U, nullptr, Ub, dusbar, dus);
  a.weight = weight;
  switch (g->d.bs) {
    case 16:
      force_adj_launch<T, 16>(g, a, st);
      break;
    case 24:
      force_adj_launch<T, 24>(g, a, st);
      break;
    case 32:
      force_adj_launch<T, 32>(g, a, st);
      break;
    default:
      return hipErrorInvalidValue;
  }
  theta_finalize<<<1, NT_GEN, 0, st>>>(g->d_part, g->nb, dtheta);
  return hipGetLastError();
}

hipError_t launch_force_adj(const wacm_grid* g, const wacm_params* p, double t, double weight,
                            const void* U, void* Ub, double* dtheta, double* dusbar,
                            const void* dus, hipStream_t st) {
  return g->d.dtype == WACM_F64
             ? force_adj_t(g, p, t, weight, (const double*)U, (double*)Ub, dtheta, dusbar,
                           (const double*)dus, st)
             : force_adj_t(g, p, t, weight, (const float*)U, (float*)Ub, dtheta, dusbar,
                           (const float*)dus, st);
}

// Work buffer of one adjoint step (within the 8 pool registers of
// wacm_adj_work_bytes): the stage inputs Y2, Y3, Y4 (x-split), two rhs
// adjoints and the running sum (compact), the face halos of the stage input,
// the face buffer (FP64) and the reduction partials: per slot 24 bs^3 values
// in the registers and at most 217 bs^2 (FP32) in the rest, of the 32 (bs +
// 2 ng)^3, ng >= 3, of the pool registers.
template <typename T>
struct AdjWork {
  T *y[3], *k[2], *sum, *hb;
  double *fb, *bad, *part;
};
template <typename T>
static AdjWork<T> adj_work(const wacm_grid* g, void* work) {
  const size_t cap = (size_t)g->d.capacity, bs = g->d.bs;
  const size_t reg = up256(cap * 4 * bs * bs * bs * sizeof(T)), hb = up256(cap * 72 * bs * bs * sizeof(T));
  char* w = (char*)work;
  AdjWork<T> r;
  for (int i = 0; i < 3; ++i) r.y[i] = (T*)(w + i * reg);
  for (int i = 0; i < 2; ++i) r.k[i] = (T*)(w + (3 + i) * reg);
  r.sum = (T*)(w + 5 * reg);
  r.hb = (T*)(w + 6 * reg);
  r.fb = (double*)(w + 6 * reg + hb);
  r.bad = r.fb + cap * 72 * bs * bs;
  r.part = r.bad + cap * 4;  // at most 4 stage items per block
  return r;
}

// the stage itself, grid of as many workgroups as are resident
template <typename T, int BS, int TY, bool FIRST, bool LAST>
static void adj_stage_main(const AdjStage<T>& a, hipStream_t st) {
  static const int resident = [] {
    int n = 0, dev = 0, cus = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, adj_stage_kernel<T, BS, TY, FIRST, LAST>,
                                                     BS * TY, 0) != hipSuccess ||
        n < 1)
      n = 1;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        cus < 1)
      cus = 256;
    return n * cus;
  }();
  const int64_t items = a.nb * (BS / TY);
  adj_stage_kernel<T, BS, TY, FIRST, LAST>
      <<<(unsigned)std::min<int64_t>(items, resident), BS * TY, 0, st>>>(a);
}

// one stage backwards
template <typename T, int BS, int TY>
static hipError_t adj_stage_launch(const wacm_grid* g, const AdjStage<T>& a, double* fb,
                                   double* dtheta, hipStream_t st) {
  const AdjPlan& pl = g->plan[1];
  if (g->n_cface > 0)
    adj_face_kernel<T, BS><<<grid_n(g->n_cface), NT_GEN, 0, st>>>(g->d_tab, g->d_cface,
                                                                  g->n_cface, a, fb);
  if (!a.kn)
    adj_stage_main<T, BS, TY, false, true>(a, st);
  else if (!a.sum)
    adj_stage_main<T, BS, TY, true, false>(a, st);
  else
    adj_stage_main<T, BS, TY, false, false>(a, st);
  if (a.p.mask || a.p.sponge) {
    const int64_t n = a.nb * (BS / ADJ_PZ);
    adj_pen_kernel<T, BS, BS / TY><<<grid_n(n, 8192), NT_GEN, 0, st>>>(a);
    if (a.p.mask) theta_finalize<<<1, NT_GEN, 0, st>>>(a.part, n, dtheta);
  }
  if (pl.nrows > 0)
    adj_gather_kernel<T><<<grid_n((pl.nrows + NT_GEN - 1) / NT_GEN), NT_GEN, 0, st>>>(
        pl.d_dst, pl.d_ptr, pl.d_src, pl.nrows, BS, fb, a);
  return hipGetLastError();
}

// One RK4 step backwards: recompute the stage inputs from the checkpoint Un,
// then sweep the stages in reverse:
//   kb_4 = dt/6 lam, kb_3 = dt/3 lam + dt B_4, kb_2 = dt/3 lam + dt/2 B_3,
//   kb_1 = dt/6 lam + dt/2 B_2, with B_s = S^T J_rhs(U_s)^T kb_s, and
//   lam_n = lam + B_4 + B_3 + B_2 + B_1.
// Each stage is four kernels: what the faces next to other levels return
// (from kb and the input), the stage itself, the mask's and sponge's pointwise
// terms, and the gather of the former.
// 1632 blocks of 16^3 (plate), FP32, three steps of the functional and its
// gradient: 51.4 -> 10.3 ms.
template <typename T>
static hipError_t rk4_adj_t(const wacm_grid* g, const wacm_params* p, double t, double dt,
                            const T* Un, T* lam, double* dtheta, double* dusbar, const T* dus,
                            void* work, hipStream_t st) {
  if (g->nb == 0) return hipSuccess;
  const Layout L = pool_L(g);
  Layout Lc;
  Lc.P = g->d.bs;
  Lc.ng = 0;
  Lc.fstride = (int64_t)g->d.bs * g->d.bs * g->d.bs;
  Lc.bstride = 4 * Lc.fstride;
  Layout Lx = Lc;
  Lx.xs = 1;
  const AdjWork<T> w = adj_work<T>(g, work);
  const T* in[4] = {Un, w.y[0], w.y[1], w.y[2]};
  const double cs[4] = {0.0, 0.5, 0.5, 1.0};
  const double lamw[4] = {dt / 6.0, dt / 3.0, dt / 3.0, dt / 6.0};
  hipError_t e;
  for (int s = 1; s < 4; ++s)
    if ((e = launch_stage_input(g, p, s, t, dt, Un, in[s - 1], w.y[s - 1], w.hb, dus, st)) !=
        hipSuccess)
      return e;
  AdjStage<T> a{};
  a.tab = g->d_tab;
  a.nb = g->nb;
  a.hb = w.hb;
  a.lam = lam;
  a.Lp = L;
  a.Lc = Lc;
  a.Ldom = g->d.L;
  a.p = *p;
  a.dus = dus;
  a.dusbar = dusbar;
  a.bad = w.bad;
  a.part = w.part;
  for (int s = 3; s >= 0; --s) {
    a.u = in[s];
    a.Lu = s == 0 ? L : Lx;
    a.t = t + cs[s] * dt;
    a.v = s == 3 ? lam : w.k[(s + 1) & 1];
    a.Lv = s == 3 ? L : Lc;
    a.vs = s == 3 ? T(lamw[3]) : T(1);
    a.sum = s == 3 ? nullptr : w.sum;
    a.sout = s == 0 ? lam : w.sum;
    a.Lso = s == 0 ? L : Lc;
    a.kn = s == 0 ? nullptr : w.k[s & 1];
    a.lamw = s == 0 ? T(0) : T(lamw[s - 1]);
    a.kw = T(cs[s] * dt);
    if ((e = launch_nlface(g, a.u, a.Lu, w.hb, st)) != hipSuccess) return e;
    switch (g->d.bs) {
      case 16:
        e = adj_stage_launch<T, 16, 16>(g, a, w.fb, dtheta, st);
        break;
      case 24:
        e = adj_stage_launch<T, 24, 8>(g, a, w.fb, dtheta, st);
        break;
      case 32:
        e = adj_stage_launch<T, 32, 8>(g, a, w.fb, dtheta, st);
        break;
      default:
        e = hipErrorInvalidValue;
    }
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_rk4_adj(const wacm_grid* g, const wacm_params* p, double t, double dt,
                          const void* Un, void* lam, double* dtheta, double* dusbar,
                          const void* dus, void* work, hipStream_t st) {
  return g->d.dtype == WACM_F64
             ? rk4_adj_t(g, p, t, dt, (const double*)Un, (double*)lam, dtheta, dusbar,
                         (const double*)dus, work, st)
             : rk4_adj_t(g, p, t, dt, (const float*)Un, (float*)lam, dtheta, dusbar,
                         (const float*)dus, work, st);
}

}  // namespace wacm
