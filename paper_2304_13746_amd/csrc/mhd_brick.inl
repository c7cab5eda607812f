// mhd_brick.inl -- one FP64 stage of the default scheme on small boxes (gfx950).
//
// The marching kernel (mhd_stage.inl) solves the x-, y- and z-face of a column one after
// another, plane after plane.  A box that cannot fill the GPU with such columns is bound
// by that chain: with one plane per block a 32^3 stage took 27 us, three planes of 7 us
// and the loads before them, at one wave per SIMD.  Here a block owns a brick of cells and
// every face of it, and of the ring that the corner EMFs read, is a task of its own: 924
// faces of an 8 x 4 x 4 brick over 1024 threads, or 348 of a 4 x 4 x 2 brick over 512.
// Faces near the ring are solved by several blocks (7 and 11 per cell, against 4 in the
// march), so it pays only where every block has a CU of its own (launch_stage has the
// rule).  Measured per RK2 cycle, march against bricks: 16^3 51 against 29 us (8x4x4)
// and 20 us (4x4x2), 32^3 58 against 38 us; 48^3, 864 bricks, 89 against 118 us.
//
// Phases, a barrier between them: primitives of the brick and its halo to LDS; faces and
// cell EMFs; corner EMFs; updates.  The direction of a face or an edge is a number, not
// a template argument, so a wave never runs two directions' code.  Every expression is
// that of the marching kernel, so results have its bits.  (In FP32 the compiler contracts
// some of them differently here, so FP32 boxes march at every size.)
#pragma once

namespace mhd {

template <typename R, bool HY, int SHAPE>
struct Brick {
  static constexpr int BX = kBrick[SHAPE].x, BY = kBrick[SHAPE].y, BZ = kBrick[SHAPE].z;
  static constexpr int NT = kBrick[SHAPE].threads;
  static constexpr int CELLS = BX * BY * BZ;
  // primitives with a two-cell halo
  static constexpr int WX = BX + 4, WY = BY + 4, WZ = BZ + 4, NW = WX * WY * WZ;
  // cells with a one-cell halo: own faces' fields and cell EMFs
  static constexpr int RX = BX + 2, RY = BY + 2, RZ = BZ + 2, NR = RX * RY * RZ;
  // faces per direction: with corner EMFs a ring around the brick in the transverse
  // directions, without (the field-free build) the brick's own
  static constexpr int G = HY ? 0 : 1;  // ring width
  static constexpr int NX = (BX + 1) * (BY + 2 * G) * (BZ + 2 * G);
  static constexpr int NY = (BX + 2 * G) * (BY + 1) * (BZ + 2 * G);
  static constexpr int NZ = (BX + 2 * G) * (BY + 2 * G) * (BZ + 1);
  static constexpr int NF = NX + NY + NZ;
  // edges per direction
  static constexpr int EX = BX * (BY + 1) * (BZ + 1), EY = (BX + 1) * BY * (BZ + 1);
  static constexpr int EZ = (BX + 1) * (BY + 1) * BZ, NE = EX + EY + EZ;
  static constexpr int NV = HY ? 5 : 8;
  struct Smem {
    R w[NV][NW];
    R cons[5][NF], cmax[NF];           // grid-frame fluxes and signal speeds
    R ea[HY ? 1 : NF], eb[HY ? 1 : NF];  // the faces' EMFs along t2 and t1
    R bf[HY ? 1 : 3][HY ? 1 : NR];     // face fields
    R er[HY ? 1 : 3][HY ? 1 : NR];     // cell EMFs
    R e[HY ? 1 : NE];                  // corner EMFs
    R red[NT / 64];
  };
  __device__ static int wi(int i, int j, int k) { return ((k + 2) * WY + (j + 2)) * WX + (i + 2); }
  __device__ static int ri(int i, int j, int k) { return ((k + 1) * RY + (j + 1)) * RX + (i + 1); }
  // number of the lower face in direction d of cell (i, j, k)
  __device__ static int face(int d, int i, int j, int k) {
    const int sx = d == 0 ? BX + 1 : BX + 2 * G, sy = d == 1 ? BY + 1 : BY + 2 * G;
    const int oi = d == 0 ? 0 : G, oj = d == 1 ? 0 : G, ok = d == 2 ? 0 : G;
    return (d == 0 ? 0 : d == 1 ? NX : NX + NY) + ((k + ok) * sy + (j + oj)) * sx + (i + oi);
  }
  __device__ static void face_cell(int f, int& d, int& i, int& j, int& k) {
    d = f < NX ? 0 : f < NX + NY ? 1 : 2;
    f -= d == 0 ? 0 : d == 1 ? NX : NX + NY;
    const int sx = d == 0 ? BX + 1 : BX + 2 * G, sy = d == 1 ? BY + 1 : BY + 2 * G;
    i = f % sx;
    j = f / sx % sy;
    k = f / (sx * sy);
    i -= d == 0 ? 0 : G;
    j -= d == 1 ? 0 : G;
    k -= d == 2 ? 0 : G;
  }
  // number of the edge along d at the low corner of cell (i, j, k)
  __device__ static int edge(int d, int i, int j, int k) {
    const int sx = d == 0 ? BX : BX + 1, sy = d == 1 ? BY : BY + 1;
    return (d == 0 ? 0 : d == 1 ? EX : EX + EY) + (k * sy + j) * sx + i;
  }
  __device__ static void edge_cell(int n, int& d, int& i, int& j, int& k) {
    d = n < EX ? 0 : n < EX + EY ? 1 : 2;
    n -= d == 0 ? 0 : d == 1 ? EX : EX + EY;
    const int sx = d == 0 ? BX : BX + 1, sy = d == 1 ? BY : BY + 1;
    i = n % sx;
    j = n / sx % sy;
    k = n / (sx * sy);
  }
};

__device__ __forceinline__ int next_dir(int d) { return d == 2 ? 0 : d + 1; }

template <typename R, int SOLVER, int MODE, int SHAPE>
__global__ void __launch_bounds__(kBrick[SHAPE].threads)
__attribute__((amdgpu_waves_per_eu(kBrick[SHAPE].threads / 256)))
brick_kernel(BatchArgs ba) {
  constexpr bool HY = SOLVER == SOLVER_HLLC;
  using T = Brick<R, HY, SHAPE>;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  typename T::Smem& S = *reinterpret_cast<typename T::Smem*>(smem_raw);
  int b = blockIdx.x;
  int box = 0;
  while (box + 1 < ba.nbox && ba.start[box + 1] <= b) ++box;
  b -= ba.start[box];
  const BoxDesc* desc = ba.desc[box];
  StageArgs<R> a;
  const int si = ba.src[box], di = ba.dst[box], bi = ba.base[box];
  for (int f = 0; f < 8; ++f) {
    a.src[f] = static_cast<const R*>(desc->buf[si][f]);
    a.dst[f] = static_cast<R*>(desc->buf[di][f]);
  }
  a.boff = static_cast<const R*>(desc->buf[bi][0]) - static_cast<const R*>(desc->buf[di][0]);
  a.w = (R)ba.w;
  a.w0 = (R)ba.w0;
  a.nx = desc->nx; a.ny = desc->ny; a.nz = desc->nz;
  for (int q = 0; q < 3; ++q) a.idl[q] = (R)desc->idl[q];
  a.gamma = (R)desc->gamma;
  a.gm1 = (R)(desc->gamma - 1.0);
  a.igm1 = (R)(1.0 / (desc->gamma - 1.0));
  a.scw = desc->sc;
  const int nbx = (a.nx + T::BX - 1) / T::BX, nby = (a.ny + T::BY - 1) / T::BY;
  const int x0 = b % nbx * T::BX, y0 = b / nbx % nby * T::BY, z0 = b / (nbx * nby) * T::BZ;
  const int t = threadIdx.x;

  // cycle control, as in the marching kernel
  double dtd;
  if (MODE == MODE_STAGE1 && ba.first) {
    dtd = clip_step(ld_agent(&a.scw->dt_next), ld_agent(&a.scw->t), ba.t_stop[box]);
    if (b == 0 && t == 0) st_agent(&a.scw->dt[ba.par], dtd);
  } else {
    dtd = ld_agent(&a.scw->dt[ba.par]);
  }
  if (MODE == MODE_COMBINE && ba.last && b == 0 && t == 0)
    end_cycle(a.scw, ba.par, ba.t_stop[box]);
  const R dt = (R)dtd;
  const R tau[3] = {dt * a.idl[0], dt * a.idl[1], dt * a.idl[2]};
  const long long plane = (long long)a.nx * a.ny;

  // ---- primitives of the brick and its halo
  bool bad = false;
  for (int n = t; n < T::NW; n += T::NT) {
    const int i = n % T::WX - 2, j = n / T::WX % T::WY - 2, k = n / (T::WX * T::WY) - 2;
    const int out = (i < -1 || i > T::BX) + (j < -1 || j > T::BY) + (k < -1 || k > T::BZ);
    if (out > 1) continue;  // no face reads it
    const int gi = wrap_index(x0 + i, a.nx), gj = wrap_index(y0 + j, a.ny), gk = wrap_index(z0 + k, a.nz);
    const int gi1 = gi + 1 == a.nx ? 0 : gi + 1, gj1 = gj + 1 == a.ny ? 0 : gj + 1;
    const int gk1 = gk + 1 == a.nz ? 0 : gk + 1;
    Raw<R> r;
    Cell<R> c;
    load_raw<HY>(a, gi, gi1, gj, gj1, gk, gk1, r);
    to_prim(r.rho, r.mx, r.my, r.mz, r.en, r.bxl, r.bxr, r.byl, r.byr, r.bzl, r.bzr, a.gm1, c);
    put_cell<HY>(S, n, c);
    if constexpr (!HY) {
      if (out == 0) {
        const int m = T::ri(i, j, k);
        S.bf[0][m] = r.bxl;
        S.bf[1][m] = r.byl;
        S.bf[2][m] = r.bzl;
      }
    }
    if (i >= 0 && i < T::BX && j >= 0 && j < T::BY && k >= 0 && k < T::BZ && x0 + i < a.nx &&
        y0 + j < a.ny && z0 + k < a.nz)
      bad |= bad_cell(c);
  }
  __syncthreads();

  // ---- cell EMFs -(v x B), and every face
  if constexpr (!HY) {
    for (int n = t; n < T::NR; n += T::NT) {
      const int i = n % T::RX - 1, j = n / T::RX % T::RY - 1, k = n / (T::RX * T::RY) - 1;
      Cell<R> c;
      get_cell<HY>(S, T::wi(i, j, k), c);
      S.er[0][n] = c.vz * c.by - c.vy * c.bz;
      S.er[1][n] = c.vx * c.bz - c.vz * c.bx;
      S.er[2][n] = c.vy * c.bx - c.vx * c.by;
    }
  }
  for (int f = t; f < T::NF; f += T::NT) {
    int d, i, j, k;
    T::face_cell(f, d, i, j, k);
    const int d1 = next_dir(d), d2 = next_dir(d1);
    const int o = T::wi(i, j, k), step = d == 0 ? 1 : d == 1 ? T::WX : T::WX * T::WY;
    // the face-frame variables' fields in LDS
    const int var[7] = {0, 1 + d, 1 + d1, 1 + d2, HY ? 0 : 4 + d1, HY ? 0 : 4 + d2, HY ? 4 : 7};
    R ql[7], qr[7];
#pragma unroll
    for (int v = 0; v < 7; ++v) {
      if (HY && (v == 4 || v == 5)) {
        ql[v] = qr[v] = R(0);
        continue;
      }
      const R* q = S.w[var[v]] + o;
      const R q0 = q[-2 * step], q1 = q[-step], q2 = q[0], q3 = q[step];
      ql[v] = recon_hi<RECON_PLM>(q0, q1, q2);
      qr[v] = recon_lo<RECON_PLM>(q1, q2, q3);
    }
    const R bn = HY ? R(0) : S.bf[HY ? 0 : d][HY ? 0 : T::ri(i, j, k)];
    R g[7], cmax;
    riemann<SOLVER>(a.gamma, a.igm1, as_prim(ql), as_prim(qr), bn, g, cmax);
    S.cons[0][f] = g[0];
    S.cons[1 + d][f] = g[1];
    S.cons[1 + d1][f] = g[2];
    S.cons[1 + d2][f] = g[3];
    S.cons[4][f] = g[4];
    S.cmax[f] = cmax;
    if constexpr (!HY) {
      S.ea[f] = -g[5];
      S.eb[f] = g[6];
    }
  }
  __syncthreads();

  // ---- corner EMFs
  if constexpr (!HY) {
    for (int n = t; n < T::NE; n += T::NT) {
      int d, i, j, k;
      T::edge_cell(n, d, i, j, k);
      const int p = next_dir(d), q = next_dir(p);
      auto back = [&](int dir, int& bi_, int& bj_, int& bk_) {
        bi_ = i - (dir == 0);
        bj_ = j - (dir == 1);
        bk_ = k - (dir == 2);
      };
      int pi, pj, pk, qi, qj, qk;
      back(p, pi, pj, pk);
      back(q, qi, qj, qk);
      const int a1 = T::face(p, i, j, k), a2 = T::face(p, qi, qj, qk);
      const int b1 = T::face(q, i, j, k), b2 = T::face(q, pi, pj, pk);
      const int c11 = T::ri(i, j, k), c01 = T::ri(pi, pj, pk), c10 = T::ri(qi, qj, qk);
      const int c00 = c01 + c10 - c11;
      const R* er = S.er[d];
      S.e[n] = corner_emf<EMF_EC>(S.ea[a1], S.ea[a2], S.eb[b1], S.eb[b2], er[c00], er[c10], er[c01],
                                  er[c11], S.cons[0][a1], S.cons[0][a2], S.cons[0][b1], S.cons[0][b2]);
    }
    __syncthreads();
  }

  // ---- updates: threads over (field, cell); the CFL condition by those of field 0
  R inv = R(0);
  {
    static_assert(T::NT % T::CELLS == 0, "a thread keeps its cell");
    const int c = t % T::CELLS;
    const int i = c % T::BX, j = c / T::BX % T::BY, k = c / (T::BX * T::BY);
    const int gi = x0 + i, gj = y0 + j, gk = z0 + k;
    if (gi < a.nx && gj < a.ny && gk < a.nz) {
      const long long o = (long long)gk * plane + (long long)gj * a.nx + gi;
      const int f0 = T::face(0, i, j, k), f1 = T::face(1, i, j, k), f2 = T::face(2, i, j, k);
      const int n0 = T::face(0, i + 1, j, k), n1 = T::face(1, i, j + 1, k), n2 = T::face(2, i, j, k + 1);
      if constexpr (MODE != MODE_COMBINE) {
        if (t < T::CELLS) {
          const R cx = S.cmax[f0] > S.cmax[n0] ? S.cmax[f0] : S.cmax[n0];
          const R cy = S.cmax[f1] > S.cmax[n1] ? S.cmax[f1] : S.cmax[n1];
          const R cz = S.cmax[f2] > S.cmax[n2] ? S.cmax[f2] : S.cmax[n2];
          const R cxy = cx * a.idl[0] + cy * a.idl[1];
          const R v = cxy + cz * a.idl[2];
          inv = v > inv ? v : inv;
        }
      }
      for (int q = t / T::CELLS; q < 8; q += T::NT / T::CELLS) {
        const R* src = a.src[0];
        R* dst = a.dst[0];
#pragma unroll
        for (int f = 1; f < 8; ++f) {
          src = q == f ? a.src[f] : src;
          dst = q == f ? a.dst[f] : dst;
        }
        R un;
        if (q < 5) {
          const R* F = S.cons[q];
          const R part = (gld(src, o) - tau[0] * (F[n0] - F[f0])) - tau[1] * (F[n1] - F[f1]);
          un = part - tau[2] * (F[n2] - F[f2]);
        } else if constexpr (HY) {
          gst(dst, o, R(0));
          continue;
        } else {
          const int d = q - 5, p = next_dir(d), r = next_dir(p);
          const int er0 = T::edge(r, i, j, k), ep0 = T::edge(p, i, j, k);
          const int er1 = T::edge(r, i + (p == 0), j + (p == 1), k + (p == 2));
          const int ep1 = T::edge(p, i + (r == 0), j + (r == 1), k + (r == 2));
          const R tp = p == 0 ? tau[0] : p == 1 ? tau[1] : tau[2];
          const R tr = r == 0 ? tau[0] : r == 1 ? tau[1] : tau[2];
          un = (S.bf[d][T::ri(i, j, k)] - tp * (S.e[er1] - S.e[er0])) + tr * (S.e[ep1] - S.e[ep0]);
        }
        if constexpr (MODE == MODE_COMBINE) un = a.w * un + a.w0 * gld<R>(dst, o + a.boff);
        gst(dst, o, un);
      }
    }
  }
  if constexpr (MODE != MODE_COMBINE) {
    for (int off = 32; off > 0; off >>= 1) {
      const R o = __shfl_xor(inv, off);
      inv = o > inv ? o : inv;
    }
    if ((t & 63) == 0) S.red[t >> 6] = inv;
    __syncthreads();
    if (t == 0) {
      for (int q = 1; q < T::NT / 64; ++q) inv = S.red[q] > inv ? S.red[q] : inv;
      atomic_max_pos(&a.scw->invdt_bits, inv);
    }
  }
  if (__any(bad)) {
    if ((t & 63) == 0)
      __hip_atomic_fetch_or(&a.scw->status, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

template <typename R, int SOLVER, int MODE, int SHAPE>
static hipError_t launch_brick_mode(const BatchArgs& ba, hipStream_t st, bool prepare) {
  using Smem = typename Brick<R, SOLVER == SOLVER_HLLC, SHAPE>::Smem;
  static_assert(sizeof(Smem) <= 160 * 1024, "LDS of a CU");
  auto fn = brick_kernel<R, SOLVER, MODE, SHAPE>;
  if (prepare)
    return hipFuncSetAttribute(reinterpret_cast<const void*>(fn),
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)sizeof(Smem));
  hipLaunchKernelGGL(fn, dim3(ba.total), dim3(kBrick[SHAPE].threads), sizeof(Smem), st, ba);
  return hipGetLastError();
}

template <typename R, int SOLVER, int SHAPE>
static hipError_t launch_brick(const BatchArgs& ba, hipStream_t st, bool prepare) {
  if (prepare) {
    hipError_t e = launch_brick_mode<R, SOLVER, MODE_STAGE1, SHAPE>(ba, st, true);
    return e == hipSuccess ? launch_brick_mode<R, SOLVER, MODE_COMBINE, SHAPE>(ba, st, true) : e;
  }
  if (ba.mode == MODE_STAGE1) return launch_brick_mode<R, SOLVER, MODE_STAGE1, SHAPE>(ba, st, false);
  if (ba.mode == MODE_COMBINE) return launch_brick_mode<R, SOLVER, MODE_COMBINE, SHAPE>(ba, st, false);
  return hipErrorInvalidValue;
}

}  // namespace mhd
