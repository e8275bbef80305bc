// Momentum sub-step (Sec. 3, Eq. (substep1)) on single-level meshes: H(v) = -A[v] + nu D[v]
// with QUICK convection in flux form (upwinded on the advecting velocity, frozen at u^n) and
// 7-point diffusion, for explicit Euler / Adams-Bashforth steps and the Jacobi iterations of
// the Crank-Nicolson system.
//
// QUICK reaches two cells upwind, so the halo is two layers deep.  The y and z layers of a
// neighbour are rows and planes of its cube (whole lines), read from the field itself, which
// no pass writes while it is read (the iteration alternates between two arrays).  The x
// layers are two values per row: the first pass of a step reads them from the caller's field,
// the Crank-Nicolson sweeps from a face buffer that each pass writes for its own output (and
// the first pass for the x component of u^n): per cube and component [face][k][j][2], the
// cells i = 0, 1 of face 0 (-x) and i = n-2, n-1 of face 1 (+x), in the order of i.  On a
// domain face the two ghost layers mirror the cube's own two boundary layers: Dirichlet value
// g gives 2 g - v, zero gradient gives v (inflow: every component Dirichlet, the normal one
// U_in into the domain; slip: normal component Dirichlet 0, tangential zero gradient; open:
// zero gradient).
//
// Layout: lane l of a cube's n^2 lanes owns column (i, j) and walks it plane by plane, with the
// z neighbours k-2..k+2 in a register window and the flux through the lower z face carried up.
// The x neighbours are other lanes of the same row of 16 lanes, fetched by DPP row shifts whose
// out-of-row lanes take the halo values; the y neighbours go through LDS (two planes in turn,
// one barrier a plane), where each lane also puts its share of the ring rows.  What plane k + 1
// needs is loaded before plane k is computed.  Arithmetic is FP64 whatever the field type.
//
// What bounds it: HBM, with what two waves a SIMD keep in flight.  A Crank-Nicolson sweep of
// 33.5M cells in FP64 takes 0.81 ms and moves 4.0 GB (96 bytes per cell are 3.2 GB; the rest is
// halo rows, planes and the face buffers), 4.9 TB/s; the VALU is busy 43% of it.  With every
// neighbour through LDS, two barriers a plane and nothing loaded ahead it took 1.00 ms, and a
// separate export pass 0.2 ms a step.  About 250 registers: three waves a SIMD spill 90 of them
// and take three times as long; reading the y neighbours from memory instead of LDS keeps the L1
// path busy 65% of the time (0.98 ms).
#include "kernels.hpp"
#include "tile.hpp"

namespace bcm {

namespace {

template <int NL>
struct Mom {
  static constexpr int N2 = NL * NL, N3 = N2 * NL;
  static constexpr int CPB = NL >= 16 ? 1 : 256 / N2;
  static constexpr int FS = 4 * N2;  // face-buffer values per cube and component
  __device__ static int fidx(int f, int j, int q) { return (f * N2 + j) * 2 + q; }  // + 2 NL k
};

// Value v of component comp mirrored across domain face f of kind kd.
__device__ __forceinline__ double mom_ghost(double v, int kd, int f, int comp, double U_in) {
  const int d = f >> 1;
  if (kd == FK_INFLOW) return 2.0 * (comp == d ? ((f & 1) ? -U_in : U_in) : 0.0) - v;
  if (kd == FK_SLIP && comp == d) return -v;
  return v;  // an open face, or a tangential component on a slip wall
}

// v of the lane C (a DPP control) away, within the row of 16 lanes; `old` where there is none.
template <int C>
__device__ __forceinline__ double dpp64(double old, double v) {
  const int lo = __builtin_amdgcn_update_dpp(__double2loint(old), __double2loint(v), C, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(__double2hiint(old), __double2hiint(v), C, 0xf, 0xf, false);
  return __hiloint2double(hi, lo);
}
constexpr int kRowShl = 0x100, kRowShr = 0x110;  // + distance: from the lane above / below

// The cells i-2, i-1, i+1, i+2 of the lane's x line from its cell v and the halo value hx (on
// lanes i = 0, 1: cells -2, -1; on i = n-2, n-1: cells n, n+1).
template <int NL>
__device__ __forceinline__ void x_line(double v, double hx, int i, double (&w)[5]) {
  const double hm = dpp64<kRowShl + 1>(hx, hx), hp = dpp64<kRowShr + 1>(hx, hx);
  w[2] = v;
  if constexpr (NL == 16) {  // a line is a DPP row
    w[0] = dpp64<kRowShr + 2>(hx, v);
    w[1] = dpp64<kRowShr + 1>(hm, v);
    w[3] = dpp64<kRowShl + 1>(hp, v);
    w[4] = dpp64<kRowShl + 2>(hx, v);
  } else {
    const double m2 = dpp64<kRowShr + 2>(v, v), m1 = dpp64<kRowShr + 1>(v, v);
    const double p1 = dpp64<kRowShl + 1>(v, v), p2 = dpp64<kRowShl + 2>(v, v);
    w[0] = i < 2 ? hx : m2;
    w[1] = i < 1 ? hm : m1;
    w[3] = i > NL - 2 ? hp : p1;
    w[4] = i > NL - 3 ? hx : p2;
  }
}

// QUICK value on the face between b and c of the line a, b, c, d, upwind on U.
__device__ __forceinline__ double quick(double U, double a, double b, double c, double d) {
  const bool pos = U >= 0.0;
  const double near = pos ? b : c, next = pos ? c : b, far = pos ? a : d;
  return 0.75 * near + 0.375 * next - 0.125 * far;
}

// What the lane reads for one plane besides its own column: the x halo value of each component,
// the right-hand side (or previous H), its share of the y ring and, in a Crank-Nicolson sweep,
// the advecting velocity's x component (own and halo) and y component.
template <typename TF, int RN>
struct MomPlane {
  TF x[3], q[3], ring[RN], ax, hax, ay;
};

// One pass of H over every cube (see MomArgs for the modes).  OFF: the type of a byte offset
// within one field (32 bits where the fields are below 4 GiB: a load is then a scalar base
// plus one register).  NT: the output and a sweep's right-hand side bypass the caches.
template <typename TF, int NL, int MODE, typename OFF, bool NT>
__global__ __launch_bounds__(256, 2) void k_mom(MomArgs<TF> a) {
  using M = Mom<NL>;
  constexpr bool ITER = MODE == MOM_CN_ITER;
  constexpr int NA = ITER ? 4 : 3;            // arrays in LDS: v and, in a sweep, a_y
  constexpr int PL = (NL + 4) * NL;           // one of their planes, with two ring rows a side
  constexpr int RE = (ITER ? 14 : 12) * NL;   // ring values of a plane (a_y needs one row a side)
  constexpr int RN = (RE + M::N2 - 1) / M::N2;
  __shared__ double pl[2][M::CPB][NA][PL];    // planes k and k + 1 in turn: one barrier a plane
  __shared__ double red[8];
  const int t = threadIdx.x;
  const int s = M::CPB == 1 ? 0 : t / M::N2, l = M::CPB == 1 ? t : t % M::N2, i = l % NL, j = l / NL;
  const int units = col_units(M::CPB, a.n_cubes);
  const bool xlo = i < 2, xhi = i >= NL - 2;  // lanes that hold x halo values
  auto ld = [](const TF* p, OFF byte) { return *reinterpret_cast<const TF*>(reinterpret_cast<const char*>(p) + byte); };
  auto ldn = [](const TF* p, OFF byte) { return ld_nt(reinterpret_cast<const TF*>(reinterpret_cast<const char*>(p) + byte)); };
  constexpr OFF B = sizeof(TF);
  double acc = 0.0;
  for (int u = blockIdx.x; u < units; u += gridDim.x) {
    const int p = M::CPB == 1 ? u : ((u >> 3) * M::CPB + s) * 8 + (u & 7);
    int c = p < a.n_cubes ? a.launch[p] : -1;
    if (M::N2 >= 64) c = __builtin_amdgcn_readfirstlane(c);  // one cube per wavefront
    const bool live = M::CPB == 1 || c >= 0;
    const int ce = live ? c : 0;
    const CubeMeta& m = a.meta[ce];
    int kd[6], nb[6];  // face kinds; the cube across, or this one behind a domain face
#pragma unroll
    for (int f = 0; f < 6; ++f) {
      kd[f] = m.kind[f];
      nb[f] = kd[f] == FK_SAME ? m.nbr[f][0] : ce;
      if (M::N2 >= 64) {
        kd[f] = __builtin_amdgcn_readfirstlane(kd[f]);
        nb[f] = __builtin_amdgcn_readfirstlane(nb[f]);
      }
    }
    const double ih = 1.0 / m.h, ih2 = ih * ih;
    const OFF own = ((OFF)ce * M::N3 + l) * B;
    // the lane's ring values: array e / (4 NL), ring row e / NL % 4 (j = -2, -1, NL, NL + 1; of
    // a_y only the inner two), cell e % NL
    const TF* rp[RN];
    int rdst[RN], rwall = 0;
#pragma unroll
    for (int r = 0; r < RN; ++r) {
      const int e = l + r * M::N2, arr = e / (4 * NL);
      int q = e / NL % 4;
      if (arr == 3) q += 1;  // rows NL * 12.. : j = -1 and NL
      const int f = q < 2 ? 2 : 3, ii = e % NL;
      const bool same = kd[f] == FK_SAME;
      const int row = q < 2 ? (same ? NL - 2 + q : 1 - q) : (same ? q - 2 : NL + 1 - q);
      const TF* base = arr == 0 ? a.v[0] : arr == 1 ? a.v[1] : arr == 2 ? a.v[2] : a.a[1];
      rp[r] = base + (size_t)nb[f] * M::N3 + row * NL + ii;
      rdst[r] = e < RE ? arr * PL + (q < 2 ? q : NL + q) * NL + ii : -1;
      if (!same) rwall |= 1 << r;
    }
    const bool xwall = (xlo && kd[0] != FK_SAME) || (xhi && kd[1] != FK_SAME);
    const int xf = xlo ? 0 : 1, xk = xlo ? kd[0] : kd[1];
    // x halo of the lane's row (lanes xlo, xhi; the others read a value that is not used): the
    // neighbour's cell, or this cube's mirrored one; in the field and in the face buffers
    const int xcube = xlo ? nb[0] : nb[1];
    const int xcell = xlo ? (xwall ? 1 - i : NL - 2 + i) : xhi ? (xwall ? 2 * NL - 3 - i : i - (NL - 2)) : 0;
    const int side = xwall ? xf : 1 - xf;
    const OFF xo = ITER ? ((OFF)xcube * M::FS + M::fidx(side, j, xlo || xhi ? xcell - (side ? NL - 2 : 0) : 0)) * B
                        : ((OFF)xcube * M::N3 + j * NL + xcell) * B;
    const OFF fb = ((OFF)ce * M::FS + M::fidx(xf, j, xlo ? i : i - (NL - 2))) * B;  // the lane's own cell there
    // z windows of the lane's column, rotated plane by plane: v at k-2..k+2 and a_z at k-1..k+1.
    // Byte offset of plane k of the column, -2 <= k < NL + 2 (behind a wall: of its mirror)
    auto plane = [&](int k) -> OFF {
      const int kl = kd[4] == FK_SAME ? k + NL : -1 - k, kh = kd[5] == FK_SAME ? k - NL : 2 * NL - 1 - k;
      const int cube = k < 0 ? nb[4] : k < NL ? ce : nb[5], kk = k < 0 ? kl : k < NL ? k : kh;
      return ((OFF)cube * M::N3 + kk * M::N2 + l) * B;
    };
    const bool zwall_lo = kd[4] != FK_SAME, zwall_hi = kd[5] != FK_SAME;
    using In = MomPlane<TF, RN>;
    auto fetch = [&](In& in, int k) __attribute__((always_inline)) {
#pragma unroll
      for (int comp = 0; comp < 3; ++comp) {
        in.x[comp] = ITER ? ld(a.vf[comp] + k * (2 * NL), xo) : ld(a.v[comp] + k * M::N2, xo);
        in.q[comp] = TF(0);
        if (ITER) in.q[comp] = NT ? ldn(a.rhs[comp] + k * M::N2, own) : ld(a.rhs[comp] + k * M::N2, own);
        if (MODE == MOM_EXPLICIT && a.hprev[comp]) in.q[comp] = ld(a.hprev[comp] + k * M::N2, own);
      }
#pragma unroll
      for (int r = 0; r < RN; ++r) in.ring[r] = rp[r][k * M::N2];
      if (ITER) {
        in.ax = ld(a.a[0] + k * M::N2, own);
        in.hax = ld(a.af + k * (2 * NL), xo);
        in.ay = ld(a.a[1] + k * M::N2, own);
      }
    };
    double wv[3][5], za[3], fz[3];
    In cur;
    {
      TF wr[3][5], zr[3];
#pragma unroll
      for (int q = 0; q < 5; ++q) {
        const OFF o = plane(q - 2);
#pragma unroll
        for (int comp = 0; comp < 3; ++comp) wr[comp][q] = ld(a.v[comp], o);
        if (ITER && q > 0 && q < 4) zr[q - 1] = ld(a.a[2], o);
      }
      fetch(cur, 0);
#pragma unroll
      for (int comp = 0; comp < 3; ++comp) {
#pragma unroll
        for (int q = 0; q < 5; ++q) {
          wv[comp][q] = double(wr[comp][q]);
          if (q < 2 && zwall_lo) wv[comp][q] = mom_ghost(wv[comp][q], kd[4], 4, comp, a.U_in);
        }
      }
#pragma unroll
      for (int q = 0; q < 3; ++q) za[q] = ITER ? double(zr[q]) : wv[2][q + 1];
      if (ITER && zwall_lo) za[0] = mom_ghost(za[0], kd[4], 4, 2, a.U_in);
    }
    {
      const double U = 0.5 * (za[0] + za[1]);  // flux through the -z face, carried upwards
#pragma unroll
      for (int comp = 0; comp < 3; ++comp) fz[comp] = U * quick(U, wv[comp][0], wv[comp][1], wv[comp][2], wv[comp][3]);
    }
    double po[3] = {0.0, 0.0, 0.0}, ph[3] = {0.0, 0.0, 0.0}, pr[3] = {0.0, 0.0, 0.0}, pa = 0.0;
    auto put = [&](int kp) __attribute__((always_inline)) {
      if (!live) return;
      auto st = [](TF* p, OFF byte, double v) { *reinterpret_cast<TF*>(reinterpret_cast<char*>(p) + byte) = TF(v); };
      auto stn = [](TF* p, OFF byte, double v) { st_nt(reinterpret_cast<TF*>(reinterpret_cast<char*>(p) + byte), TF(v)); };
#pragma unroll
      for (int comp = 0; comp < 3; ++comp) {
        if (NT) stn(a.out[comp] + kp * M::N2, own, po[comp]);
        else st(a.out[comp] + kp * M::N2, own, po[comp]);
        if (MODE == MOM_CN_START) st(a.rhs[comp] + kp * M::N2, own, pr[comp]);
        if (!ITER && a.hout[comp]) st(a.hout[comp] + kp * M::N2, own, ph[comp]);
      }
      if (MODE != MOM_EXPLICIT && (xlo || xhi)) {
#pragma unroll
        for (int comp = 0; comp < 3; ++comp) st(a.outf[comp] + kp * (2 * NL), fb, po[comp]);
        if (!ITER) st(a.af + kp * (2 * NL), fb, pa);
      }
    };
    // Plane k: the outputs of plane k - 1 are stored, the loads of plane k + 1 issued, and
    // plane k is computed from what was loaded a plane before (the vector-memory counter is in
    // order: a load issued after a store is not consumed before the store completes).
    auto step = [&](const In& in, In& next, int k, int buf) __attribute__((always_inline)) {
      if (k > 0) put(k - 1);
      TF nv[3], naz = TF(0);
      {
        const OFF o3 = plane(k + 3 <= NL + 1 ? k + 3 : NL + 1);  // (past the last one: not used)
#pragma unroll
        for (int comp = 0; comp < 3; ++comp) nv[comp] = ld(a.v[comp], o3);
        if (ITER) naz = ld(a.a[2], plane(k + 2));
      }
      if (k + 1 < NL) fetch(next, k + 1);
      double* y = &pl[buf][s][0][0];
      const int at = (j + 2) * NL + i;
#pragma unroll
      for (int comp = 0; comp < 3; ++comp) y[comp * PL + at] = wv[comp][2];
      const double ay1 = ITER ? double(in.ay) : wv[1][2];
      if (ITER) y[3 * PL + at] = ay1;
#pragma unroll
      for (int r = 0; r < RN; ++r) {
        double v = double(in.ring[r]);
        if (rwall >> r & 1) {
          const int e = l + r * M::N2, arr = e / (4 * NL), q = e / NL % 4 + (arr == 3 ? 1 : 0);
          v = mom_ghost(v, q < 2 ? kd[2] : kd[3], q < 2 ? 2 : 3, arr == 3 ? 1 : arr, a.U_in);
        }
        if (RE % M::N2 == 0 || rdst[r] >= 0) y[rdst[r]] = v;
      }
      double hx[3], hax = double(in.hax);
#pragma unroll
      for (int comp = 0; comp < 3; ++comp) hx[comp] = double(in.x[comp]);
      if (xwall) {
#pragma unroll
        for (int comp = 0; comp < 3; ++comp) hx[comp] = mom_ghost(hx[comp], xk, xf, comp, a.U_in);
        if (ITER) hax = mom_ghost(hax, xk, xf, 0, a.U_in);
      }
      double xa[5];
      x_line<NL>(ITER ? double(in.ax) : wv[0][2], ITER ? hax : hx[0], i, xa);
      __syncthreads();
      const int ya = (ITER ? 3 : 1) * PL + at;
      const double Ux[2] = {0.5 * (xa[1] + xa[2]), 0.5 * (xa[2] + xa[3])};
      const double Uy[2] = {0.5 * (y[ya - NL] + ay1), 0.5 * (ay1 + y[ya + NL])};
      const double Uz[2] = {0.5 * (za[0] + za[1]), 0.5 * (za[1] + za[2])};
      // interior Jacobi diagonal of H (Crank-Nicolson iterations): the coefficient of v(i)
      // in the two QUICK face values of each axis, and the diffusion's -6 nu / h^2
      double inv_diag = 0.0;
      if (ITER) {
        double dg = 0.0;  // Up (Up >= 0 ? 3/4 : 3/8) - Um (Um >= 0 ? 3/8 : 3/4) per axis
#pragma unroll
        for (int d = 0; d < 3; ++d) {
          const double Um = d == 0 ? Ux[0] : d == 1 ? Uy[0] : Uz[0];
          const double Up = d == 0 ? Ux[1] : d == 1 ? Uy[1] : Uz[1];
          dg += 0.5625 * (Up - Um) + 0.1875 * (fabs(Up) + fabs(Um));
        }
        dg *= ih;
        inv_diag = 1.0 / fmax(1.0 + 0.5 * a.dt * (6.0 * a.nu * ih2 + dg), 0.5);
      }
#pragma unroll
      for (int comp = 0; comp < 3; ++comp) {
        double w[5], H;
        const double v0 = wv[comp][2];
        const double* yc = y + comp * PL + at;
        const double y0 = yc[-2 * NL], y1 = yc[-NL], y3 = yc[NL], y4 = yc[2 * NL];
        x_line<NL>(v0, hx[comp], i, w);
        H = a.nu * ((w[3] - 2.0 * v0 + w[1]) * ih2) -
            (Ux[1] * quick(Ux[1], w[1], v0, w[3], w[4]) - Ux[0] * quick(Ux[0], w[0], w[1], v0, w[3])) * ih;
        H += a.nu * ((y3 - 2.0 * v0 + y1) * ih2) -
             (Uy[1] * quick(Uy[1], y1, v0, y3, y4) - Uy[0] * quick(Uy[0], y0, y1, v0, y3)) * ih;
        const double* z = wv[comp];
        const double up = Uz[1] * quick(Uz[1], z[1], v0, z[3], z[4]);
        H += a.nu * ((z[3] - 2.0 * v0 + z[1]) * ih2) - (up - fz[comp]) * ih;
        fz[comp] = up;
        if (MODE == MOM_EXPLICIT) {
          po[comp] = v0 + a.dt * (a.c1 * H + a.c2 * double(in.q[comp]));
        } else if (MODE == MOM_CN_START) {
          pr[comp] = v0 + 0.5 * a.dt * H;
          if (live) acc += pr[comp] * pr[comp];
          po[comp] = v0 + a.dt * H;  // Euler predictor as the first iterate
        } else {
          const double r = double(in.q[comp]) + 0.5 * a.dt * H - v0;
          if (live) acc += r * r;
          po[comp] = v0 + r * inv_diag;
        }
        ph[comp] = H;
      }
      pa = wv[0][2];
#pragma unroll
      for (int comp = 0; comp < 3; ++comp) {
#pragma unroll
        for (int q = 0; q < 4; ++q) wv[comp][q] = wv[comp][q + 1];
        wv[comp][4] = double(nv[comp]);
      }
      if (ITER) {
        za[0] = za[1];
        za[1] = za[2];
        za[2] = double(naz);
      }
      if (zwall_hi && k + 3 >= NL) {
#pragma unroll
        for (int comp = 0; comp < 3; ++comp) wv[comp][4] = mom_ghost(wv[comp][4], kd[5], 5, comp, a.U_in);
        if (ITER && k + 2 >= NL) za[2] = mom_ghost(za[2], kd[5], 5, 2, a.U_in);
      }
      if (!ITER) {
#pragma unroll
        for (int q = 0; q < 3; ++q) za[q] = wv[2][q + 1];
      }
    };
#pragma unroll 1
    for (int k = 0; k < NL; k += 2) {
      In alt;
      step(cur, alt, k, 0);
      step(alt, cur, k + 1, 1);
    }
    put(NL - 1);
  }
  if (a.part) {
    const double tsum = block_sum(acc, red);
    if (threadIdx.x == 0) a.part[blockIdx.x] = tsum;
  }
}

}  // namespace

#define BCM_MOM_NL(NLV, CALL)                         \
  switch (NLV) {                                      \
    case 16: { constexpr int NLC = 16; CALL; } break; \
    case 8: { constexpr int NLC = 8; CALL; } break;   \
    case 4: { constexpr int NLC = 4; CALL; } break;   \
    default: return hipErrorInvalidValue;             \
  }

template <typename TF, typename OFF, bool NT>
static hipError_t launch_mom_as(int NL, int mode, const MomArgs<TF>& a, int grid, hipStream_t s) {
  switch (mode) {
    case MOM_EXPLICIT:
      BCM_MOM_NL(NL, hipLaunchKernelGGL((k_mom<TF, NLC, MOM_EXPLICIT, OFF, NT>), dim3(grid), dim3(256), 0, s, a));
      break;
    case MOM_CN_START:
      BCM_MOM_NL(NL, hipLaunchKernelGGL((k_mom<TF, NLC, MOM_CN_START, OFF, NT>), dim3(grid), dim3(256), 0, s, a));
      break;
    case MOM_CN_ITER:
      BCM_MOM_NL(NL, hipLaunchKernelGGL((k_mom<TF, NLC, MOM_CN_ITER, OFF, NT>), dim3(grid), dim3(256), 0, s, a));
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <typename TF>
hipError_t launch_mom(int NL, int mode, const MomArgs<TF>& a, int grid, hipStream_t s) {
  const size_t field = size_t(a.n_cubes) * NL * NL * NL * sizeof(TF);
  // 32-bit byte offsets of cells and of face-buffer entries (at most one per cell)
  const bool small = field <= 0xFFFFFFFFull;
  // streamed once a sweep's twelve words per cell exceed the 256 MB last-level cache (33.5M
  // cells in FP64: 13.9 -> 13.6 ms a Crank-Nicolson step; 2M cells in FP32, which fit: 45 us
  // an AB2 step against 50 streamed)
  if (!small) return launch_mom_as<TF, size_t, true>(NL, mode, a, grid, s);
  if (12 * field > (size_t(256) << 20)) return launch_mom_as<TF, uint32_t, true>(NL, mode, a, grid, s);
  return launch_mom_as<TF, uint32_t, false>(NL, mode, a, grid, s);
}

template hipError_t launch_mom<float>(int, int, const MomArgs<float>&, int, hipStream_t);
template hipError_t launch_mom<double>(int, int, const MomArgs<double>&, int, hipStream_t);

}  // namespace bcm
