// les_adjoint.hip -- reverse mode (adjoint) of the residual and of one
// Runge-Kutta step, written as gather kernels.
//
// For a residual weight Rbar on the interior, Qbar = (dR/dQ)^T Rbar is the
// reverse of the residual's composition (Eq. 12-15 with the Turkel-Vatsa
// dissipation): node primitives -> node gradients -> stress / heat flux /
// eddy viscosity -> node fluxes and spectral radii / sensors -> face fluxes
// -> residual.  Every backward step that would scatter is written as a
// gather, so no atomics are needed, and every gather stays on the chip: two
// tiled passes march in k as the stage kernel does (les_stage.hip), with
// W = J Rbar (zero off the interior):
//   flux pass (k_adj_flux): the node flux adjoint is Hbar_d(n) = (W(n-e_d) -
//      W(n+e_d))/2; reverses node flux, viscous stress, heat flux,
//      Smagorinsky and Sutherland viscosity and the node gradients, and maps
//      the primitive adjoint to conserved variables;
//   dissipation pass (k_adj_diss): reverses the faces, radii and sensors and
//      adds the flux pass's part.  Output nodes are the interior nodes and
//      the ghost nodes that are images of interior nodes;
//   faces (k_adj_face): pulls the adjoint of a boundary face's ghosts back to
//      the face's boundary node through the face rule's Jacobian;
//   fold (k_adj_fold, interior nodes with ghost images): adds the adjoint of
//      every periodic or face ghost to its interior node (frozen Dirichlet
//      ghosts carry no dependence).
// Non-smooth points take the derivative of the active branch: d|x|/dx =
// sign(x) with 0 at 0, max(a, b) follows a when a >= b, and the eddy
// viscosity's |S| has derivative 0 at |S| = 0.
//
// les_adjoint_step applies it stage by stage in reverse from the stage
// inputs saved by les_rk_step: for l = 5..1, fbar += alpha_l dt qbar on the
// source plane and qbar' = (dR/dQ|Q^(l-1))^T (-alpha_l dt qbar); finally Qbar
// is the sum of all qbar (k_adj_sum).  The fbar update runs inside the
// dissipation pass and the fold of the stage whose result it takes.
#include "les_adjoint.hpp"
#include "les_tile.hpp"

namespace les {

namespace {

// Work-array field indices (library layout, one field each).
enum {
  W_FL = 0,   // flux part at the output nodes: 5 fields
  W_GG = 5,   // adjoint at the ghost images of interior nodes: 5
  W_Z = 10,   // Runge-Kutta reverse: the stages' results, 5 x 5 fields
  W_NF = 35
};

// Anisotropic scaling Lam_d and its partial derivatives w.r.t. (lam_d, lam_e,
// lam_f) for an exponent other than 1/2 (which k_adj_diss<true> takes by roots).
__device__ __forceinline__ double aniso_d(double ld, double le, double lf, const Phys& P, double& dd, double& de,
                                          double& df) {
  const double a = P.alpha;
  const double re = pow(le / ld, a), rf = pow(lf / ld, a);
  dd = 1.0 + (1.0 - a) * (re + rf);
  de = a * re * ld / le;
  df = a * rf * ld / lf;
  return ld * (1.0 + re + rf);
}

__device__ __forceinline__ double sgn(double x) { return x > 0.0 ? 1.0 : (x < 0.0 ? -1.0 : 0.0); }

struct AdjK {
  Layout L;
  Phys P;
  const double* M;
  int bc0, bc1, bc2;
  int per[3];          // period of each axis: n (periodic), n - 1 (superposed), 0 (Dirichlet)
  int lo[3], hi[3];    // output box: ghost layers of periodic axes and of active faces included
  Faces F;             // boundary faces
  int nband[3], band[3][4];  // coordinates of the interior nodes that have images along each axis, ascending
  int axis;            // j = 0 is the polar axis (bc1 == 3)
  Machine mach;
};

AdjK make_adjk(const AdjArgs& a) {
  AdjK A;
  A.L = a.L;
  A.P = a.P;
  A.M = a.M;
  A.bc0 = a.bc0;
  A.bc1 = a.bc1;
  A.bc2 = a.bc2;
  A.F = a.F;
  A.axis = a.axis;
  A.mach = a.mach;
  const int bc[3] = {a.bc0, a.bc1, a.bc2}, nn[3] = {a.L.ni, a.L.nj, a.L.nk};
  for (int d = 0; d < 3; ++d) {
    // bc 3 (polar axis, j only): its lo side is the axis, whose cross-axis
    // ghosts are images of interior nodes; its hi side is Dirichlet
    const bool per_like_lo = bc[d] == 0 || bc[d] == 2 || bc[d] == 3;
    const bool per_like_hi = bc[d] == 0 || bc[d] == 2;
    A.per[d] = bc[d] == 0 ? nn[d] : (bc[d] == 2 ? nn[d] - 1 : 0);
    const bool flo = bc[d] == 1 && a.F.type[2 * d] != 0;
    const bool fhi = (bc[d] == 1 || bc[d] == 3) && a.F.type[2 * d + 1] != 0;
    A.lo[d] = (per_like_lo || flo) ? -2 : 0;
    A.hi[d] = (per_like_hi || fhi) ? nn[d] + 1 : nn[d] - 1;
    const int p = A.per[d], n = nn[d];
    A.nband[d] = 0;
    for (int x = 0; x < n; ++x) {
      if (x == 4 && n > 8) x = n - 4;  // (images lie within two nodes of a side)
      const bool in = p ? (x + p >= n && x + p <= n + 1) || (x - p >= -2 && x - p <= -1)
                        : (x == 0 && flo) || (x == n - 1 && fhi) || (bc[d] == 3 && (x == 1 || x == 2));
      if (in) A.band[d][A.nband[d]++] = x;
    }
  }
  return A;
}

// ---------------------------------------------------------------------------
// Flux pass: the adjoint of the node fluxes (inviscid, viscous, SGS), complete
// at every output node.
//
// Blocks of 32 x 16 threads march a 30 x 14 tile of output nodes in k as the
// stage kernel does (les_stage.hip): the patch is the tile and a one-node
// ring, whose gradient weights the tile's outer nodes collect.  Per plane
//   B  stores u, v, w, T and W = coef J Rbar of the patch (and of the second
//      ring along the axes) to LDS;
//   C  recomputes the node's gradients, stress and viscosities, reverses its
//      node flux, stress, heat flux and viscosities with the node flux
//      adjoints Hbar_d = (W(n-e_d) - W(n+e_d))/2, and forms the
//      gradient-stencil weights a_{q,d} = J m_d . gbar_q; the xi differences
//      of the weights come from the adjacent lanes, the zeta differences from
//      the planes t -+ 1 through registers;
//   E  takes the eta differences through LDS, finishes plane t-1 (its upper
//      zeta neighbour is known now), maps it to conserved variables and
//      stores it (W_FL: interior nodes, and the ghost nodes that are images
//      of interior nodes).
// One read of Q, the metrics and Rbar and one write of five fields: the
// weights, the primitive adjoint and the direct terms (22 fields of the
// one-thread-per-node pass this replaces, written, and read by the gather at
// the neighbours) stay on the chip.  Bound by the FP64
// issue rate at two waves a SIMD (255 registers); 49 us on the 128 x 64 x 64
// jet, the node pass without the gather took 70.
// ---------------------------------------------------------------------------
constexpr int BX = 32, BY = 16, NT = BX * BY;  // patch (threads)
constexpr int TX = BX - 2, TY = BY - 2;        // output tile of the flux pass
constexpr int EX = BX + 2, EY = BY + 2;        // patch and second ring (LDS planes)
constexpr int NH2 = 2 * TY + 2 * TX;           // second-ring nodes
constexpr int NW = NT / 64;

struct TileArgs {
  AdjK A;
  const double* Q;
  const double* qb;
  double coef;
  double Rg, inv_gm1;  // gas constant, 1 / (gamma - 1)
  double* Wk;
  int ntx, nty;
  Schedule sch;
  int per_xcd, nxcd;
};

__device__ __forceinline__ int clampi(int x, int lo, int hi) { return x < lo ? lo : (x > hi ? hi : x); }

__global__ void __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(2, 2))) k_adj_flux(TileArgs a) {
  __shared__ double su[EY][EX], sv[EY][EX], sw[EY][EX], st[EY][EX];
  __shared__ double sW[5][EY][EX];
  __shared__ double sa[4][BY][TX];  // eta weights, patch columns 1..TX
  __shared__ double mbw[NW][10][2][BX];
  const Layout& L = a.A.L;
  typedef __attribute__((address_space(4))) const TileArgs CArgs;
  CArgs* const ka = (CArgs*)__builtin_amdgcn_kernarg_segment_ptr();
  const long long fe = L.fe;
  const int hb = blockIdx.x;
  const int v = (hb % a.nxcd) * a.per_xcd + hb / a.nxcd;
  if (v >= a.sch.nblocks) return;
  const int tid = threadIdx.x;
  const int tx = tid % BX, ty = tid / BX, ex = tx + 1, ey = ty + 1;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const bool xh = (tx == 0 || tx == BX - 1), yh = (ty == 0 || ty == BY - 1);
  const unsigned sk = (unsigned)L.sk;
  const double coef = a.coef;
  int hx2 = 0, hy2 = 0;  // second-ring slot of helper thread tid < NH2
  if (tid < NH2) {
    const int h = tid;
    if (h < TY) { hx2 = 0; hy2 = 2 + h; }
    else if (h < 2 * TY) { hx2 = EX - 1; hy2 = 2 + h - TY; }
    else if (h < 2 * TY + TX) { hy2 = 0; hx2 = 2 + h - 2 * TY; }
    else { hy2 = EY - 1; hx2 = 2 + h - 2 * TY - TX; }
  }
  for (int wq = v; wq < a.sch.nseg; wq += a.sch.nblocks) {
    const Segment seg = segment_at(a.sch, a.ntx * a.nty, a.A.hi[2] - a.A.lo[2] + 1, wq);
    const int tile = seg.tile;
    const int kb = a.A.lo[2] + seg.k0, ke = a.A.lo[2] + seg.k1;  // output planes
    const int i = a.A.lo[0] - 1 + (tile % a.ntx) * TX + tx, j = a.A.lo[1] - 1 + (tile / a.ntx) * TY + ty;
    const bool in_ij = i >= 0 && i < L.ni && j >= (a.A.axis ? 1 : 0) && j < L.nj;  // W may be nonzero
    // nodes with weights: [-1, n]^3 (not on or below the polar axis, where
    // the node flux is constant or serves only the axis)
    const bool b1_ij = i >= -1 && i <= L.ni && j >= (a.A.axis ? 1 : -1) && j <= L.nj;
    const bool out_ok = !xh && !yh && i <= a.A.hi[0] && j <= a.A.hi[1];
    const int hi = i - tx + hx2 - 1, hj = j - ty + hy2 - 1;
    const bool h_use = tid < NH2;
    const bool h_in = hi >= 0 && hi < L.ni && hj >= (a.A.axis ? 1 : 0) && hj < L.nj;
    // per-thread offsets from plane kb - 2 (nodes clamped into the padded box)
    const int kr = kb - kStageSpan.below;
    const long long sb = (long long)kr * L.sk;
    const unsigned col = (unsigned)((long long)clampi(i, -2, L.ni + 1) + (long long)clampi(j, -2, L.nj + 1) * L.sj + L.o);
    const unsigned hcol =
        (unsigned)((long long)clampi(hi, -2, L.ni + 1) + (long long)clampi(hj, -2, L.nj + 1) * L.sj + L.o);
    auto off = [&](unsigned c, int k) { return c + (unsigned)(clampi(k, -2, L.nk + 1) - kr) * sk; };
    // row copies of the metrics (rows 2 wave, 2 wave + 1; see les_stage.hip)
    const int fsel = lane >> 5, rsel = (lane / 16) % 2, pr = lane % 16;
    int icp = i - tx + 2 * pr;
    if (icp > L.ni) icp = L.ni - ((LEAD + L.ni) & 1);
    const int jcp = clampi(j - ty + 2 * wave + rsel, -2, L.nj + 1);
    const long long lane_el = (long long)fsel * fe + L.o + icp + (long long)jcp * L.sj;
    const long long fstep2 = 2 * fe * (long long)sizeof(double);
    double* const mdst = &mbw[wave][0][0][0];

    double up1[4], rp1 = 0, um1[4], rc = 0, rm1 = 0;  // u, v, w, T and rho at t+1 (at B: t), t-1; rho at t, t-1
    double Wm[5], Wc[5];                              // W at t-1; at t (at B)
    double qn[5], bn[5], Jn;                          // Q, Rbar and J of plane t+1 (loaded one plane ahead)
    double a2[4] = {0, 0, 0, 0};                      // zeta weights of plane t-1
    double pf[10];                                    // plane t-1: rho, u, v, w, p, T adjoint, direct Q1..Q4
    auto prims = [&](const Phys& P, const double q[5], double uu[4], double& rr) {
      double p;
      rr = q[0];
      prim_from_q_fast(q[0], q[1], q[2], q[3], q[4], P, uu[0], uu[1], uu[2], p, uu[3]);
    };
    auto load5 = [&](const double* f, unsigned o, double x[5]) {
#pragma unroll
      for (int c = 0; c < 5; ++c) x[c] = ldo(f + sb + c * fe, o);
    };
    auto Wset = [&](bool in, int k, const double b[5], double J, double W[5]) {
      const bool ok = in && k >= 0 && k < L.nk;
      const double s = coef * J;
#pragma unroll
      for (int c = 0; c < 5; ++c) W[c] = ok ? s * b[c] : 0.0;
    };
    {
      CArgs* kp4 = ka;
      asm volatile("" : "+s"(kp4));
      const TileArgs* kp = (const TileArgs*)kp4;
      const char* msrc = (const char*)(kp->A.M + lane_el + (long long)clampi(kb - 1, -2, L.nk + 1) * L.sk);
#pragma unroll
      for (int q = 0; q < 5; ++q) copy_to_lds(msrc + q * fstep2, mdst + q * 128);
      const unsigned o0 = off(col, kb - 2), o1 = off(col, kb - 1), o2 = off(col, kb);
      double q0[5], b0[5], q1[5], b1[5];
      load5(kp->Q, o0, q0);
      load5(kp->qb, o0, b0);
      load5(kp->Q, o1, q1);
      load5(kp->qb, o1, b1);
      const double J0 = ldo(kp->A.M + sb + 9 * fe, o0), J1 = ldo(kp->A.M + sb + 9 * fe, o1);
      load5(kp->Q, o2, qn);
      load5(kp->qb, o2, bn);
      Jn = ldo(kp->A.M + sb + 9 * fe, o2);
      prims(kp->A.P, q0, um1, rm1);
      prims(kp->A.P, q1, up1, rp1);
      Wset(in_ij, kb - 2, b0, J0, Wm);
      Wset(in_ij, kb - 1, b1, J1, Wc);
      wait_vm<0>();
    }
#pragma unroll
    for (int c = 0; c < 10; ++c) pf[c] = 0.0;

    for (int t = kb - 1; t <= ke; ++t) {
      CArgs* kq4 = ka;
      asm volatile("" : "+s"(kq4));
      const TileArgs* kq = (const TileArgs*)kq4;
      const Phys& P = kq->A.P;
      // ---- B ----
      su[ey][ex] = up1[0]; sv[ey][ex] = up1[1]; sw[ey][ex] = up1[2]; st[ey][ex] = up1[3];
#pragma unroll
      for (int c = 0; c < 5; ++c) sW[c][ey][ex] = Wc[c];
      rc = rp1;
      if (h_use) {
        double hq[5], hv[5], hu[4], hr, hW[5];
        const unsigned ho = off(hcol, t);
        load5(kq->Q, ho, hq);
        load5(kq->qb, ho, hv);
        const double hJ = ldo(kq->A.M + sb + 9 * fe, ho);
        prims(P, hq, hu, hr);
        Wset(h_in, t, hv, hJ, hW);
        su[hy2][hx2] = hu[0]; sv[hy2][hx2] = hu[1]; sw[hy2][hx2] = hu[2]; st[hy2][hx2] = hu[3];
#pragma unroll
        for (int c = 0; c < 5; ++c) sW[c][hy2][hx2] = hW[c];
      }
      lds_barrier();

      // ---- C ----
      prims(P, qn, up1, rp1);  // plane t+1
      double Wp[5];
      Wset(in_ij, t + 1, bn, Jn, Wp);
      double m[9], J;
      read_metric_rows(&mbw[wave][0][ty & 1][tx], m, J);
      const char* const msrc = (const char*)(kq->A.M + lane_el + (long long)clampi(t + 1, -2, L.nk + 1) * L.sk);
      const unsigned on = off(col, t + 2);
      auto load_ahead = [&](int q) {
        if (t < ke) {
          copy_to_lds(msrc + q * fstep2, mdst + q * 128);
          qn[q] = ldo(kq->Q + sb + q * fe, on);
          bn[q] = ldo(kq->qb + sb + q * fe, on);
          if (q == 4) Jn = ldo(kq->A.M + sb + 9 * fe, on);
        }
        __builtin_amdgcn_sched_barrier(0);
      };
      double g[4][3];
      {
        const double(*F[4])[EX] = {su, sv, sw, st};
        const double Jh = 0.5 * J;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const double dx = F[q][ey][ex + 1] - F[q][ey][ex - 1];
          const double dy = F[q][ey + 1][ex] - F[q][ey - 1][ex];
          const double dz = up1[q] - um1[q];
#pragma unroll
          for (int x = 0; x < 3; ++x) g[q][x] = Jh * (m[x] * dx + m[3 + x] * dy + m[6 + x] * dz);
        }
      }
      load_ahead(0);
      const double uu[3] = {su[ey][ex], sv[ey][ex], sw[ey][ex]}, T = st[ey][ex], rho = rc;
      const double S11 = g[0][0], S22 = g[1][1], S33 = g[2][2];
      const double S12 = 0.5 * (g[0][1] + g[1][0]), S13 = 0.5 * (g[0][2] + g[2][0]), S23 = 0.5 * (g[1][2] + g[2][1]);
      const double skk3 = (S11 + S22 + S33) * (1.0 / 3.0);
      const double th = T * P.inv_Tref;
      const double ithS = rcp_nr(th + P.S);
      const double mu = P.mu_ref * P.one_plus_S * th * sqrt_pos(th) * ithS;
      double mus = 0.0, Smag = 0.0, cd2 = 0.0, ss = 0.0, cid2 = 0.0;
      if (P.sgs) {
        ss = S11 * S11 + S22 * S22 + S33 * S33 + 2.0 * (S12 * S12 + S13 * S13 + S23 * S23);
        Smag = sqrt_nn(2.0 * ss);
        const double d2 = icbrt(J);  // (1/J)^(1/3)
        cd2 = P.Cs2 * d2 * d2;
        mus = rho * cd2 * Smag;
        // isotropic SGS stress: sigma_kk / 3 = CI43 rho D^2 S:S, added to the
        // pressure of the momentum and energy fluxes
        cid2 = P.CI43 * d2 * d2;
      }
      const double mt2 = 2.0 * (mu + mus);
      const double t11 = mt2 * (S11 - skk3), t22 = mt2 * (S22 - skk3), t33 = mt2 * (S33 - skk3);
      const double t12 = mt2 * S12, t13 = mt2 * S13, t23 = mt2 * S23;
      const double kap = mu * P.Cp_over_Pr + mus * P.Cp_over_Prsgs;
      load_ahead(1);
      // ---- reverse of the node fluxes ----
      double rb = 0, ub[3] = {0, 0, 0}, pb = 0, qd[4] = {0, 0, 0, 0};
      double tb11 = 0, tb22 = 0, tb33 = 0, tb12 = 0, tb13 = 0, tb23 = 0, thb[3] = {0, 0, 0};
      {
        const double p = rho * T * kq->Rg;
        const double eh = p * kq->inv_gm1 + 0.5 * rho * (uu[0] * uu[0] + uu[1] * uu[1] + uu[2] * uu[2]) + p +
                          rho * cid2 * ss;  // e + p + sigma_kk / 3
#pragma unroll
        for (int d = 0; d < 3; ++d) {
          double Hb[5];
#pragma unroll
          for (int c = 0; c < 5; ++c)
            Hb[c] = 0.5 * (d == 0   ? sW[c][ey][ex - 1] - sW[c][ey][ex + 1]
                           : d == 1 ? sW[c][ey - 1][ex] - sW[c][ey + 1][ex]
                                    : Wm[c] - Wp[c]);
          const double mx = m[3 * d], my = m[3 * d + 1], mz = m[3 * d + 2];
          const double U = mx * uu[0] + my * uu[1] + mz * uu[2];
          // H_0 = rho U, H_{1+a} = Q_{1+a} U + m_a p - m . tau_a, H_4 = (e + p) U - m . Theta
          const double Ub = rho * (Hb[0] + Hb[1] * uu[0] + Hb[2] * uu[1] + Hb[3] * uu[2]) + Hb[4] * eh;
          rb += Hb[0] * U;
          qd[0] += Hb[1] * U;
          qd[1] += Hb[2] * U;
          qd[2] += Hb[3] * U;
          qd[3] += Hb[4] * U;
          pb += Hb[1] * mx + Hb[2] * my + Hb[3] * mz + Hb[4] * U;
          tb11 -= Hb[1] * mx;
          tb22 -= Hb[2] * my;
          tb33 -= Hb[3] * mz;
          tb12 -= Hb[1] * my + Hb[2] * mx;
          tb13 -= Hb[1] * mz + Hb[3] * mx;
          tb23 -= Hb[2] * mz + Hb[3] * my;
          thb[0] -= Hb[4] * mx;
          thb[1] -= Hb[4] * my;
          thb[2] -= Hb[4] * mz;
          ub[0] += Ub * mx;
          ub[1] += Ub * my;
          ub[2] += Ub * mz;
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      load_ahead(2);
      // Theta_x = u_a tau_ax + kappa dT/dx
      ub[0] += thb[0] * t11 + thb[1] * t12 + thb[2] * t13;
      ub[1] += thb[0] * t12 + thb[1] * t22 + thb[2] * t23;
      ub[2] += thb[0] * t13 + thb[1] * t23 + thb[2] * t33;
      tb11 += uu[0] * thb[0];
      tb22 += uu[1] * thb[1];
      tb33 += uu[2] * thb[2];
      tb12 += uu[0] * thb[1] + uu[1] * thb[0];
      tb13 += uu[0] * thb[2] + uu[2] * thb[0];
      tb23 += uu[1] * thb[2] + uu[2] * thb[1];
      const double kapb = thb[0] * g[3][0] + thb[1] * g[3][1] + thb[2] * g[3][2];
      // tau = 2 (mu + mu_sgs) (S - delta S_kk / 3); the off-diagonal adjoints
      // are those of the pair (12, 21), ...
      const double mtb = 2.0 * ((S11 - skk3) * tb11 + (S22 - skk3) * tb22 + (S33 - skk3) * tb33 + S12 * tb12 +
                                S13 * tb13 + S23 * tb23);
      const double trb = (tb11 + tb22 + tb33) * (1.0 / 3.0);
      double Sb11 = mt2 * (tb11 - trb), Sb22 = mt2 * (tb22 - trb), Sb33 = mt2 * (tb33 - trb);
      double Sb12 = mt2 * tb12, Sb13 = mt2 * tb13, Sb23 = mt2 * tb23;
      const double mub = mtb + kapb * P.Cp_over_Pr;
      if (P.sgs) {
        const double musb = mtb + kapb * P.Cp_over_Prsgs;
        rb += musb * cd2 * Smag + pb * cid2 * ss;
        // (|S| > 0 fails for a NaN too: a node whose flux no residual uses may
        // have a strain of ghosts that nothing reads, and its weights stay 0)
        if (Smag > 0.0) {
          const double sb2 = 2.0 * pb * rho * cid2 + 2.0 * musb * rho * cd2 * rcp_nr(Smag);
          Sb11 += S11 * sb2;
          Sb22 += S22 * sb2;
          Sb33 += S33 * sb2;
          Sb12 += 2.0 * S12 * sb2;
          Sb13 += 2.0 * S13 * sb2;
          Sb23 += 2.0 * S23 * sb2;
        }
      }
      // Sutherland: dmu/dT = mu (3/(2 th) - 1/(th + S)) / T_ref
      double Tb = mub * mu * (1.5 * rcp_nr(th) - ithS) * P.inv_Tref;
      load_ahead(3);
      // gradient-stencil weights (half of them: the halves of the central
      // differences): a_{q,d} = J/2 m_d . gbar_q, gbar_3 = kappa Theta-bar
      double aw[4][3];
      {
        const double Jh = 0.5 * J, kh = kap;
        const double G[4][3] = {{Sb11, 0.5 * Sb12, 0.5 * Sb13},
                                {0.5 * Sb12, Sb22, 0.5 * Sb23},
                                {0.5 * Sb13, 0.5 * Sb23, Sb33},
                                {kh * thb[0], kh * thb[1], kh * thb[2]}};
        const bool act = b1_ij && t >= -1 && t <= L.nk;
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int d = 0; d < 3; ++d) {
            const double x = Jh * (m[3 * d] * G[q][0] + m[3 * d + 1] * G[q][1] + m[3 * d + 2] * G[q][2]);
            aw[q][d] = act ? x : 0.0;
          }
        if (!act) {
          rb = pb = Tb = 0.0;
#pragma unroll
          for (int c = 0; c < 3; ++c) ub[c] = 0.0;
#pragma unroll
          for (int c = 0; c < 4; ++c) qd[c] = 0.0;
        }
      }
      load_ahead(4);
      if (!xh) {
#pragma unroll
        for (int q = 0; q < 4; ++q) sa[q][ty][tx - 1] = aw[q][1];
      }
      // zeta: the weights of plane t complete plane t-1, those of t-1 open plane t
      double dphi[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        pf[q < 3 ? 1 + q : 5] -= aw[q][2];
        dphi[q] = a2[q] + (lane_prev(aw[q][0]) - lane_next(aw[q][0]));
        a2[q] = aw[q][2];
      }
      __builtin_amdgcn_sched_barrier(0);
      // finish plane t-1: map to conserved variables
      double o[5];
      {
        const double ir = rcp_nr(rm1);
        const bool any = pf[0] != 0.0 || pf[1] != 0.0 || pf[2] != 0.0 || pf[3] != 0.0 || pf[4] != 0.0 || pf[5] != 0.0;
        const double pt = pf[4] + pf[5] * P.inv_R * ir, gp = P.gm1 * pt;
        const double ut = um1[0] * um1[0] + um1[1] * um1[1] + um1[2] * um1[2];
        o[0] = pf[0] - pf[5] * um1[3] * ir + 0.5 * gp * ut - (pf[1] * um1[0] + pf[2] * um1[1] + pf[3] * um1[2]) * ir;
        o[1] = pf[6] + pf[1] * ir - gp * um1[0];
        o[2] = pf[7] + pf[2] * ir - gp * um1[1];
        o[3] = pf[8] + pf[3] * ir - gp * um1[2];
        o[4] = pf[9] + gp;
        // (nodes without any adjoint skip the map: unused ghost corners may hold anything)
        o[0] = any ? o[0] : 0.0;
#pragma unroll
        for (int c = 1; c < 5; ++c) o[c] = any ? o[c] : pf[5 + c];
      }
      lds_barrier();

      // ---- E ----
      if (out_ok) {
#pragma unroll
        for (int q = 0; q < 4; ++q) dphi[q] += sa[q][ty - 1][tx - 1] - sa[q][ty + 1][tx - 1];
      }
      pf[0] = rb;
      pf[1] = ub[0] + dphi[0];
      pf[2] = ub[1] + dphi[1];
      pf[3] = ub[2] + dphi[2];
      pf[4] = pb;
      pf[5] = Tb + dphi[3];
#pragma unroll
      for (int c = 0; c < 4; ++c) pf[6 + c] = qd[c];
      um1[0] = su[ey][ex]; um1[1] = sv[ey][ex]; um1[2] = sw[ey][ex]; um1[3] = st[ey][ex];
      rm1 = rc;
#pragma unroll
      for (int c = 0; c < 5; ++c) {
        Wm[c] = sW[c][ey][ex];
        Wc[c] = Wp[c];
      }
      __builtin_amdgcn_sched_barrier(0);
      wait_vm<0>();  // the loads of this plane, before the stores (see les_stage.hip)
      if (out_ok && t > kb) {
        const unsigned on1 = col + (unsigned)(t - 1 - kr) * sk;
#pragma unroll
        for (int c = 0; c < 5; ++c) sto(kq->Wk + (W_FL + c) * fe + sb, on1, o[c]);
      }
      // (the next B overwrites LDS that this plane's C read: every wave is past
      // the barrier above; E reads only the eta weights, next written after
      // the next plane's first barrier, and the thread's own node)
    }
  }
}

// Does interior node (i, j, k) have ghost images: a periodic image along an
// axis of period p (x + p in [n, n + 1] or x - p in [-2, -1]), or face ghosts
// (x at an active boundary face of a Dirichlet axis)?
__device__ __forceinline__ bool has_images(const AdjK& A, int i, int j, int k) {
  const int id[3] = {i, j, k}, nn[3] = {A.L.ni, A.L.nj, A.L.nk}, bc[3] = {A.bc0, A.bc1, A.bc2};
  // rings j = 1, 2 are the images of the ghosts across the polar axis
  if (A.axis && (j == 1 || j == 2)) return true;
  for (int d = 0; d < 3; ++d) {
    const int p = A.per[d];
    if (p) {
      if ((id[d] + p >= nn[d] && id[d] + p <= nn[d] + 1) || (id[d] - p <= -1 && id[d] - p >= -2)) return true;
    } else if (bc[d] == 1 || bc[d] == 3) {
      if ((id[d] == 0 && bc[d] == 1 && A.F.type[2 * d] != 0) || (id[d] == nn[d] - 1 && A.F.type[2 * d + 1] != 0))
        return true;
    }
  }
  return false;
}

// ---------------------------------------------------------------------------
// Dissipation pass: the adjoint of the Turkel-Vatsa faces, complete at every
// output node, added to the flux pass's part.
//
// For the face (a, b = a + e_d) used by an interior residual,
// D = Lf (eps2 dQ - eps4 d3Q) is reversed with Dbar = W(b) - W(a):
//   - directly to the four states of its stencil: +-F and +-G with
//     F = Lf (eps2 + 3 eps4) Dbar, G = Lf eps4 Dbar;
//   - through the face mean Lf: half of sum_c Dbar_c (eps2 dQ - eps4 d3Q)_c to
//     Lambda_d of either end, and by V_d = dLambda_d / dQ to the end's state;
//   - through eps2 and eps4 to the sensor of the end that wins the maximum (a
//     on ties; max(0, k4 - eps2) follows 0 on ties), and from
//     nu = |p+ - 2p + p-| / Sigma to p at the end and its two neighbours.
// An output node therefore depends on the faces n-2e .. n+e of each line and
// on states up to three nodes away: blocks of 32 x 16 threads own a patch
// whose inner 28 x 12 nodes are the tile, march in k like the stage kernel and
// evaluate every face of the patch once.  Per plane t
//   B  stores Q, p and W of the patch (Q, p also of one ring along the axes);
//   C  forms the radii, sensors and V_d of the plane's nodes and the whole xi
//      direction (a patch row is 32 lanes: neighbours by lane shifts), then the
//      zeta face (t-1, t) from registers;
//   D  evaluates the eta faces (one per node and row) into LDS;
//   E  gathers the eta faces, and stores plane t-2, which the zeta face
//      completed.
// One read of Q, the metrics, Rbar and the flux part and one write, instead of
// two passes that wrote and re-read 45 fields through the caches.  The xi
// faces and V_d stay in registers; V_1 and the eta faces go through LDS, and
// the loads of the next plane are issued after the zeta face, because the 512
// threads' 256 registers do not hold them beside it (with all of it in
// registers: 183 spills and 300 us on the 128 x 64 x 64 jet).  Bound by the
// FP64 issue rate, a patch having 1.5 times its tile's nodes: 92 us on that
// jet and 131 us on the 128 x 64 x 121 O-grid, where the passes replaced took
// 199 and 404 us (with the flux pass: 269 to 141 and 536 to 212 us).
// ---------------------------------------------------------------------------
constexpr int DTX = BX - 4, DTY = BY - 4;  // output tile of the dissipation pass
constexpr int DNH = 2 * DTX + 2 * DTY;     // ring nodes
// (the march starts two planes before the segment, with Q of the plane before
// that, and ends two planes after it, loading Q two planes ahead)
constexpr Span kDissSpan{3, 4};

struct DissArgs {
  TileArgs t;
  double* qout;
  double* fbar;
  double fw;
  int i_f;
};

// eps2, eps4 and the reversed sensor part of one face; e2b is the adjoint of
// eps2 (with eps4's share where it is active)
__device__ __forceinline__ void face_rev(const Phys& P, double La, double Lb, double nsa, double nsb,
                                         const double qam[5], const double qa[5], const double qb[5],
                                         const double qbp[5], const double Db[5], bool ok, double F[5], double G[5],
                                         double& LH, double& NA, double& NB) {
  const double na = fabs(nsa), nb = fabs(nsb);
  const bool aw = na >= nb;
  const double e2 = P.k2 * (aw ? na : nb);
  const double e4r = P.k4 - e2;
  const bool act = !(0.0 >= e4r);
  const double e4 = act ? e4r : 0.0;
  const double Lf = 0.5 * (La + Lb);
  double s1 = 0.0, s3 = 0.0;
  const double wf = Lf * (e2 + 3.0 * e4), wg = Lf * e4;
#pragma unroll
  for (int c = 0; c < 5; ++c) {
    const double d1 = qb[c] - qa[c];
    const double d3 = qbp[c] - 3.0 * qb[c] + 3.0 * qa[c] - qam[c];
    s1 += Db[c] * d1;
    s3 += Db[c] * d3;
    F[c] = ok ? wf * Db[c] : 0.0;
    G[c] = ok ? wg * Db[c] : 0.0;
  }
  const double e2b = P.k2 * Lf * (act ? s1 + s3 : s1);
  LH = ok ? 0.5 * (e2 * s1 - e4 * s3) : 0.0;
  NA = ok && aw ? e2b : 0.0;
  NB = ok && !aw ? e2b : 0.0;
}

// HALF: the anisotropy exponent is 1/2 (no pow in that instantiation)
template <bool HALF>
__global__ void __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(2, 2))) k_adj_diss(DissArgs a) {
  __shared__ double sq[5][EY][EX], sp[EY][EX];
  __shared__ double sW[5][BY][BX];
  __shared__ double ly[BY][DTX], ny[BY][DTX], cy[BY][DTX];  // eta radius, signed sensor, 1 / Sigma; columns 2..DTX+1
  __shared__ double fF[5][BY - 1][DTX], fG[5][BY - 1][DTX], fL[BY - 1][DTX], fA[BY - 1][DTX], fB[BY - 1][DTX];
  __shared__ double sV[5][BY][DTX];  // V_1 of the plane
  __shared__ unsigned sh[DNH];       // columns of the ring nodes
  __shared__ double mbw[NW][10][2][BX];
  const TileArgs& ta = a.t;
  const Layout& L = ta.A.L;
  typedef __attribute__((address_space(4))) const DissArgs CArgs;
  CArgs* const ka = (CArgs*)__builtin_amdgcn_kernarg_segment_ptr();
  const long long fe = L.fe;
  const int hb = blockIdx.x;
  const int v = (hb % ta.nxcd) * ta.per_xcd + hb / ta.nxcd;
  if (v >= ta.sch.nblocks) return;
  const int tid = threadIdx.x;
  const int tx = tid % BX, ty = tid / BX, ex = tx + 1, ey = ty + 1, cx = tx - 2;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const bool cx_ok = tx >= 2 && tx < BX - 2, ry_ok = ty >= 2 && ty < BY - 2;
  const unsigned sk = (unsigned)L.sk;
  const double coef = ta.coef;
  const int axis = ta.A.axis;
  // ring slot of helper thread h < DNH; formed again in each plane, and its
  // column kept in LDS: as spilled registers, their reloads would wait for the
  // stores before them (the counter of outstanding operations is in order)
  auto ring = [&](int h, int& hx2, int& hy2) {
    if (h < 2 * DTY) {
      hx2 = h < DTY ? 0 : EX - 1;
      hy2 = 3 + (h < DTY ? h : h - DTY);
    } else {
      const int g = h - 2 * DTY;
      hy2 = g < DTX ? 0 : EY - 1;
      hx2 = 3 + (g < DTX ? g : g - DTX);
    }
  };
  for (int wq = v; wq < ta.sch.nseg; wq += ta.sch.nblocks) {
    const Segment seg = segment_at(ta.sch, ta.ntx * ta.nty, ta.A.hi[2] - ta.A.lo[2] + 1, wq);
    const int tile = seg.tile;
    const int kb = ta.A.lo[2] + seg.k0, ke = ta.A.lo[2] + seg.k1;  // output planes
    // (tiles start one node before the output box in i, so that row copies are
    // 16-byte aligned)
    const int i = ta.A.lo[0] - 3 + (tile % ta.ntx) * DTX + tx, j = ta.A.lo[1] - 2 + (tile / ta.ntx) * DTY + ty;
    const bool ii = i >= 0 && i < L.ni, jj = j >= 0 && j < L.nj;
    const bool in_ij = ii && jj && !(axis && j == 0);               // W may be nonzero
    const bool b1_ij = i >= -1 && i <= L.ni && j >= -1 && j <= L.nj;  // radii and sensors exist
    const bool fx_ij = jj && i >= -1 && i < L.ni && tx < BX - 1;     // xi face (i, i + 1)
    const bool fy_ij = ii && j >= -1 && j < L.nj && ty < BY - 1 && cx_ok;
    int hx = 0, hy = 0;
    ring(tid < DNH ? tid : 0, hx, hy);
    const int hi = i - tx + hx - 1, hj = j - ty + hy - 1;
    // Edge ghosts of the two directions when neither is periodic: frozen, in
    // no face's stencil (the residual reads only the first of them, for
    // gradients) and not read by the fold.  They may hold anything, so they
    // load a column next to the interior and are not stored.
    auto edge = [&](int x, int y) {
      return (x < 0 || x >= L.ni) && (y < 0 || y >= L.nj) && ta.A.per[0] == 0 && ta.A.per[1] == 0;
    };
    auto column = [&](int x, int y) {
      const int yc = edge(x, y) ? clampi(y, 0, L.nj - 1) : clampi(y, -2, L.nj + 1);
      return (unsigned)((long long)clampi(x, -2, L.ni + 1) + (long long)yc * L.sj + L.o);
    };
    const bool out_ok = cx_ok && ry_ok && i >= ta.A.lo[0] && i <= ta.A.hi[0] && j <= ta.A.hi[1] &&
                        !edge(i, j);
    const int kr = kb - kDissSpan.below;
    const long long sb = (long long)kr * L.sk;
    const unsigned col = column(i, j), hcol = column(hi, hj);
    auto off = [&](unsigned c, int k) { return c + (unsigned)(clampi(k, -2, L.nk + 1) - kr) * sk; };
    const int fsel = lane >> 5, rsel = (lane / 16) % 2, pr = lane % 16;
    int icp = i - tx + 2 * pr;
    if (icp > L.ni) icp = L.ni - ((LEAD + L.ni) & 1);
    const int jcp = clampi(j - ty + 2 * wave + rsel, -2, L.nj + 1);
    const long long lane_el = (long long)fsel * fe + L.o + icp + (long long)jcp * L.sj;
    const long long fstep2 = 2 * fe * (long long)sizeof(double);
    double* const mdst = &mbw[wave][0][0][0];

    double qm2[5], qm1[5], qw[5], qa[5], qn[5];  // Q at t-2, t-1, t (at B), t+1 and t+2 (in flight)
    double hq[5];                                // ring node, next plane
    double bn[5], Jn;                            // Rbar and J of the next plane (in flight)
    double Wm[5], Wc[5];                         // W at t-1, t (at B)
    double pm1, pc, pp1;                         // p at t-1, t, t+1
    double L2 = 0, ns2 = 0, iS2 = 0, nbz = 0;    // plane t-1: zeta radius, sensor, 1 / Sigma, sensor adjoint of its lower face
    double V2[5], Gz[5], om1[5], om2[5], pb1 = 0, pb2 = 0;  // V_2 at t-1; G of the last zeta face; planes t-1, t-2
    auto load5 = [&](const double* f, unsigned o, double x[5]) {
#pragma unroll
      for (int c = 0; c < 5; ++c) x[c] = ldo(f + sb + c * fe, o);
    };
    auto Wset = [&](int k, double W[5]) {
      const bool ok = in_ij && k >= 0 && k < L.nk;
      const double s = coef * Jn;
#pragma unroll
      for (int c = 0; c < 5; ++c) W[c] = ok ? s * bn[c] : 0.0;
    };
    auto pres = [&](const Phys& P, const double q[5]) {
      return P.gm1 * (q[4] - 0.5 * (q[1] * q[1] + q[2] * q[2] + q[3] * q[3]) * rcp_nr(q[0]));
    };
    {
      CArgs* kp4 = ka;
      asm volatile("" : "+s"(kp4));
      const DissArgs* kp = (const DissArgs*)kp4;
      const char* msrc = (const char*)(kp->t.A.M + lane_el + (long long)clampi(kb - 2, -2, L.nk + 1) * L.sk);
#pragma unroll
      for (int q = 0; q < 5; ++q) copy_to_lds(msrc + q * fstep2, mdst + q * 128);
      load5(kp->t.Q, off(col, kb - 3), qm1);
      load5(kp->t.Q, off(col, kb - 2), qw);
      load5(kp->t.Q, off(col, kb - 1), qa);
      if (tid < DNH) {
        sh[tid] = hcol;
        load5(kp->t.Q, off(hcol, kb - 2), hq);
      }
      load5(kp->t.qb, off(col, kb - 2), bn);
      Jn = ldo(kp->t.A.M + sb + 9 * fe, off(col, kb - 2));
      pm1 = pres(kp->t.A.P, qm1);
      pp1 = pres(kp->t.A.P, qw);
      Wset(kb - 2, Wc);
      wait_vm<0>();
    }
#pragma unroll
    for (int c = 0; c < 5; ++c) {
      qm2[c] = qm1[c];
      Wm[c] = V2[c] = Gz[c] = om1[c] = om2[c] = qn[c] = 0.0;
    }

    for (int t = kb - 2; t <= ke + 1; ++t) {
      CArgs* kq4 = ka;
      asm volatile("" : "+s"(kq4));
      const DissArgs* kq = (const DissArgs*)kq4;
      const Phys& P = kq->t.A.P;
      const bool inner = t >= kb && t < ke && t >= 0 && t < L.nk;  // in-plane faces of output nodes
      // (LDS addresses are formed again in each plane: kept over the loop they
      // would spill)
      int tl = tid;
      asm volatile("" : "+v"(tl));
      const int tx = tl % BX, ty = tl / BX, ex = tx + 1, ey = ty + 1, cx = tx - 2;
      // ---- B ----
      pc = pp1;
#pragma unroll
      for (int c = 0; c < 5; ++c) sq[c][ey][ex] = qw[c];
      sp[ey][ex] = pc;
#pragma unroll
      for (int c = 0; c < 5; ++c) sW[c][ty][tx] = Wc[c];
      if (tl < DNH) {
        int hx2, hy2;
        ring(tl, hx2, hy2);
#pragma unroll
        for (int c = 0; c < 5; ++c) sq[c][hy2][hx2] = hq[c];
        sp[hy2][hx2] = pres(P, hq);
      }
      lds_barrier();

      // ---- C ----
      pp1 = pres(P, qa);
      double m[9], J;
      read_metric_rows(&mbw[wave][0][ty & 1][tx], m, J);
      const char* const msrc = (const char*)(kq->t.A.M + lane_el + (long long)clampi(t + 1, -2, L.nk + 1) * L.sk);
      const unsigned on = off(col, t + 2), ob = off(col, t + 1);
      auto load_ahead = [&](int q) {
        if (t <= ke) {
          copy_to_lds(msrc + q * fstep2, mdst + q * 128);
        }
        __builtin_amdgcn_sched_barrier(0);
      };
      load_ahead(0);
      const bool b1 = b1_ij && t >= -1 && t <= L.nk;
      const bool rad = b1 && !(axis && j <= 0);  // (on and below the polar axis the radii are constants, 0)
      double oc[5] = {0, 0, 0, 0, 0}, pbc = 0.0;  // plane t: conserved and pressure adjoint
      double Lam0, Lam1, Lam2, V0[5], V2n[5];
      {
        // radii, Lambda_d and V_d = dLambda_d / dQ
        const double rho = sq[0][ey][ex], ir = rcp_nr(rho);
        const double u[3] = {sq[1][ey][ex] * ir, sq[2][ey][ex] * ir, sq[3][ey][ex] * ir};
        const double c2 = P.gamma * pc * ir;
        const double cs = sqrt_pos(c2);
        double lam[3], sg[3], nrm[3];
#pragma unroll
        for (int e = 0; e < 3; ++e) {
          const double mx = m[3 * e], my = m[3 * e + 1], mz = m[3 * e + 2];
          const double U = mx * u[0] + my * u[1] + mz * u[2];
          nrm[e] = sqrt_pos(mx * mx + my * my + mz * mz);
          lam[e] = fabs(U) + cs * nrm[e];
          sg[e] = sgn(U);
        }
        __builtin_amdgcn_sched_barrier(0);
        double w[3][3], Lam[3];  // w[d][e] = dLambda_d / dlam_e
        if (HALF) {
          const double s0 = sqrt_pos(lam[0]), s1 = sqrt_pos(lam[1]), s2 = sqrt_pos(lam[2]);
          const double h0 = 0.5 * rcp_nr(s0), h1 = 0.5 * rcp_nr(s1), h2 = 0.5 * rcp_nr(s2);
          Lam[0] = lam[0] + s0 * (s1 + s2);
          Lam[1] = lam[1] + s1 * (s2 + s0);
          Lam[2] = lam[2] + s2 * (s0 + s1);
          w[0][0] = 1.0 + (s1 + s2) * h0; w[0][1] = s0 * h1; w[0][2] = s0 * h2;
          w[1][1] = 1.0 + (s2 + s0) * h1; w[1][2] = s1 * h2; w[1][0] = s1 * h0;
          w[2][2] = 1.0 + (s0 + s1) * h2; w[2][0] = s2 * h0; w[2][1] = s2 * h1;
        } else {
#pragma unroll
          for (int d = 0; d < 3; ++d)
            Lam[d] = aniso_d(lam[d], lam[(d + 1) % 3], lam[(d + 2) % 3], P, w[d][d], w[d][(d + 1) % 3], w[d][(d + 2) % 3]);
        }
        Lam0 = rad ? Lam[0] : 0.0;
        Lam1 = rad ? Lam[1] : 0.0;
        Lam2 = rad ? Lam[2] : 0.0;
        const double ir2 = 0.5 * ir, kp = P.gamma * rcp_nr(cs) * ir2, ke2 = u[0] * u[0] + u[1] * u[1] + u[2] * u[2];
#pragma unroll
        for (int dd = 0; dd < 3; ++dd) {
          const int d = (dd + 1) % 3;
          double V[5];
          // lam_e = |U_e| + c |m_e|, c = sqrt(gamma p / rho)
          const double w0 = w[d][0] * sg[0], w1 = w[d][1] * sg[1], w2 = w[d][2] * sg[2];
          const double ux = w0 * m[0] + w1 * m[3] + w2 * m[6];
          const double uy = w0 * m[1] + w1 * m[4] + w2 * m[7];
          const double uz = w0 * m[2] + w1 * m[5] + w2 * m[8];
          const double cb = w[d][0] * nrm[0] + w[d][1] * nrm[1] + w[d][2] * nrm[2];
          const double gp = P.gm1 * cb * kp;
          V[0] = rad ? 0.5 * gp * ke2 - cb * cs * ir2 - (ux * u[0] + uy * u[1] + uz * u[2]) * ir : 0.0;
          V[1] = rad ? ux * ir - gp * u[0] : 0.0;
          V[2] = rad ? uy * ir - gp * u[1] : 0.0;
          V[3] = rad ? uz * ir - gp * u[2] : 0.0;
          V[4] = rad ? gp : 0.0;
#pragma unroll
          for (int c = 0; c < 5; ++c) {
            if (d == 0) V0[c] = V[c];
            if (d == 1 && cx_ok) sV[c][ty][cx] = V[c];
            if (d == 2) V2n[c] = V[c];
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      load_ahead(1);
      // ---- xi direction ----
      if (inner) {
        const double pa = sp[ey][ex + 1], pz = sp[ey][ex - 1];
        const double iS = b1 ? rcp_nr(pa + 2.0 * pc + pz) : 0.0;
        const double ns = b1 ? (pa - 2.0 * pc + pz) * iS : 0.0;
        double F[5], G[5], LH, NA, NB;
        {
          double q_b[5], q_c[5], q_d[5], q_e[5], Db[5];
          const double Ln = lane_next(Lam0), nn = lane_next(ns);
          const int xn = tx < BX - 1 ? tx + 1 : tx, e2 = ex < EX - 2 ? ex + 2 : ex;
#pragma unroll
          for (int c = 0; c < 5; ++c) {
            q_b[c] = sq[c][ey][ex - 1]; q_c[c] = sq[c][ey][ex];
            q_d[c] = sq[c][ey][ex + 1]; q_e[c] = sq[c][ey][e2];
            Db[c] = sW[c][ty][xn] - sW[c][ty][tx];
          }
          face_rev(P, Lam0, Ln, ns, nn, q_b, q_c, q_d, q_e, Db, fx_ij, F, G, LH, NA, NB);
        }
        const double Lb = lane_prev(LH) + LH, nub = lane_prev(NB) + NA;
        const double sd = sgn(ns) * iS, sv = fabs(ns) * iS, cp = nub * (sd - sv);
        pbc += -2.0 * nub * (sd + sv) + lane_prev(cp) + lane_next(cp);
#pragma unroll
        for (int c = 0; c < 5; ++c)
          oc[c] += Lb * V0[c] + lane_prev(F[c] - lane_prev(G[c])) - (F[c] - lane_next(G[c]));
        __builtin_amdgcn_sched_barrier(0);
        if (cx_ok) {
          const double qa1 = sp[ey + 1][ex], qz1 = sp[ey - 1][ex];
          const double jS = b1 ? rcp_nr(qa1 + 2.0 * pc + qz1) : 0.0;
          ly[ty][cx] = Lam1;
          ny[ty][cx] = b1 ? (qa1 - 2.0 * pc + qz1) * jS : 0.0;
          cy[ty][cx] = jS;
        }
      }
      load_ahead(2);
      // ---- zeta face (t-1, t) ----
      {
        // (only columns of interior nodes have zeta faces; in the others the
        // second k-ghost may be one that nothing reads)
        const bool zs = in_ij && t >= -1 && t <= L.nk;
        const double iS = zs ? rcp_nr(pp1 + 2.0 * pc + pm1) : 0.0;
        const double ns = zs ? (pp1 - 2.0 * pc + pm1) * iS : 0.0;
        double F[5], G[5], LH, NA, NB;
        {
          double qc[5], Db[5];
#pragma unroll
          for (int c = 0; c < 5; ++c) {
            qc[c] = sq[c][ey][ex];
            Db[c] = sW[c][ty][tx] - Wm[c];
          }
          const bool ok = ii && jj && t >= 0 && t <= L.nk && t > kb - 2;
          face_rev(P, L2, Lam2, ns2, ns, qm2, qm1, qc, qa, Db, ok, F, G, LH, NA, NB);
        }
        const double nub = nbz + NA, sd = sgn(ns2) * iS2, sv = fabs(ns2) * iS2, cp = nub * (sd - sv);
        pb2 += cp;
        pb1 -= 2.0 * nub * (sd + sv);
        pbc += cp;
#pragma unroll
        for (int c = 0; c < 5; ++c) {
          om2[c] += G[c];
          om1[c] += LH * V2[c] - F[c];
          oc[c] += LH * V2n[c] + F[c] - Gz[c];
          Gz[c] = G[c];
          V2[c] = V2n[c];
        }
        nbz = NB;
        L2 = Lam2;
        ns2 = ns;
        iS2 = iS;
      }
      load_ahead(3);
      load_ahead(4);
      // (the own column's loads before that arithmetic, the others after it: 16
      // together wait to issue)
      load5(kq->t.Q, on, qn);
      __builtin_amdgcn_sched_barrier(0);
      // plane t-2 is complete: the pressure adjoint to conserved variables
      double o[5];
      {
        const double ir = rcp_nr(qm2[0]), g = P.gm1 * pb2;
        const double u = qm2[1] * ir, vv = qm2[2] * ir, w = qm2[3] * ir;
        const bool any = pb2 != 0.0;  // (unused ghost corners may hold anything)
        o[0] = om2[0] + (any ? 0.5 * g * (u * u + vv * vv + w * w) : 0.0);
        o[1] = om2[1] - (any ? g * u : 0.0);
        o[2] = om2[2] - (any ? g * vv : 0.0);
        o[3] = om2[3] - (any ? g * w : 0.0);
        o[4] = om2[4] + g;
      }
#pragma unroll
      for (int c = 0; c < 5; ++c) {
        pin(o[c]);
        pin(om1[c]);
        pin(oc[c]);
        pin(Gz[c]);
      }
      pin(pb1);
      pin(pbc);
      pin(nbz);
      if (tl < DNH) load5(kq->t.Q, off(sh[tl], t + 1), hq);
      load5(kq->t.qb, ob, bn);
      Jn = ldo(kq->t.A.M + sb + 9 * fe, ob);
      __builtin_amdgcn_sched_barrier(0);
      lds_barrier();

      // ---- D: eta faces (ty, ty + 1) ----
      if (inner && ty < BY - 1 && cx_ok) {
        double q_b[5], q_c[5], q_d[5], q_e[5], Db[5], F[5], G[5], LH, NA, NB;
        const bool axf = axis && j == 0;
#pragma unroll
        for (int c = 0; c < 5; ++c) {
          q_c[c] = sq[c][ey][ex];
          q_d[c] = sq[c][ey + 1][ex];
          q_e[c] = sq[c][ey + 2][ex];
          // the face between the axis and j = 1 takes the cross-axis value by
          // linear extrapolation: d3 = Q(2) - 2 Q(1) + Q(0)
          q_b[c] = sq[c][ey - 1][ex];
          Db[c] = sW[c][ty + 1][tx] - sW[c][ty][tx];
        }
        if (axf) {
#pragma unroll
          for (int c = 0; c < 5; ++c) q_b[c] = 2.0 * q_c[c] - q_d[c];
        }
        face_rev(P, ly[ty][cx], ly[ty + 1][cx], ny[ty][cx], ny[ty + 1][cx], q_b, q_c, q_d, q_e, Db, fy_ij, F, G, LH, NA,
                 NB);
#pragma unroll
        for (int c = 0; c < 5; ++c) {
          fF[c][ty][cx] = F[c];
          fG[c][ty][cx] = G[c];
        }
        fL[ty][cx] = LH;
        fA[ty][cx] = NA;
        fB[ty][cx] = NB;
      }
      // what plane t-2's store needs
      const int k = t - 2;
      const bool st = out_ok && k >= kb;  // (k < ke always)
      const bool own = ii && jj && k >= 0 && k < L.nk;
      const unsigned ot = st ? col + (unsigned)(k - kr) * sk : col + kDissSpan.below * sk;
      double fl[5];
#pragma unroll
      for (int c = 0; c < 5; ++c) fl[c] = ldo(kq->t.Wk + (W_FL + c) * fe + sb, ot);
      lds_barrier();

      // ---- E: gather of the eta faces ----
      if (inner && cx_ok && ry_ok) {
        // faces below (ty - 1, ty) and above (ty, ty + 1), and one further on
        // either side
        const double Lb = fL[ty - 1][cx] + fL[ty][cx];
        const double n0 = fB[ty - 1][cx] + fA[ty][cx], nm = fB[ty - 2][cx] + fA[ty - 1][cx];
        const double np = fB[ty][cx] + fA[ty + 1][cx];
        auto cpw = [&](int r, double nub, double f) {  // nub times (sd - sv) or -2 (sd + sv) of row r's sensor
          const double ns = ny[r][cx], iS = cy[r][cx];
          const double sd = sgn(ns) * iS, sv = fabs(ns) * iS;
          return f == 1.0 ? nub * (sd - sv) : -2.0 * nub * (sd + sv);
        };
        pbc += cpw(ty, n0, 0.0) + cpw(ty - 1, nm, 1.0) + cpw(ty + 1, np, 1.0);
        // the face between the axis and j = 1: the axis node takes
        // -(A2 + A4) Dbar, node j = 1 takes (A2 + 2 A4) Dbar and the ghost
        // below the axis nothing
        const double x1 = axis && j == 1 ? 1.0 : 0.0, x0 = axis && j == 0 ? 2.0 : 0.0, xg = axis && j == -1 ? 0.0 : 1.0;
#pragma unroll
        for (int c = 0; c < 5; ++c) {
          oc[c] += Lb * sV[c][ty][cx] + (fF[c][ty - 1][cx] - x1 * fG[c][ty - 1][cx]) - (fF[c][ty][cx] - x0 * fG[c][ty][cx]) -
                   fG[c][ty - 2][cx] + xg * fG[c][ty + 1][cx];
          __builtin_amdgcn_sched_barrier(0);
        }
      }
#pragma unroll
      for (int c = 0; c < 5; ++c) {
        om2[c] = om1[c];
        om1[c] = oc[c];
        qm2[c] = qm1[c];
        qm1[c] = sq[c][ey][ex];
        Wm[c] = sW[c][ty][tx];
        qw[c] = qa[c];
        qa[c] = qn[c];
      }
      pb2 = pb1;
      pb1 = pbc;
      pm1 = pc;
      Wset(t + 1, Wc);
      __builtin_amdgcn_sched_barrier(0);
      wait_vm<0>();  // all loads of this plane, before the stores (see les_stage.hip)
      if (st) {
#pragma unroll
        for (int c = 0; c < 5; ++c) o[c] += fl[c];
        if (own) {
#pragma unroll
          for (int c = 0; c < 5; ++c) sto(kq->qout + c * fe + sb, ot, o[c]);
          // (the fold finishes the nodes with images)
          if (kq->fbar && i == kq->i_f && !has_images(kq->t.A, i, j, k)) {
#pragma unroll
            for (int c = 0; c < 5; ++c) kq->fbar[((long long)c * L.nk + k) * L.nj + j] += kq->fw * o[c];
          }
        } else {
#pragma unroll
          for (int c = 0; c < 5; ++c) sto(kq->t.Wk + (W_GG + c) * fe + sb, ot, o[c]);
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Face ghosts: the adjoint Gbar of each ghost G = face_value(q_r) of an active
// face (both layers, and their periodic images) becomes its pull-back to the
// boundary node, (dG/dq_r)^T Gbar, in place (W_GG).  Ghosts of two Dirichlet
// directions are frozen and carry nothing.  One thread per ghost, all five
// columns of the Jacobian from one evaluation of the rule; the fold then adds
// face ghosts as it adds periodic images.  (One thread per boundary node and
// column, which evaluated the rule for each image in turn, took 41 us on the
// 128 x 64 x 121 O-grid with a far-field face; this takes 12.)
// ---------------------------------------------------------------------------
// ghosts of face f = 2 d + hi: two layers, and the other two directions with
// the ghosts of periodic ones
__host__ __device__ inline int face_extent(const AdjK& A, int e) {
  return A.per[e] ? (e == 0 ? A.L.ni : (e == 1 ? A.L.nj : A.L.nk)) + 4 : (e == 0 ? A.L.ni : (e == 1 ? A.L.nj : A.L.nk));
}
inline long long face_ghosts(const AdjK& A) {
  long long n = 0;
  for (int f = 0; f < 6; ++f)
    if (A.F.type[f] != 0) n += 2LL * face_extent(A, (f / 2 + 1) % 3) * face_extent(A, (f / 2 + 2) % 3);
  return n;
}

__global__ void __launch_bounds__(64) k_adj_face(AdjK A, const double* __restrict__ Q, double* __restrict__ G,
                                                 unsigned total) {
  const Layout& L = A.L;
  unsigned x = blockIdx.x * 64 + threadIdx.x;
  if (x >= total) return;
  const int nn[3] = {L.ni, L.nj, L.nk};
  int d = 0, hi = 0;
  unsigned m1 = 1, m2 = 1;  // extents of the other directions
  for (int f = 0; f < 6; ++f) {
    if (A.F.type[f] == 0) continue;
    d = f / 2;
    hi = f & 1;
    m1 = face_extent(A, (d + 1) % 3);
    m2 = face_extent(A, (d + 2) % 3);
    if (x < 2 * m1 * m2) break;
    x -= 2 * m1 * m2;
  }
  const unsigned row = x / m1, layer = row / m2;
  int g[3], r[3];  // the ghost and its boundary node
  const int u[2] = {(int)(x - row * m1), (int)(row - layer * m2)};
#pragma unroll
  for (int e = 0; e < 3; ++e) {
    if (e == d) {
      g[e] = hi ? nn[e] + (int)layer : -1 - (int)layer;
      r[e] = hi ? nn[e] - 1 : 0;
    } else {
      const int p = A.per[e], y = u[e == (d + 1) % 3 ? 0 : 1] - (p ? 2 : 0);
      g[e] = y;
      r[e] = p && y < 0 ? y + p : (p && y >= nn[e] ? y - p : y);
    }
  }
  const long long fe = L.fe, ng = L.at(g[0], g[1], g[2]), nr = L.at(r[0], r[1], r[2]);
  double gb[5], qo[5] = {0, 0, 0, 0, 0}, nv[3];
  Dual5 qr[5], out[5];
#pragma unroll
  for (int c = 0; c < 5; ++c) {
    gb[c] = G[c * fe + ng];
    qr[c].v = Q[c * fe + nr];
    qr[c].d[c] = 1.0;
    if (A.F.outside) qo[c] = A.F.outside[c * fe + ng];
  }
  face_normal(L, A.F, d, hi, r[0], r[1], r[2], nv);
  face_value<Dual5>(A.F.type[2 * d + hi], A.F.gamma, A.F.p_exit[2 * d + hi], nv, qr, qo, out);
#pragma unroll
  for (int c = 0; c < 5; ++c) {  // column c of the Jacobian
    double dot = 0.0;
#pragma unroll
    for (int m = 0; m < 5; ++m) dot += out[m].d[c] * gb[m];
    G[c * fe + ng] = dot;
  }
}

// ---------------------------------------------------------------------------
// Fold: every interior node with ghost images adds their adjoints (W_GG), in a
// fixed order: periodic images (x +- period along each periodic axis, all
// combinations), the face ghosts pulled back to it, and the images across
// the polar axis.  Only nodes with a coordinate in the band of some axis have
// images; threads enumerate them as three disjoint slabs (band of k; core of
// k x band of j; core of k and j x band of i): 12 us on that O-grid, where a
// pass over every interior node took 21.
// ---------------------------------------------------------------------------
__device__ __forceinline__ int core_coord(const AdjK& A, int d, int u) {
#pragma unroll
  for (int q = 0; q < 4; ++q)  // (bands are ascending)
    if (q < A.nband[d] && u >= A.band[d][q]) ++u;
  return u;
}

__global__ void __launch_bounds__(256) k_adj_fold(AdjK A, const double* __restrict__ Wk, double* __restrict__ qout,
                                                  double* __restrict__ fbar, int i_f, double fw) {
  const Layout& L = A.L;
  const int nn[3] = {L.ni, L.nj, L.nk};
  const unsigned ni = nn[0], nj = nn[1];
  const unsigned b0 = A.nband[0], b1 = A.nband[1], c1 = nj - b1, c2 = nn[2] - A.nband[2];
  const unsigned S2 = A.nband[2] * nj * ni, S1 = c2 * b1 * ni, S0 = c2 * c1 * b0;
  unsigned t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= S2 + S1 + S0) return;
  int i, j, k;
  if (t < S2) {
    const unsigned row = t / ni, kk = row / nj;
    i = (int)(t - row * ni);
    j = (int)(row - kk * nj);
    k = A.band[2][kk];
  } else if (t < S2 + S1) {
    t -= S2;
    const unsigned row = t / ni, kk = row / b1;
    i = (int)(t - row * ni);
    j = A.band[1][row - kk * b1];
    k = core_coord(A, 2, (int)kk);
  } else {
    t -= S2 + S1;
    const unsigned row = t / b0, kk = row / c1;
    i = A.band[0][t - row * b0];
    j = core_coord(A, 1, (int)(row - kk * c1));
    k = core_coord(A, 2, (int)kk);
  }
  const int id[3] = {i, j, k}, bc[3] = {A.bc0, A.bc1, A.bc2};
  int cand[3][3], nc[3];
  bool face[3];  // the images along d are face ghosts
  for (int d = 0; d < 3; ++d) {
    nc[d] = 1;
    cand[d][0] = id[d];
    face[d] = false;
    const int p = A.per[d];
    if (p) {
      if (id[d] + p >= nn[d] && id[d] + p <= nn[d] + 1) cand[d][nc[d]++] = id[d] + p;
      if (id[d] - p <= -1 && id[d] - p >= -2) cand[d][nc[d]++] = id[d] - p;
    } else if (id[d] == 0 && bc[d] == 1 && A.F.type[2 * d] != 0) {
      cand[d][1] = -1;
      cand[d][2] = -2;
      nc[d] = 3;
      face[d] = true;
    } else if (id[d] == nn[d] - 1 && (bc[d] == 1 || bc[d] == 3) && A.F.type[2 * d + 1] != 0) {
      cand[d][1] = nn[d];
      cand[d][2] = nn[d] + 1;
      nc[d] = 3;
      face[d] = true;
    }
  }
  const long long fe = L.fe, n0 = L.at(i, j, k);
  const double* G = Wk + (long long)W_GG * fe;
  double s[5];
  for (int c = 0; c < 5; ++c) s[c] = qout[c * fe + n0];
  for (int a = 0; a < nc[0]; ++a)
    for (int b = 0; b < nc[1]; ++b)
      for (int e = 0; e < nc[2]; ++e) {
        if (!(a | b | e)) continue;
        const int nface = (a && face[0]) + (b && face[1]) + (e && face[2]);
        if (nface > 1) continue;  // edge ghost: frozen
        const long long g = L.at(cand[0][a], cand[1][b], cand[2][e]);
        for (int c = 0; c < 5; ++c) s[c] += G[c * fe + g];
      }
  if (A.axis && (j == 1 || j == 2)) {
    // ghosts (i', -j, k') across the polar axis copy node (w(i'), j,
    // (w(k') + (nk - 1)/2) mod (nk - 1)), w wrapping a ghost index (i' a
    // periodic image of i; ghosts of a Dirichlet i side below the axis are
    // edges and keep their values)
    // the ghost azimuths kk in [-2, nk + 1] with ((w(kk) + half) mod p) = k,
    // w(kk) = kk on [0, nk) and (kk + p) mod p outside, in ascending kk:
    // -2, -1, t0, t0 + p (when t0 = 0), nk, nk + 1 with t0 = (k - half) mod p
    const int p = L.nk - 1, half = p / 2;
    const int t0 = ((k - half) % p + p) % p;
    const int kks[6] = {-2, -1, t0, t0 + p, L.nk, L.nk + 1};
    for (int a = 0; a < nc[0]; ++a) {
      if (a && face[0]) continue;
      for (int q = 0; q < 6; ++q) {
        const int kk = kks[q];
        if (q == 3 && kk >= L.nk) continue;  // t0 + p lies in [0, nk) only for t0 = 0
        const int w2 = (kk >= 0 && kk < L.nk) ? kk : (kk + p) % p;
        if ((w2 + half) % p != k) continue;
        const long long g = L.at(cand[0][a], -j, kk);
        for (int c = 0; c < 5; ++c) s[c] += G[c * fe + g];
      }
    }
  }
  for (int c = 0; c < 5; ++c) qout[c * fe + n0] = s[c];
  if (fbar && i == i_f)
    for (int c = 0; c < 5; ++c) fbar[((long long)c * L.nk + k) * L.nj + j] += fw * s[c];
}

// Reverse of the centerline condition: the forward writes the mean of the ring
// (i, 1, k'), k' = 0 .. nk - 2, to every axis node (i, 0, k), k = 0 .. nk - 1;
// so every ring node receives the sum of the axis adjoints over k divided by
// nk - 1, and the axis adjoints are consumed (set to 0).  Per (i, variable)
// lane l sums k = l, l + 64, ... ascending, and the partial sums are added by
// a fixed shuffle tree; blocks of 16 i x 64 lanes read and write row segments
// of 16 nodes (128 x 64 x 121: 5.8 us, one i a block 7.5).
__global__ void __launch_bounds__(1024) k_axis_avg_adj(Layout L, double* __restrict__ q) {
  __shared__ double part[64][17], mean[16];
  const int ni16 = (L.ni + 15) / 16;
  const int f = blockIdx.x / ni16, ii = threadIdx.x % 16, l = threadIdx.x / 16;
  const int i = blockIdx.x % ni16 * 16 + ii;
  double* a = q + f * L.fe;
  double sum = 0.0;
  if (i < L.ni)
    for (int k = l; k < L.nk; k += 64) {
      const long long n = L.at(i, 0, k);
      sum += a[n];
      a[n] = 0.0;
    }
  part[l][ii] = sum;
  __syncthreads();
  sum = wave_sum(part[threadIdx.x % 64][threadIdx.x / 64]);
  if (threadIdx.x % 64 == 0) mean[threadIdx.x / 64] = sum / (double)(L.nk - 1);
  __syncthreads();
  const double share = mean[ii];
  if (i < L.ni)
    for (int k = l; k < L.nk - 1; k += 64) a[L.at(i, 1, k)] += share;
}

// fbar[c][k][j] += w q_c on the source plane i_f (interior nodes).
__global__ void __launch_bounds__(256) k_adj_source(Layout L, const double* __restrict__ q, double* __restrict__ fbar,
                                                    int i_f, double w) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= L.nj * L.nk) return;
  const int j = t % L.nj, k = t / L.nj;
  const long long n = L.at(i_f, j, k);
  for (int c = 0; c < 5; ++c) fbar[((long long)c * L.nk + k) * L.nj + j] += w * q[c * L.fe + n];
}

// Adjoints of the six stage states of a step (5 fields each).
struct Terms {
  double* p[6];
};

// Qbar = the sum of the stages' adjoints, in order from Qbar itself (p[0]) to
// the last stage's, on the interior; blockIdx.y is the component.  Bound by
// memory: 6 reads and 1 write a component and step, where a running sum kept
// by every stage took 10 reads and 5 writes and a copy of Qbar (24 us on the
// 128 x 64 x 64 jet; taken inside the last stage's dissipation pass, whose few
// waves wait for the loads, it cost 115).
__global__ void __launch_bounds__(256) k_adj_sum(Layout L, Terms z) {
  const unsigned t = blockIdx.x * blockDim.x + threadIdx.x;
  const unsigned ni = L.ni, nij = (unsigned)L.ni * L.nj;
  if (t >= nij * (unsigned)L.nk) return;
  const long long n = L.at((int)(t % ni), (int)((t % nij) / ni), (int)(t / nij)) + blockIdx.y * L.fe;
  double x = z.p[0][n];
#pragma unroll
  for (int m = 1; m < 6; ++m) x += z.p[m][n];
  z.p[0][n] = x;
}

inline unsigned nb(long long n, int b) { return (unsigned)((n + b - 1) / b); }

// A tiled pass: blocks over tiles of tx x ty output nodes, whose first column
// lies `lead` before the output box.
struct Pass {
  int tx, ty, lead;
  Span span;
  int halo;  // planes marched around a segment
};
constexpr Pass kFluxPass{TX, TY, 0, kStageSpan, 2}, kDissPass{DTX, DTY, 1, kDissSpan, 4};

Schedule pass_schedule(const AdjK& A, const Pass& p, int& ntx, int& nty) {
  ntx = (A.hi[0] - A.lo[0] + p.lead + p.tx) / p.tx;
  nty = (A.hi[1] - A.lo[1] + p.ty) / p.ty;
  return segment_schedule((long long)ntx * nty, A.hi[2] - A.lo[2] + 1, A.mach.cus, segment_kmax(A.L, p.span),
                          p.halo);
}

// qout = (dR/dQ|Q)^T (coef * qb) on the interior; in the Runge-Kutta
// reverse, fbar[c][k][j] += fw qout_c on the source plane i_f (fbar non-null).
hipError_t residual_vjp(hipStream_t s, const AdjK& A, const double* Q, const double* qb, double coef, double* Wk,
                        double* qout, double* fbar = nullptr, int i_f = -1, double fw = 0.0) {
  const Layout& L = A.L;
  // nodes with ghost images (see k_adj_fold)
  const long long c1 = L.nj - A.nband[1], c2 = L.nk - A.nband[2];
  const long long nBand = ((long long)A.nband[2] * L.nj + c2 * A.nband[1]) * L.ni + c2 * c1 * A.nband[0];
  auto tiles = [&](const Pass& p) {
    TileArgs ta{A, Q, qb, coef, A.P.gamma_R / A.P.gamma, 1.0 / A.P.gm1, Wk, 0, 0, {}, 0, A.mach.xcds};
    ta.sch = pass_schedule(A, p, ta.ntx, ta.nty);
    ta.per_xcd = (ta.sch.nblocks + ta.nxcd - 1) / ta.nxcd;
    return ta;
  };
  const TileArgs tf = tiles(kFluxPass);
  k_adj_flux<<<tf.per_xcd * tf.nxcd, NT, 0, s>>>(tf);
  const DissArgs td{tiles(kDissPass), qout, fbar, fw, i_f};
  if (A.P.alpha_half)
    k_adj_diss<true><<<td.t.per_xcd * td.t.nxcd, NT, 0, s>>>(td);
  else
    k_adj_diss<false><<<td.t.per_xcd * td.t.nxcd, NT, 0, s>>>(td);
  const long long ng = face_ghosts(A);
  if (ng > 0) k_adj_face<<<nb(ng, 64), 64, 0, s>>>(A, Q, Wk + (long long)W_GG * L.fe, (unsigned)ng);
  if (nBand > 0) k_adj_fold<<<nb(nBand, 256), 256, 0, s>>>(A, Wk, qout, fbar, i_f, fw);
  return hipGetLastError();
}

}  // namespace

bool adjoint_fits(const Layout& L) {
  const long long box = (long long)(L.ni + 4) * (L.nj + 4) * (L.nk + 4);
  return box < (1LL << 30) && segment_kmax(L, kDissSpan) >= 1;
}

void adjoint_segments(const AdjArgs& a, bool diss, SegmentBounds& b) {
  const AdjK A = make_adjk(a);
  const Pass& p = diss ? kDissPass : kFluxPass;
  int ntx, nty;
  b = {0, A.lo[2], A.hi[2], p.span.below, p.span.ahead};
  if (segment_kmax(a.L, p.span) < 1) return;
  const Schedule s = pass_schedule(A, p, ntx, nty);
  b.planes = s.kl > s.kc ? s.kl : s.kc;
}

size_t adjoint_work_elems(const Layout& L) { return (size_t)W_NF * (size_t)L.fe; }

hipError_t launch_axis_avg_adjoint(hipStream_t s, const Layout& L, double* qbar) {
  k_axis_avg_adj<<<5 * nb(L.ni, 16), 1024, 0, s>>>(L, qbar);
  return hipGetLastError();
}

hipError_t run_residual_vjp(hipStream_t s, const AdjArgs& a, const double* Q, const double* Rbar, double* Qbar,
                            double* work) {
  const AdjK A = make_adjk(a);
  hipError_t e = residual_vjp(s, A, Q, Rbar, 1.0, work, Qbar);
  // the residual reads the state after the centerline condition
  if (e == hipSuccess && A.axis) e = launch_axis_avg_adjoint(s, a.L, Qbar);
  return e;
}

hipError_t run_adjoint_step(hipStream_t s, const AdjArgs& a, const double* ckpt, double dt, double* Qbar,
                            double* fbar, double* work) {
  const AdjK A = make_adjk(a);
  const Layout& L = a.L;
  const long long fe = L.fe;
  const long long nIn = (long long)L.ni * L.nj * L.nk;
  // With the polar axis every stage input and the step's result pass
  // through the centerline condition C (linear): Q^{n+1} = C(Z_5) and the
  // stage input of stage l > 1 is C(Z_l) for the raw stage output Z_l, so
  // the reverse applies C^T to Qbar first, to each stage's result before it
  // is used, and to the final sum (the step's input was C(Q^n)).  The
  // source-plane update then takes the transformed adjoint, in a pass of its
  // own.
  const bool want_f = fbar && a.i_f >= 0;
  hipError_t e = hipSuccess;
  if (A.axis && (e = launch_axis_avg_adjoint(s, L, Qbar)) != hipSuccess) return e;
  // fbar += alpha_5 dt Qbar
  if (want_f) k_adj_source<<<nb((long long)L.nj * L.nk, 256), 256, 0, s>>>(L, Qbar, fbar, a.i_f, rk_alpha(4) * dt);
  // Every stage's result has a buffer of its own and the sum is taken once.
  Terms z;
  z.p[0] = Qbar;
  for (int m = 1; m < 6; ++m) z.p[m] = work + (long long)(W_Z + 5 * (m - 1)) * fe;
  for (int l = 4; l >= 0; --l) {
    const double al = rk_alpha(l) * dt;
    // qbar_{l-1} = (dR/dQ|Q^(l-1))^T (-alpha_l dt qbar_l),
    // fbar += alpha_{l-1} dt qbar_{l-1}
    const double* Ql = ckpt + (long long)l * 5 * fe;
    double* const qnext = z.p[5 - l];
    const bool f_next = want_f && l > 0;
    const bool f_here = f_next && !A.axis;
    e = residual_vjp(s, A, Ql, z.p[4 - l], -al, work, qnext, f_here ? fbar : nullptr, a.i_f,
                     f_here ? rk_alpha(l - 1) * dt : 0.0);
    if (e != hipSuccess) return e;
    if (A.axis && l > 0) {
      e = launch_axis_avg_adjoint(s, L, qnext);
      if (e != hipSuccess) return e;
      if (f_next) k_adj_source<<<nb((long long)L.nj * L.nk, 256), 256, 0, s>>>(L, qnext, fbar, a.i_f,
                                                                                rk_alpha(l - 1) * dt);
    }
  }
  k_adj_sum<<<dim3(nb(nIn, 256), 5), 256, 0, s>>>(L, z);
  // (the centerline condition of the step's input acts on the sum)
  if (A.axis && (e = launch_axis_avg_adjoint(s, L, Qbar)) != hipSuccess) return e;
  return hipGetLastError();
}

}  // namespace les
