// les_dynamic.hip -- dynamic SGS closure for gfx950: the per-column
// coefficients of mu_sgs = C rho D^2 |S| and kappa_sgs = Cp D_T rho D^2 |S|
// (the paper fixes Pr_sgs = 0.9 for static closures only, Sec. 3, Eq. 5).
//
// Germano's identity between the grid filter and a test filter of twice its
// width, in the Favre form of Moin, Squires, Cabot and Lee (1991), with
// Lilly's least squares summed over the periodic k direction:
//   C   = max(0, <L^d : M> / <M : M>),   D_T = max(0, <K . N> / <N . N>),
//   L_ij = (rho u_i u_j)^ - (rho u_i)^ (rho u_j)^ / rho^,
//   M_ij = 2 (D^2 rho |S| S^d_ij)^ - 2 (2D)^2 rho^ |S~| S~^d_ij,
//   K_j  = (rho u_j T)^ - (rho u_j)^ (rho T)^ / rho^,
//   N_j  = (D^2 rho |S| dT/dx_j)^ - (2D)^2 rho^ |S~| dT~/dx_j,
// ^ the test filter (weights 1/4, 1/2, 1/4 along each index), u~ and T~ the
// test-filtered Favre velocity and temperature, D = (1/J)^(1/3).
//
// Two launches per evaluation:
//   k_dyn_fused   per (i, j) tile and chunk of k planes: the 23 grid-level
//                 fields (rho, rho u, rho T, rho u u, rho u T and the 9 strain
//                 and temperature-gradient products), the test filter along
//                 i, j and k, the test-filtered gradients and the four
//                 contractions, summed over the chunk's k in ascending order;
//   k_dyn_coef    per padded column: the chunk sums added in ascending
//                 order (a fixed order) and the clipped ratios; ghost
//                 columns take the wrapped (periodic) or nearest interior
//                 (Dirichlet) column, across the polar axis the ring column
//                 of the same radius; the axis column takes ring 1's.
// The sums over k run over the distinct planes (nk - 1 along a superposed
// direction).  On the polar axis (a node of zero volume) the strain and
// temperature-gradient products are 0 and no contractions are formed.
// The filter is separable and applied along i, then j, then k, each a
// three-point sum evaluated left to right.

#include "les_dynamic.hpp"

namespace les {

namespace {

constexpr int NRAW = 23;
// symmetric index pairs (a <= b) in the order of the raw fields: 00 01 02 11 12 22
__device__ constexpr int pair_a(int q) { return q < 3 ? 0 : (q < 5 ? 1 : 2); }
__device__ constexpr int pair_b(int q) { return q < 3 ? q : (q < 5 ? q - 2 : 2); }

// strain rate's deviatoric part (by pairs) and |S| = sqrt(2 S:S) from du[a][x]
__device__ __forceinline__ void dyn_strain(const double du[][3], double Sd[6], double& mag) {
  double ss = 0.0;
#pragma unroll
  for (int q = 0; q < 6; ++q) {
    const int a = pair_a(q), b = pair_b(q);
    Sd[q] = a == b ? du[a][a] : 0.5 * (du[a][b] + du[b][a]);
    ss += (a == b ? 1.0 : 2.0) * Sd[q] * Sd[q];
  }
  const double tr = (Sd[0] + Sd[3] + Sd[5]) * (1.0 / 3.0);
  Sd[0] -= tr;
  Sd[3] -= tr;
  Sd[5] -= tr;
  double r = sqrt_pos(2.0 * ss);
  pin(r);  // (no branch)
  mag = ss > 0.0 ? r : 0.0;
}

// Patch of 32 x 16 nodes (one thread each) whose inner 28 x 12 nodes are the
// tile a block contracts.
constexpr int DBX = 32, DBY = 16, DNT = DBX * DBY;
constexpr int DTI = DBX - 4, DTJ = DBY - 4;

struct DynArgs {
  Layout L;
  Phys P;
  Wrap wrap;
  const double* M;
  double* Xp;
  int axis, nks, nch, kc, ntx, nblocks, per_xcd, nxcd, nseg;
};

// One pass: raw fields, test filter and contractions, marching in k.  In
// step t of a segment a thread
//   C  forms the base fields of plane t+1 and the other 18 of plane t from
//      primitives in registers (the xi neighbours' by lane shifts, a patch row
//      being 32 lanes; the eta neighbours' from LDS), filters them along i
//      across lanes, and writes the sums to LDS;
//   E  filters along j from LDS and along k in registers, carried as the
//      pending sum of two planes and the last plane: the base fields of plane
//      t and the others of plane t-1 are complete, so the test-filtered
//      velocity and temperature are known at planes t-2 .. t and plane t-1 is
//      contracted.
// The filter's sums are taken with the weights 1, 2, 1, so filtered fields are
// 64 times and contractions 64^2 times their values (exactly: the rounding is
// that of the scaled weights), which the ratios of contractions cancel.
// Q and the metrics are read once per patch node (1.5 times in all), and no
// field is written: the two passes this replaces wrote 23 filtered fields,
// read them back and used full divisions and cube roots.  Bound by the VALU
// issue rate (about 800 instructions a node and step, a quarter of them lane
// shifts, at two waves a SIMD).  Each sum keeps its two earlier planes in
// registers (92 of 256), so the order of E keeps few other values at a time.
// Measured on the 256 x 128 x 128 jet: 274 us, the two passes 490 + 302; on a
// 60 x 44 x 33 block about 27 us, 480.  (Priorities: see wave_priority; 1 % of
// a step on either block.)
template <class QI>
__global__ void __launch_bounds__(DNT) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_dyn_fused(DynArgs a, const QI* __restrict__ Q) {
  __shared__ double sF[NRAW][DBY][DBX];
  __shared__ double sP[4][DBY][DBX];  // u, v, w, T of plane t
  __shared__ double sU[4][DBY][DBX];  // test-filtered u, v, w, T of plane t-1
  const int v = (blockIdx.x % a.nxcd) * a.per_xcd + blockIdx.x / a.nxcd;
  if (v >= a.nblocks) return;
  const Layout& L = a.L;
  const long long fe = L.fe;
  const int tx = threadIdx.x % DBX, ty = threadIdx.x / DBX;
  const long long ncoli = (long long)L.ni * L.nj;
  for (int wq = v; wq < a.nseg; wq += a.nblocks) {
    const int ntiles = a.nseg / a.nch;
    const int ch = wq / ntiles, tile = wq % ntiles;
    const int kb = ch * a.kc, ke = min(a.nks, kb + a.kc);
    const int i = (tile % a.ntx) * DTI - 2 + tx, j = (tile / a.ntx) * DTJ - 2 + ty;
    const bool out = tx >= 2 && tx < DBX - 2 && ty >= 2 && ty < DBY - 2 && i < L.ni && j < L.nj;
    // on the polar axis (a node of zero volume) the strain is 0/0: 0 there
    const bool grad = !(a.axis && j == 0);
    // (nodes off the padded box repeat its edge; no output depends on them)
    const int ic = min(i, L.ni + 1), jc = min(j, L.nj + 1);
    const unsigned col = (unsigned)L.at(ic, jc, 0);
    const unsigned qcol = wrap_column(L, a.wrap, ic, jc);
    auto load_state = [&](int k, QI q[5]) {
      const PlaneRef p = wrap_plane(L, a.wrap, min(max(k, -2), L.nk + 1));
      const unsigned qo = wrap_offset(qcol, p);
#pragma unroll
      for (int c = 0; c < 5; ++c) q[c] = ldo(Q + p.base + c * fe, qo);
    };
    auto load_metrics = [&](int k, int c0, double m[10]) {  // five of the ten fields
      const double* const Mk = a.M + (long long)min(max(k, -2), L.nk + 1) * L.sk;
#pragma unroll
      for (int c = 0; c < 5; ++c) m[c0 + c] = ldo(Mk + (c0 + c) * fe, col);
    };
    auto prims = [&](const QI q[5], double p[5]) {
      p[0] = (double)q[0];
      const double ir = rcp_nr(p[0]);
      p[1] = (double)q[1] * ir;
      p[2] = (double)q[2] * ir;
      p[3] = (double)q[3] * ir;
      const double pr = a.P.gm1 * ((double)q[4] - 0.5 * p[0] * (p[1] * p[1] + p[2] * p[2] + p[3] * p[3]));
      p[4] = pr * ir * a.P.inv_R;
    };
    double pend[NRAW], last[NRAW], s[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int q = 0; q < NRAW; ++q) pend[q] = last[q] = 0.0;
    double pm[4], pc[5], pn[5];   // primitives of planes t-1, t, t+1
    double um[4], uc[4], rc = 0;  // test-filtered u, v, w, T of planes t-2, t-1; rho^ of plane t-1
    double mo[9], do2 = 0.0;      // J m and D^2 of plane t-1
    QI qn[5];                     // Q of plane t+1 (in flight until C)
    double mn[10];                // metrics of plane t (in flight until C)
    load_state(kb - 2, qn);
    load_metrics(kb - 3, 0, mn);
    load_metrics(kb - 3, 5, mn);
#pragma unroll
    for (int c = 0; c < 4; ++c) pm[c] = um[c] = uc[c] = 0.0;
#pragma unroll
    for (int c = 0; c < 5; ++c) pc[c] = 0.0;
#pragma unroll
    for (int c = 0; c < 9; ++c) mo[c] = 0.0;

    for (int t = kb - 3; t <= ke; ++t) {
      const bool full = t >= kb - 1, con = t > kb;  // (both uniform)
      int tl = threadIdx.x;  // (LDS addresses are formed again in each step)
      asm volatile("" : "+v"(tl));
      const int tx = tl % DBX, ty = tl / DBX;
      const int yp = ty < DBY - 1 ? ty + 1 : ty, ym = ty > 0 ? ty - 1 : ty;
      // ---- C ----
      wave_priority<3>();
      auto put = [&](int q, double f) { sF[q][ty][tx] = fma(2.0, f, lane_prev(f)) + lane_next(f); };
      prims(qn, pn);
      put(0, pn[0]);
#pragma unroll
      for (int c = 1; c < 5; ++c) put(c, pn[0] * pn[c]);
      double de[4];  // eta differences of the test-filtered fields, plane t-1
#pragma unroll
      for (int c = 0; c < 4; ++c) de[c] = 0.5 * (sU[c][yp][tx] - sU[c][ym][tx]);
      double m[9], d2;
      {
        const double J = mn[9];
#pragma unroll
        for (int c = 0; c < 9; ++c) m[c] = J * mn[c];
        const double D = icbrt(fabs(J));  // (D^2 has no sign: left-handed grids, J < 0)
        d2 = D * D;
      }
      wave_priority<2>();
      __builtin_amdgcn_sched_barrier(0);
      if (full) {
        const double rho = pc[0];
        {
          const double ru[3] = {rho * pc[1], rho * pc[2], rho * pc[3]};
#pragma unroll
          for (int q = 0; q < 6; ++q) put(5 + q, ru[pair_a(q)] * pc[1 + pair_b(q)]);
#pragma unroll
          for (int c = 0; c < 3; ++c) put(11 + c, ru[c] * pc[4]);
        }
        wave_priority<1>();
        __builtin_amdgcn_sched_barrier(0);
        double du[4][3];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const double d0 = 0.5 * (lane_next(pc[1 + c]) - lane_prev(pc[1 + c]));
          const double d1 = 0.5 * (sP[c][yp][tx] - sP[c][ym][tx]);
          const double dz = 0.5 * (pn[1 + c] - pm[c]);
#pragma unroll
          for (int x = 0; x < 3; ++x) du[c][x] = m[x] * d0 + m[3 + x] * d1 + m[6 + x] * dz;
        }
        double Sd[6], mag;
        dyn_strain(du, Sd, mag);
        const double w = d2 * rho * mag;
#pragma unroll
        for (int q = 0; q < 6; ++q) put(14 + q, grad ? w * Sd[q] : 0.0);
#pragma unroll
        for (int c = 0; c < 3; ++c) put(20 + c, grad ? w * du[3][c] : 0.0);
      }
      // (the next plane's 15 loads in three groups: issued together in E they
      // wait in the memory pipeline's queue, 5680 against 5510 us for two steps)
      load_state(t + 2, qn);
      lds_barrier();

      // ---- E ----
      wave_priority<3>();
      load_metrics(t + 1, 0, mn);
      // (the LDS reads run one field ahead of the sums)
      double r0 = sF[0][ym][tx], r1 = sF[0][ty][tx], r2 = sF[0][yp][tx];
      auto take = [&](int q, int qnext) {
        const double g0 = r0, g1 = r1, g2 = r2;
        r0 = sF[qnext][ym][tx];
        r1 = sF[qnext][ty][tx];
        r2 = sF[qnext][yp][tx];
        __builtin_amdgcn_sched_barrier(0);
        const double g = fma(2.0, g1, g0) + g2;
        const double f = pend[q] + g;
        pend[q] = fma(2.0, g, last[q]);
        last[q] = g;
        pin(pend[q]);
        pin(last[q]);
        __builtin_amdgcn_sched_barrier(0);
        return f;
      };
      double rn, un[4];
      rn = take(0, 1);
#pragma unroll
      for (int c = 0; c < 4; ++c) un[c] = take(1 + c, 2 + c);
      {
        const double ir = rcp_nr(rn);
#pragma unroll
        for (int c = 0; c < 4; ++c) un[c] *= ir;
      }
      // plane t-1: (2 D)^2 rho^ |S~|, S~^d and dT~
      double w = 0.0, Sd[6], dT[3];
      {
        double du[4][3];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const double dx = 0.5 * (lane_next(uc[c]) - lane_prev(uc[c])), dz = 0.5 * (un[c] - um[c]);
#pragma unroll
          for (int x = 0; x < 3; ++x) du[c][x] = mo[x] * dx + mo[3 + x] * de[c] + mo[6 + x] * dz;
        }
        double mag;
        dyn_strain(du, Sd, mag);
        w = 4.0 * do2 * rc * mag;
#pragma unroll
        for (int x = 0; x < 3; ++x) pin(dT[x] = du[3][x]);
#pragma unroll
        for (int q = 0; q < 6; ++q) pin(Sd[q]);
        pin(w);
      }
      load_metrics(t + 1, 5, mn);
      wave_priority<2>();
      __builtin_amdgcn_sched_barrier(0);
      if (full) {
        double Lm[6];
#pragma unroll
        for (int q = 0; q < 6; ++q) Lm[q] = take(5 + q, q < 5 ? 6 + q : 14) - rc * (uc[pair_a(q)] * uc[pair_b(q)]);
        const double tr = (Lm[0] + Lm[3] + Lm[5]) * (1.0 / 3.0);
        Lm[0] -= tr;
        Lm[3] -= tr;
        Lm[5] -= tr;
        wave_priority<1>();
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < 6; ++q) {
          const double Mq = 2.0 * take(14 + q, q < 5 ? 15 + q : 11) - 2.0 * w * Sd[q];
          const double two = pair_a(q) == pair_b(q) ? 1.0 : 2.0;
          s[0] += two * Lm[q] * Mq;
          s[1] += two * Mq * Mq;
        }
        wave_priority<0>();
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          const double K = take(11 + c, 20 + c) - rc * (uc[c] * uc[3]);
          const double N = take(20 + c, c < 2 ? 12 + c : 22) - w * dT[c];
          s[2] += K * N;
          s[3] += N * N;
        }
        if (!con) {  // (plane kb - 1 is not the chunk's)
#pragma unroll
          for (int q = 0; q < 4; ++q) s[q] = 0.0;
        }
      }
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        sU[c][ty][tx] = un[c];
        sP[c][ty][tx] = pn[1 + c];
        um[c] = uc[c];
        uc[c] = un[c];
        pm[c] = pc[1 + c];
      }
      rc = rn;
#pragma unroll
      for (int c = 0; c < 5; ++c) pc[c] = pn[c];
#pragma unroll
      for (int c = 0; c < 9; ++c) mo[c] = m[c];
      do2 = d2;
      lds_barrier();
    }
    if (out) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
        a.Xp[((long long)q * a.nch + ch) * ncoli + (long long)j * L.ni + i] = grad ? s[q] : 0.0;
    }
  }
}

__device__ inline int dyn_src(int x, int n, int bc) {
  if (bc == 3) {
    // polar axis (j): column -m across the axis is ring column m, the axis
    // column takes ring 1's, the far side is Dirichlet
    const int y = x < 0 ? -x : (x < n ? x : n - 1);
    return y == 0 ? 1 : y;
  }
  if (x >= 0 && x < n) return x;
  if (bc == 1) return x < 0 ? 0 : n - 1;  // Dirichlet: nearest interior column
  const int p = bc == 2 ? n - 1 : n;      // periodic (superposed: period n - 1)
  return ((x % p) + p) % p;
}

// per padded column: the segment sums of its source column added in
// ascending segment order, then the clipped ratios
__global__ void __launch_bounds__(256) k_dyn_coef(Layout L, int bc0, int bc1, int nseg, const double* __restrict__ Xp,
                                                  double* __restrict__ dyn) {
  const long long c = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const long long ncol = dyn_ncol(L);
  if (c >= ncol) return;
  const int i = (int)(c % (L.ni + 4)) - 2, j = (int)(c / (L.ni + 4)) - 2;
  const int is = dyn_src(i, L.ni, bc0), js = dyn_src(j, L.nj, bc1);
  const long long ncoli = (long long)L.ni * L.nj, col = (long long)js * L.ni + is;
  double s[4] = {0.0, 0.0, 0.0, 0.0};
  for (int g = 0; g < nseg; ++g)
    for (int q = 0; q < 4; ++q) s[q] += Xp[((long long)q * nseg + g) * ncoli + col];
  dyn[c] = s[1] > 0.0 ? fmax(0.0, s[0] / s[1]) : 0.0;
  dyn[ncol + c] = s[3] > 0.0 ? fmax(0.0, s[2] / s[3]) : 0.0;
}

inline unsigned nblk(long long n, int b) { return (unsigned)((n + b - 1) / b); }

template <class QI>
hipError_t run(hipStream_t s, const Layout& L, const Machine& mach, const Wrap& wrap, const int bc[3], const Phys& P,
               const double* M, const QI* Q, double* X, double* dyn) {
  DynArgs a{L, P, wrap, M, X, bc[1] == 3};
  a.nks = bc[2] == 2 ? L.nk - 1 : L.nk;
  a.ntx = (L.ni + DTI - 1) / DTI;
  const int ntiles = a.ntx * ((L.nj + DTJ - 1) / DTJ);
  // (equal chunks: the second size's arguments alone cost the kernel 85 register spills)
  const Schedule sch = segment_schedule(ntiles, a.nks, mach.cus, a.nks, 4, false);
  a.kc = sch.kc;
  a.nch = (a.nks + sch.kc - 1) / sch.kc;
  a.nseg = ntiles * a.nch;
  a.nblocks = sch.nblocks;
  a.nxcd = mach.xcds;
  a.per_xcd = (sch.nblocks + a.nxcd - 1) / a.nxcd;
  k_dyn_fused<QI><<<a.per_xcd * a.nxcd, DNT, 0, s>>>(a, Q);
  k_dyn_coef<<<nblk(dyn_ncol(L), 256), 256, 0, s>>>(L, bc[0], bc[1], a.nch, X, dyn);
  return hipGetLastError();
}

}  // namespace

// (at most one k chunk per plane)
long long dynamic_work_elems(const Layout& L) { return 4LL * L.ni * L.nj * L.nk; }

hipError_t launch_dynamic(hipStream_t s, const Layout& L, const Machine& mach, const Wrap& wrap, const int bc[3], const Phys& P,
                          const double* M, const double* Q, double* work, double* dyn) {
  return run<double>(s, L, mach, wrap, bc, P, M, Q, work, dyn);
}

hipError_t launch_dynamic_f32(hipStream_t s, const Layout& L, const Machine& mach, const Wrap& wrap, const int bc[3], const Phys& P,
                              const double* M, const float* Q, double* work, double* dyn) {
  return run<float>(s, L, mach, wrap, bc, P, M, Q, work, dyn);
}

}  // namespace les
