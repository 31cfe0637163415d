// les_stage.hip -- fused residual + Runge-Kutta stage kernel for gfx950.
//
// One launch evaluates R(Q^(l-1)) at every interior node and writes
// Q^(l) = Q^(0) - alpha_l dt R (Sec. 4, Alg. 2: inviscid flux, artificial
// dissipation, viscous flux, RHS and the stage update of one RK stage,
// fused), plus per-block partial norms of R (first stage) or per-block
// minima of the local CFL bound of the updated state (last stage: the time
// step of the next step is pointwise in Q^{n+1}, so it is reduced while the
// state is in registers instead of by a pass of its own).
//
// Decomposition.  A block of 32 x 16 threads owns the nodes of a 32 x 16
// patch of one k-plane: the 30 x 14 output tile and a one-node halo ring.
// Blocks are persistent (one per CU of the device) and take (k chunk, tile)
// segments round robin in chunk-major order, so the blocks that run together
// on one XCD work on neighbouring tiles at the same planes and read the halo
// lines they share while those are still in the XCD's L2.
// Each thread keeps the k-direction stencil of its own column in
// registers (conserved variables at t-2 .. t+1, primitives at t-1 and t+1,
// the zeta node flux and the partial residual of the plane below), so the
// zeta direction needs no LDS.  The in-plane (xi, eta) stencil works in three
// phases per plane with two barriers:
//   B  fill:  every node of the patch (and a second halo ring along the
//             axes, written by helper threads) stores Q, p, u, v, w, T to LDS;
//   C  node:  every node of the patch computes its velocity and temperature
//             gradient (chain rule through its metrics), the viscous stress
//             with Sutherland and Smagorinsky viscosity, the node fluxes, the
//             Turkel-Vatsa anisotropic spectral radii and the pressure
//             sensors; then the xi part of the residual, whose neighbours are
//             adjacent lanes of the same wave (a tile row is 32 lanes): node
//             fluxes, radii, sensors and the lower face by lane shifts;
//   E  face:  the eta part through LDS, the zeta face from registers, and the
//             residual and stage update of the plane below (stage 1 also
//             accumulates R^2 and max |R| per thread; the block reduces them
//             once, after its last plane).  FP64 evaluates each eta face once:
//             the row below it leaves it in LDS, and the row above adds it in
//             phase C of the next plane, before its residual is finished.
// The LDS Q plane is double-buffered, so E of one plane and B of the next
// need no barrier between them.  (Before: xi through LDS too, one Q plane and
// a third barrier; the 25 KB of the xi arrays hold the second plane now.)
// Memory.  Wave w owns patch rows 2w and 2w+1 (rows 4w .. 4w+3 with the
// 16-wide patch the shape constants also allow).  The ten metric fields of
// those rows are wave-private, so they travel as asynchronous global->LDS
// copies (16 bytes per lane) into per-wave LDS blocks with no barrier (FP32:
// nine terms from an FP32 copy, and J, straight into registers).  The copies
// of the next plane's metrics and the loads of the own column two
// planes ahead are issued one at a time between the sub-steps of C, the
// helper ring of the next plane at its start, Q^(0) of the plane being
// finished at its end.  The block barriers order LDS data only: a full
// __syncthreads would also drain every outstanding global load, store and
// copy of the wave.  All loads of a plane are waited for once, before the
// stage update's stores and on every path, so that no later use of a loaded
// value has to wait for those stores (the counter of outstanding operations
// is in order).  The own-column loads are branch-free (threads past the
// padded box load a clamped node).
// The flow constants are read from the kernel-argument segment where they
// are used, instead of occupying scalar registers across the loop.  Divisions and square roots
// use short Newton-refined sequences (valid for the positive, normal
// arguments met here).  Scheduling fences split phases C and E into short
// regions: without them the scheduler hoists LDS reads of later regions over
// the FP64 work of earlier ones and the live ranges exceed the 256 registers
// of a two-wave-per-SIMD launch.
//
// What bounds it, 256 x 128 x 128 FP64 (258 us a stage, 346 before): 6.3e7
// vector instructions a launch need 123 us of issue at the 2.0 GHz the core
// runs at under this load (2.36 GHz on a block of 32^3), and 1.06 GB between
// L2 and memory 190 us at the rate of a large copy; two waves per SIMD (LDS
// and registers allow no more) overlap the two only in part and wait for a
// third of their cycles, at the two barriers most of all.  Falling priorities
// (wave_priority) keep the two waves of a SIMD together.  At 800 x 500 x 500 the
// traffic between L2 and memory is as near.
//
// Work per thread is independent of the floating-point type T (double for
// the FP64 path, float for the mixed path, which rounds the metric terms of
// its fluxes to float); Q^(0), the stage update, J, the CFL bound's metrics
// and all reductions stay in FP64.  The FP32 path keeps the order of
// operations that its results were first defined by (its rounding is visible
// at 1e-8), the FP64 path works with twice the residual and joins the
// pressure to the normal stresses.
#include <stdlib.h>

#include "les_stage.hpp"
#include "les_launch.hpp"

namespace les {

namespace {

#ifndef LES_STAGE_BX
#define LES_STAGE_BX 32
#endif
#ifndef LES_STAGE_BY
#define LES_STAGE_BY 16
#endif
constexpr int BX = LES_STAGE_BX, BY = LES_STAGE_BY, NT = BX * BY;  // patch (threads)
constexpr int TX = BX - 2, TY = BY - 2;        // output tile
constexpr int EX = BX + 2, EY = BY + 2;        // patch + axis halo (LDS planes)
constexpr int NH2 = 2 * TY + 2 * TX;           // second-ring helper nodes
constexpr int NW = NT / 64;                    // waves per block
constexpr int RPW = 64 / BX;                   // patch rows per wave
constexpr int LPR = BX / 2;                    // lanes per row of a 16-byte row copy
constexpr int BPC = 512 / NT;                  // resident blocks per CU (two waves per SIMD)
static_assert(BX == 16 || BX == 32, "a wave covers whole patch rows");
static_assert(BY % RPW == 0 && NT % 64 == 0 && NH2 <= NT && BPC >= 1, "tile shape");

// (what a segment's start needs first, so that it comes with few cache lines)
struct KArgs {
  Layout L;
  Schedule sch;         // (chunk, tile) segments
  int ntx, nty;         // tiles in i, j
  int per_xcd;          // blocks per XCD in the remapped order
  int nxcd;             // XCDs of the device
  Wrap wrap;            // periodic ghosts read at their source
  const double* M;
  const float* M32;     // mixed: the nine metric terms in FP32
  Phys P;
  const double* f;
  const double* dyn;    // per-column dynamic SGS coefficients (P.sgs == 2)
  int axis;             // j = 0 is the polar axis
  int i_f;
};

// Two Q planes, written at B of alternate planes: the only LDS values that E
// reads at other threads' nodes and B of the next plane would overwrite.
template <class T>
struct Smem {
  T q[2][5][EY][EX];
  T p[EY][EX];
  T u[EY][EX], v[EY][EX], w[EY][EX], tem[EY][EX];
  T hy[5][BY][TX];  // eta node flux, patch columns 1..TX
  T ly[BY][TX], ny[BY][TX];
  T dy[sizeof(T) == 8 ? 5 : 0][BY - 1][TX];  // FP64: dissipation of the eta face above patch rows 0..BY-2
};

template <class T, class QI>
__device__ __forceinline__ void load_q(const QI* __restrict__ Q, long long fe, unsigned off, T q[5]) {
#pragma unroll
  for (int c = 0; c < 5; ++c) q[c] = (T)ldo(Q + c * fe, off);
}

// Dissipation of the face between nodes a and b = a + 1 along a line
// (am = a - 1, bp = b + 1), given the node spectral radii and sensors: the
// bracket X = eps2 dQ - eps4 d3Q; returns the radius factor, so that the flux
// (FP64: twice the flux, see kTwice) is the factor times X.
template <class T>
__device__ __forceinline__ T face_bracket(const Phys& P, T La, T Lb, T na, T nb, const T qam[5], const T qa[5],
                                          const T qb[5], const T qbp[5], T X[5]) {
  const T e2 = T(P.k2) * tmax(na, nb);
  const T e4 = tmax(T(0), T(P.k4) - e2);
#pragma unroll
  for (int c = 0; c < 5; ++c) {
    const T d1 = qb[c] - qa[c];
    const T d3 = qbp[c] - T(3) * qb[c] + T(3) * qa[c] - qam[c];
    X[c] = e2 * d1 - e4 * d3;
  }
  return sizeof(T) == 8 ? La + Lb : T(0.5) * (La + Lb);
}
template <class T>
__device__ __forceinline__ void face_diss(const Phys& P, T La, T Lb, T na, T nb, const T qam[5], const T qa[5],
                                          const T qb[5], const T qbp[5], T D[5]) {
  const T Lf = face_bracket(P, La, Lb, na, nb, qam, qa, qb, qbp, D);
#pragma unroll
  for (int c = 0; c < 5; ++c) D[c] *= Lf;
}

// Per-wave reduction of the threads' R^2 sums and |R| maxima into the ten
// doubles at red (all lanes of the wave must call it; lane 0 writes).
__device__ __forceinline__ void norm_wave(const double s2[5], const double sm[5], double* red, int lane) {
#pragma unroll
  for (int c = 0; c < 5; ++c) {
    const double sum = wave_sum(s2[c]);
    const double mx = wave_max(sm[c]);
    if (lane == 0) {
      red[c] = sum;
      red[5 + c] = mx;
    }
  }
}

// Per-wave row staging.  Wave w owns patch rows RPW w .. RPW w + RPW - 1 (the
// rows of its own threads: two rows of 32 or four rows of 16), so the
// metrics and Q^(0) of those rows can be copied into a wave-private LDS block
// with no barrier.  One asynchronous global->LDS copy moves 16 bytes (two
// doubles) per lane: lanes 0-31 the 64 nodes of field f (row after row),
// lanes 32-63 the same for field f+1; they land contiguously at [f][r][col]
// of the block.  src is the lane's byte address for field (lane >> 5); fstep2
// is two fields in bytes.
template <int NF>
__device__ __forceinline__ void dma_rows(const char* src, long long fstep2, double* dst) {
  static_assert(NF % 2 == 0, "two fields per copy");
#pragma unroll
  for (int q = 0; q < NF / 2; ++q) copy_to_lds(src + q * fstep2, dst + q * 128);
}

// Optional paths of the stage kernel (template bit mask EXT)
constexpr int kExtSgs = 1;   // dynamic closure coefficients, isotropic SGS stress
constexpr int kExtAxis = 2;  // the O-grid's polar axis at j = 0
// an anisotropy exponent other than 1/2: the six inlined pow calls, kept out
// of the other instantiations, cost them 1,000 static FP64 instructions and
// 84 spilled scalar registers per plane (345 -> 334 us per FP64 stage at 256 x
// 128 x 128 without them)
constexpr int kExtPow = 4;
// mixed path, a context without the FP32 copy of the metric terms: they are
// taken from the FP64 fields and converted (the same values)
constexpr int kExtM64 = 8;

template <class T, class QI, bool NORM, bool CFL, int EXT>
__global__ void __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(2, 2))) k_stage(KArgs a, const QI* __restrict__ Qin, const double* Q0, double* Qout,
                                              float* Qsh, const double* __restrict__ dtp, double dt_host,
                                              double alpha, double* __restrict__ part, double* __restrict__ cpart) {
  // FP64: phases C and E work with twice the residual, so that the halves of
  // the central differences and face means are applied once, through J / 2
  constexpr bool kTwice = sizeof(T) == 8;
  constexpr T kHalf = kTwice ? T(1) : T(0.5);
  __shared__ Smem<T> s;
  // FP32 without the CFL bound takes its metric terms from an FP32 copy (the
  // values it would convert to; J stays FP64), straight into registers: 48
  // bytes a node and stage less, of about 230 with halos.  Stage on 256 x 128
  // x 128 227 to 210 us, 400 x 250 x 250 1160 to 1083.  (A context holds the
  // copy where memory allows; kExtM64 without it.)
  constexpr bool kM32 = sizeof(T) == 4 && !CFL && !(EXT & kExtM64);
  __shared__ double mbw[kM32 ? 1 : NW][10][RPW][BX];  // per-wave metrics rows of the current plane
  __shared__ double red_s[NW][10];         // block reductions
  static_assert(sizeof(Smem<T>) + sizeof(mbw) + sizeof(red_s) <= 163840 / BPC, "LDS of BPC blocks per CU");
  const Layout& L = a.L;
  // a (the first kernel argument) sits at the start of the kernel-argument
  // segment; the loop re-reads the flow constants through this pointer
  // (scalar loads) where they are used, so that they do not hold scalar
  // registers across the loop
  typedef __attribute__((address_space(4))) const KArgs CKArgs;
  CKArgs* const ka = (CKArgs*)__builtin_amdgcn_kernarg_segment_ptr();
  const long long fe = L.fe;

  // XCD-aware order: consecutive virtual blocks land on one XCD.
  const int hb = blockIdx.x;
  const int v = (hb % a.nxcd) * a.per_xcd + hb / a.nxcd;
  if (v >= a.sch.nblocks) return;
  const int tid = threadIdx.x;
  const int tx = tid % BX, ty = tid / BX;
  const int ex = tx + 1, ey = ty + 1;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int fsel = lane >> 5, rsel = (lane / LPR) % RPW, pr = lane % LPR;  // row-copy lane geometry
  const int ty1 = ty % RPW;                                                // own row within the wave's rows
  const bool xh = (tx == 0 || tx == BX - 1), yh = (ty == 0 || ty == BY - 1);
  const unsigned sk = (unsigned)L.sk;
  const double adt = alpha * (dtp ? dtp[0] : dt_host);

  // second halo ring along the axes: helper thread h < NH2 owns LDS slot (hy2, hx2)
  int hx2 = 0, hy2 = 0;
  if (tid < NH2) {
    const int h = tid;
    if (h < TY) { hx2 = 0; hy2 = 2 + h; }
    else if (h < 2 * TY) { hx2 = EX - 1; hy2 = 2 + h - TY; }
    else if (h < 2 * TY + TX) { hy2 = 0; hx2 = 2 + h - 2 * TY; }
    else { hy2 = EY - 1; hx2 = 2 + h - 2 * TY - TX; }
  }

  auto prims = [&](const Phys& P, const T q[5], T uu[4], T& pp) {
    T u, vv, w, p, tem;
    prim_from_q_fast(q[0], q[1], q[2], q[3], q[4], P, u, vv, w, p, tem);
    uu[0] = u; uu[1] = vv; uu[2] = w; uu[3] = tem;
    pp = p;
  };

  // residual norms: per-thread running sums of R^2 and maxima of |R| over
  // all planes of the block (NORM only), reduced once at the end
  double n2[5] = {0, 0, 0, 0, 0}, nm[5] = {0, 0, 0, 0, 0};
  // CFL only (the last stage): running minimum of the local CFL bound of the
  // updated state Q^(l) = Q^{n+1} over the block's nodes
  double cmin = INFINITY;
  int qbuf = 0;  // LDS Q plane written at the next B (alternates every plane)
  for (int wq = v; wq < a.sch.nseg; wq += a.sch.nblocks) {
    // ---- one segment: planes [kb, ke) of one tile ----
    // segments are ordered k chunk by k chunk (kc planes; the last chunk may
    // be shorter) and tile by tile within a chunk, and the blocks take them
    // round robin: the blocks that run at the same time on one XCD work on
    // neighbouring tiles at the same planes, so the halo lines they share are
    // read while they are still in that XCD's L2
    const Segment g = segment_at(a.sch, a.ntx * a.nty, L.nk, wq);
    const int tile = g.tile, kb = g.k0, ke = g.k1;
    // segment base: plane kb - 2, the first the segment reads.  Per-thread
    // element offsets are taken from there, so they stay below 2^29 for any
    // segment that segment_kmax allows; field and segment bases are 64-bit.
    const int kr = kb - kStageSpan.below;
    const long long sb = (long long)kr * L.sk;
    const QI* const Qs = Qin + sb;
    const int tix = tile % a.ntx, tiy = tile / a.ntx;
    const int i0 = tix * TX, j0 = tiy * TY;
    const int i = i0 - 1 + tx, j = j0 - 1 + ty;
    const bool load_ok = i <= L.ni + 1 && j <= L.nj + 1;
    const bool node_ok = load_ok && i <= L.ni && j <= L.nj && !(xh && yh);
    const bool need_y = node_ok && !xh;  // eta node flux / sensor needed here
    const bool out_ok = !xh && !yh && i < L.ni && j < L.nj;
    const bool wave_in = __builtin_amdgcn_ballot_w64(load_ok) != 0;  // some row of the wave is in the padded box
    const bool fy_ok = !xh && ty < BY - 1 && i < L.ni && j < L.nj;  // eta face (j, j + 1) of a tile column
    const bool fx_ok = !yh && tx < BX - 1 && i < L.ni && j < L.nj;  // xi face (i, i + 1) of a tile row
    const int hi = i0 - 2 + hx2, hj = j0 - 2 + hy2;
    const bool h_ok = tid < NH2 && hi <= L.ni + 1 && hj <= L.nj + 1;
    // element offset of node (i, j, kr) from the segment base
    const unsigned col = (unsigned)((long long)i + (long long)j * L.sj + L.o);
    // columns of Q.  Own-column loads use the node clamped into the padded
    // box, so that they and their uses need no branch (threads past the box
    // load, and never publish, a copy of the box's edge node)
    const unsigned qcol = wrap_column(L, a.wrap, min(i, L.ni + 1), min(j, L.nj + 1));
    const unsigned hcol = wrap_column(L, a.wrap, min(hi, L.ni + 1), min(hj, L.nj + 1));
    auto load_plane = [&](int k, T q[5]) {
      const PlaneRef p = wrap_plane(L, a.wrap, k);
      load_q<T>(Qin + p.base, fe, wrap_offset(qcol, p), q);
    };

    // ---- column queues (own node) ----
    T qw[5], qa[5], qn[5];  // Q at t (written at B), t+1 and t+2 (prefetch)
    T qm1[5], qm2[5];       // Q at t-1, t-2
    T um1[4], up1[4];       // u, v, w, T at t-1; at t+1 (at B: plane t)
    T pm1 = 0, pp1 = 0;
    T hq[5];                // helper node, next plane
    T hz_prev[5], racc[5];  // zeta node flux at t-1; partial residual of t-1
    T lz_prev = 0, nz_prev = 0;
    double J_prev = 0.0, m_prev[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int c = 0; c < 5; ++c) qw[c] = qa[c] = qn[c] = qm1[c] = qm2[c] = hq[c] = hz_prev[c] = racc[c] = T(0);
#pragma unroll
    for (int c = 0; c < 4; ++c) um1[c] = up1[c] = T(0);

    // (the empty asm hides the pointer's origin, so the loads below are not
    // hoisted out of the loop)
    CKArgs* kp4 = ka;
    asm volatile("" : "+s"(kp4));
    const KArgs* kp = (const KArgs*)kp4;
    // prime for t = kb-1: metrics(kb-1) -> LDS; Q(kb-2), Q(kb-1) of the own
    // column; helper Q(kb-1)
    //
    // element offset (plane 0) of this lane's row copy: field fsel, row
    // RPW wave + rsel, column pair starting at i0-1+2pr (16-byte aligned);
    // pairs past i = ni (ragged last tile) re-read the last pair within the row
    int icp = i0 - 1 + 2 * pr;
    if (icp > L.ni) icp = L.ni - ((LEAD + L.ni) & 1);
    const int jcp = min(j0 - 1 + RPW * wave + rsel, L.nj);
    const long long lane_el = (long long)fsel * fe + L.o + icp + (long long)jcp * L.sj;
    const long long fstep2 = 2 * fe * (long long)sizeof(double);
    const unsigned mcol = (unsigned)((long long)min(i, L.ni + 1) + (long long)min(j, L.nj + 1) * L.sj + L.o);
    float m32[9];  // metric terms and J of the next plane (in flight; kM32)
    double j32 = 0.0;
    if (kM32) {
#pragma unroll
      for (int c = 0; c < 9; ++c) m32[c] = ldo(kp->M32 + sb + c * fe, mcol + sk);
      j32 = ldo(kp->M + sb + 9 * fe, mcol + sk);
    } else {
      dma_rows<10>((const char*)(kp->M + lane_el + (long long)(kb - 1) * L.sk), fstep2, &mbw[wave][0][0][0]);
    }
    load_plane(kb - 2, qm1);
    load_plane(kb - 1, qw);
    load_plane(kb, qa);
    prims(kp->P, qm1, um1, pm1);
    prims(kp->P, qw, up1, pp1);  // plane kb-1, written at the first B
    if (h_ok) {
      const PlaneRef p = wrap_plane(L, a.wrap, kb - 1);
      load_q<T>(Qin + p.base, fe, wrap_offset(hcol, p), hq);
    }
    wait_vm<0>();  // the first metric rows (later ones are waited for before each stage update)

    for (int t = kb - 1; t <= ke; ++t) {
      const unsigned nt = col + (unsigned)(t - kr) * sk;
      CKArgs* kq4 = ka;
      asm volatile("" : "+s"(kq4));
      const KArgs* kq = (const KArgs*)kq4;
      const Phys& P = kq->P;
      // the first and last plane of a segment only provide zeta quantities
      // of the tile columns; their in-plane fluxes and residual are not needed
      const bool inner = t >= kb && t < ke;
      T(*const sq)[EY][EX] = s.q[qbuf];
      qbuf ^= 1;

      // ---- B: fill LDS plane t ----
      if (load_ok) {
#pragma unroll
        for (int c = 0; c < 5; ++c) sq[c][ey][ex] = qw[c];
        s.p[ey][ex] = pp1;
        s.u[ey][ex] = up1[0]; s.v[ey][ex] = up1[1]; s.w[ey][ex] = up1[2]; s.tem[ey][ex] = up1[3];
      }
      if (h_ok) {
        T hu[4], hp;
        prims(P, hq, hu, hp);
#pragma unroll
        for (int c = 0; c < 5; ++c) sq[c][hy2][hx2] = hq[c];
        s.p[hy2][hx2] = hp;
        s.u[hy2][hx2] = hu[0]; s.v[hy2][hx2] = hu[1]; s.w[hy2][hx2] = hu[2]; s.tem[hy2][hx2] = hu[3];
      }
      lds_barrier();

      // ---- C: node work at plane t ----
      // the face between the axis and j = 1 takes the cross-axis value by
      // linear extrapolation (no five-point stencil across the axis): the
      // halo row below the axis holds 2 Q(0) - Q(1) for the dissipation of
      // phase E (its pressure, velocity and temperature keep the cross-axis
      // values for the sensor and the gradients; the row's own fluxes serve
      // only the axis, whose residual is not formed)
      if ((EXT & kExtAxis) && j == -1 && load_ok && kq->axis) {
#pragma unroll
        for (int c = 0; c < 5; ++c) sq[c][ey][ex] = T(2) * sq[c][ey + 1][ex] - sq[c][ey + 2][ex];
      }
      prims(P, qa, up1, pp1);  // plane t+1 of the own column
      T hz[5] = {0, 0, 0, 0, 0};
      T lz = 0, nz = 0;
      double Jn = 0.0, m_cur[9];
      T mt[9];
      {
        double md[9];
        if (kM32) {
          Jn = j32;
#pragma unroll
          for (int c = 0; c < 9; ++c) mt[c] = (T)m32[c];
        } else {
          read_metric_rows(&mbw[wave][0][ty1][tx], md, Jn);
#pragma unroll
          for (int c = 0; c < 9; ++c) mt[c] = (T)md[c];
        }
        if (CFL && sizeof(T) == 4) {
#pragma unroll
          for (int c = 0; c < 9; ++c) m_cur[c] = md[c];
        }
      }
      const unsigned moff = mcol + (unsigned)(t + 1 - kr) * sk;
      const char* const msrc = (const char*)(kq->M + lane_el + (long long)(t + 1) * L.sk);
      double* const mdst = &mbw[wave][0][0][0];
      // Loads for the following planes: the helper ring of t+1, then, after each
      // sub-step q = 1..5, one copy of the wave's metric rows of t+1 and one
      // value of the own column at t+2.  Issued together they fill the memory
      // pipeline's queue and both waves of a SIMD wait to issue; spread over
      // the node work that wait is hidden (256 x 128 x 128: 303 -> 270 us per
      // FP64 stage, 253 -> 239 us mixed).  At t = ke nothing more is needed:
      // FP64 skips the loads; FP32 issues them all the same (planes ke + 1 at
      // most, inside the padded box), because the branches between its
      // sub-steps cost more (247 against 239 us) than the loads.
      // (planes past the block's last are the only wrapped ones here)
      const QI *Q2 = Qs, *Q1 = Qs;
      const int k2 = min(t + 2, ke + 1);
      unsigned qoff2 = (qcol & 0x7fffffffu) + (unsigned)(k2 - kr) * sk;
      unsigned hoff1 = (hcol & 0x7fffffffu) + (unsigned)(t + 1 - kr) * sk;
      if (k2 >= kq->L.nk) {
        const PlaneRef p2 = wrap_plane(kq->L, kq->wrap, k2);
        Q2 = Qin + p2.base;
        qoff2 = wrap_offset(qcol, p2);
        const PlaneRef p1 = wrap_plane(kq->L, kq->wrap, t + 1);
        Q1 = Qin + p1.base;
        hoff1 = wrap_offset(hcol, p1);
      }
      auto load_ahead = [&](int q) {
        if (sizeof(T) == 4 || t < ke) {
          if (q == 0) {
            if (h_ok) load_q<T>(Q1, fe, hoff1, hq);
          } else {
            if (kM32) {
              m32[2 * q - 2] = ldo(kq->M32 + sb + (2 * q - 2) * fe, moff);
              if (q < 5)
                m32[2 * q - 1] = ldo(kq->M32 + sb + (2 * q - 1) * fe, moff);
              else
                j32 = ldo(kq->M + sb + 9 * fe, moff);
            } else {
              copy_to_lds(msrc + (q - 1) * fstep2, mdst + (q - 1) * 128);
            }
            qn[q - 1] = (T)ldo(Q2 + (q - 1) * fe, qoff2);
          }
        }
        // (FP64 only: its phases are bound by the issue rate, and gain 2 to 3 %
        // - 256 x 128 x 128 5.43 to 5.33 ms a call, 191 x 97 x 75 1985 to 1924
        // us; the mixed path, bound by memory, loses 0.4 %)
        if (sizeof(T) == 8) {
          if (q == 0) wave_priority<3>();
          if (q == 2) wave_priority<2>();
          if (q == 3) wave_priority<1>();
          if (q == 5) wave_priority<0>();
        }
        __builtin_amdgcn_sched_barrier(0);
      };
      load_ahead(0);
      T hxf[5] = {0, 0, 0, 0, 0}, lx = 0, nx = 0;  // xi node flux, radius and sensor
      // (every lane of such a wave does the node work: the values of lanes that
      // are no node are never published, and the loads between the sub-steps
      // need the whole wave)
      if (wave_in) {
        const T Jh = T(0.5) * (T)Jn;
        T g[4][3];
        {
          // derivatives along xi, eta (LDS) and zeta (registers), chain rule
          const T(*F[4])[EX] = {s.u, s.v, s.w, s.tem};
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            // (the halves of the central differences are in Jh)
            const T dx = F[q][ey][ex + 1] - F[q][ey][ex - 1];
            const T dy = F[q][ey + 1][ex] - F[q][ey - 1][ex];
            const T dz = up1[q] - um1[q];
#pragma unroll
            for (int x = 0; x < 3; ++x) g[q][x] = Jh * (mt[x] * dx + mt[3 + x] * dy + mt[6 + x] * dz);
          }
        }
        load_ahead(1);
        const T s11 = g[0][0], s22 = g[1][1], s33 = g[2][2];
        // off-diagonal strains (FP64: twice)
        const T w12 = kHalf * (g[0][1] + g[1][0]), w13 = kHalf * (g[0][2] + g[2][0]), w23 = kHalf * (g[1][2] + g[2][1]);
        const T skk3 = (s11 + s22 + s33) * T(1.0 / 3.0);
        const T rho = sq[0][ey][ex];
        const T u = s.u[ey][ex], vv = s.v[ey][ex], w = s.w[ey][ex];
        const T tn = s.tem[ey][ex];
        const T mu = sutherland_fast(tn, P);
        T mus = T(0), kaps = T(0), pis = T(0);
        if (P.sgs) {
          const T ss = s11 * s11 + s22 * s22 + s33 * s33 + T(kTwice ? 0.5 : 2.0) * (w12 * w12 + w13 * w13 + w23 * w23);
          T d2 = (T)icbrt(Jn);  // (1/J)^(1/3)
          d2 *= d2;
          const T rd = rho * d2 * sqrt_nn(T(2) * ss);
          if (!(EXT & kExtSgs) || P.sgs == 1) {
            mus = T(P.Cs2) * rd;
            kaps = mus * T(P.Cp_over_Prsgs);
          } else {  // dynamic coefficients of this column
            const long long cc = dyn_col(kq->L, min(i, L.ni + 1), min(j, L.nj + 1));
            mus = T(kq->dyn[cc]) * rd;
            kaps = T(P.Cp) * T(kq->dyn[dyn_ncol(kq->L) + cc]) * rd;
          }
          // isotropic SGS stress: sigma_kk / 3, added to the pressure of the fluxes
          if ((EXT & kExtSgs) && P.CI43 != 0.0) pis = T(P.CI43) * rho * d2 * ss;
        }
        const T mt1 = mu + mus, mt2 = T(2) * mt1;
        const T t11 = mt2 * (s11 - skk3), t22 = mt2 * (s22 - skk3), t33 = mt2 * (s33 - skk3);
        const T mtw = kTwice ? mt1 : mt2;
        const T t12 = mtw * w12, t13 = mtw * w13, t23 = mtw * w23;
        const T kap = mu * T(P.Cp_over_Pr) + kaps;
        const T th0 = u * t11 + vv * t12 + w * t13 + kap * g[3][0];
        const T th1 = u * t12 + vv * t22 + w * t23 + kap * g[3][1];
        const T th2 = u * t13 + vv * t23 + w * t33 + kap * g[3][2];
        load_ahead(2);
        const T p = s.p[ey][ex];
        const T pe = (EXT & kExtSgs) ? p + pis : p;  // pressure of the fluxes
        const T c2 = T(P.gamma_R) * tn;  // c^2 = gamma p / rho = gamma R T
        // spectral radii of the three directions and their square roots
        T lam[3], U[3], sl[3];
#pragma unroll
        for (int e = 0; e < 3; ++e) {
          const T mx = mt[3 * e], my = mt[3 * e + 1], mz = mt[3 * e + 2];
          U[e] = mx * u + my * vv + mz * w;
          lam[e] = fabs(U[e]) + sqrt_pos(c2 * (mx * mx + my * my + mz * mz));
          sl[e] = sqrt_pos(lam[e]);
        }
        // anisotropic scaling Lam_d = lam_d [1 + sum_e (lam_e / lam_d)^alpha]
        auto aniso_n = [&](int d, int e, int f) -> T {
          if (!(EXT & kExtPow) || P.alpha_half) return lam[d] + sl[d] * (sl[e] + sl[f]);
          return aniso(lam[d], lam[e], lam[f], P);
        };
        const T e11 = pe - t11, e22 = pe - t22, e33 = pe - t33;
        auto node_flux = [&](int e, T H[5]) {
          const T mx = mt[3 * e], my = mt[3 * e + 1], mz = mt[3 * e + 2];
          const T Ue = U[e];
          H[0] = rho * Ue;
          if (kTwice) {  // pressure joined to the normal stresses: six operations fewer per direction
            H[1] = sq[1][ey][ex] * Ue + mx * e11 - my * t12 - mz * t13;
            H[2] = sq[2][ey][ex] * Ue + my * e22 - mx * t12 - mz * t23;
            H[3] = sq[3][ey][ex] * Ue + mz * e33 - mx * t13 - my * t23;
          } else {
            H[1] = sq[1][ey][ex] * Ue + mx * pe - (mx * t11 + my * t12 + mz * t13);
            H[2] = sq[2][ey][ex] * Ue + my * pe - (mx * t12 + my * t22 + mz * t23);
            H[3] = sq[3][ey][ex] * Ue + mz * pe - (mx * t13 + my * t23 + mz * t33);
          }
          H[4] = (sq[4][ey][ex] + pe) * Ue - (mx * th0 + my * th1 + mz * th2);
        };
        load_ahead(3);
        if (inner) {
          node_flux(0, hxf);
          lx = aniso_n(0, 1, 2);
          const T pa = s.p[ey][ex + 1], pb = s.p[ey][ex - 1];
          nx = fabs(pa - T(2) * p + pb) * rcp_nr(pa + T(2) * p + pb);
        }
        load_ahead(4);
        if (need_y && inner) {
          T H[5];
          node_flux(1, H);
          // on the polar axis eta/J = 0: the eta node flux and radius take
          // their limit 0 (J is infinite there)
          const bool on_axis = (EXT & kExtAxis) && kq->axis && j == 0;
#pragma unroll
          for (int q = 0; q < 5; ++q) s.hy[q][ty][tx - 1] = on_axis ? T(0) : H[q];
          s.ly[ty][tx - 1] = on_axis ? T(0) : aniso_n(1, 2, 0);
          const T pa = s.p[ey + 1][ex], pb = s.p[ey - 1][ex];
          s.ny[ty][tx - 1] = fabs(pa - T(2) * p + pb) * rcp_nr(pa + T(2) * p + pb);
        }
        load_ahead(5);
        {
          node_flux(2, hz);
          lz = aniso_n(2, 0, 1);
          nz = fabs(pp1 - T(2) * p + pm1) * rcp_nr(pp1 + T(2) * p + pm1);
        }
      }
      if (kTwice && t > kb && out_ok) {  // plane t-1's eta face below this row
#pragma unroll
        for (int c = 0; c < 5; ++c) racc[c] += s.dy[c][ty - 1][tx - 1];
      }
      // xi direction of the residual: a tile row is 32 consecutive lanes of one
      // wave, so the neighbours' node fluxes, radii and sensors and the face
      // on the lower side come from the adjacent lanes
      T r[5] = {0, 0, 0, 0, 0}, rd[5] = {0, 0, 0, 0, 0};  // FP64: r; FP32: flux difference r, dissipation rd
      if (inner) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < 5; ++q) r[q] = kHalf * (lane_next(hxf[q]) - lane_prev(hxf[q]));
        const T lxn = lane_next(lx), nxn = lane_next(nx);
        T X[5] = {0, 0, 0, 0, 0}, Lf = 0;
        if (fx_ok) {
          T q_b[5], q_c[5], q_d[5], q_e[5];
#pragma unroll
          for (int c = 0; c < 5; ++c) {
            q_b[c] = sq[c][ey][ex - 1]; q_c[c] = sq[c][ey][ex];
            q_d[c] = sq[c][ey][ex + 1]; q_e[c] = sq[c][ey][ex + 2];
          }
          Lf = face_bracket(P, lx, lxn, nx, nxn, q_b, q_c, q_d, q_e, X);
        }
#pragma unroll
        for (int c = 0; c < 5; ++c) {
          const T D = Lf * X[c], Dm = lane_prev(D);
          if (kTwice)
            r[c] -= D - Dm;
          else
            rd[c] = fma(Lf, X[c], -Dm);
        }
      }
      double q0v[5] = {0, 0, 0, 0, 0};
      if (t > kb && out_ok && Q0) {
#pragma unroll
        for (int c = 0; c < 5; ++c) q0v[c] = ldo(Q0 + sb + c * fe, nt - sk);
      }
      __builtin_amdgcn_sched_barrier(0);
      lds_barrier();

      // ---- E: residual (tile nodes) ----
      if (sizeof(T) == 8) wave_priority<3>();
      if (kTwice && inner && fy_ok) {
        // FP64: the eta face above this row, subtracted from this row's
        // residual and left in LDS for the row above, which adds it in phase C
        // of the next plane
        const int cx = tx - 1;
        T q_b[5], q_c[5], q_d[5], q_e[5], D1[5];
#pragma unroll
        for (int c = 0; c < 5; ++c) {
          q_b[c] = sq[c][ey - 1][ex]; q_c[c] = sq[c][ey][ex];
          q_d[c] = sq[c][ey + 1][ex]; q_e[c] = sq[c][ey + 2][ex];
        }
        face_diss(P, s.ly[ty][cx], s.ly[ty + 1][cx], s.ny[ty][cx], s.ny[ty + 1][cx], q_b, q_c, q_d, q_e, D1);
#pragma unroll
        for (int c = 0; c < 5; ++c) {
          s.dy[c][ty][cx] = D1[c];
          r[c] -= D1[c];
        }
      }
      if (out_ok) {
        const int cx = tx - 1;  // tile-local column
        if (inner) {
          // eta direction: central difference of the node fluxes (FP32: and
          // both dissipation faces, in the order of operations that the
          // mixed path's results are defined by)
#pragma unroll
          for (int q = 0; q < 5; ++q) {
            r[q] += kHalf * (s.hy[q][ty + 1][cx] - s.hy[q][ty - 1][cx]);
            if (!kTwice) r[q] -= rd[q];
          }
          if (!kTwice) {
            T q_a[5], q_b[5], q_c[5], q_d[5], q_e[5], D1[5], D0[5];
#pragma unroll
            for (int c = 0; c < 5; ++c) {
              q_a[c] = sq[c][ey - 2][ex]; q_b[c] = sq[c][ey - 1][ex]; q_c[c] = sq[c][ey][ex];
              q_d[c] = sq[c][ey + 1][ex]; q_e[c] = sq[c][ey + 2][ex];
            }
            face_diss(P, s.ly[ty][cx], s.ly[ty + 1][cx], s.ny[ty][cx], s.ny[ty + 1][cx], q_b, q_c, q_d, q_e, D1);
            face_diss(P, s.ly[ty - 1][cx], s.ly[ty][cx], s.ny[ty - 1][cx], s.ny[ty][cx], q_a, q_b, q_c, q_d, D0);
#pragma unroll
            for (int c = 0; c < 5; ++c) r[c] -= D1[c] - D0[c];
          }
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      // CFL only: the nine metric terms of the node finished in this
      // iteration (plane t-1).  The mixed path keeps them in registers from
      // plane t-1's node work (256 x 128 x 128: 269 us for the last stage,
      // read back 321); the FP64 path has no registers left and reads them
      // back through the caches (they were copied to LDS two planes ago);
      // consumed after the update
      double cm[9];
      if (CFL && sizeof(T) == 4) {
#pragma unroll
        for (int c = 0; c < 9; ++c) {
          cm[c] = m_prev[c];
          m_prev[c] = m_cur[c];
        }
      } else if (CFL) {
        const unsigned n = (out_ok && t > kb) ? nt - sk : (unsigned)L.o;
#pragma unroll
        for (int c = 0; c < 9; ++c) cm[c] = ldo(kq->M + sb + c * fe, n);
      }
      if (sizeof(T) == 8) wave_priority<2>();
      // zeta face t - 1/2 between plane t-1 and plane t; it completes the
      // residual of plane t-1 (rs) and opens that of plane t (racc)
      T rs[5] = {0, 0, 0, 0, 0};
      if (t >= kb) {
        T qc[5], D[5];
#pragma unroll
        for (int c = 0; c < 5; ++c) qc[c] = sq[c][ey][ex];
        face_diss(P, lz_prev, lz, nz_prev, nz, qm2, qm1, qc, qa, D);
#pragma unroll
        for (int c = 0; c < 5; ++c) {
          const T fz = kHalf * (hz_prev[c] + hz[c]) - D[c];
          rs[c] = racc[c] + fz;
          racc[c] = r[c] - fz;
        }
      } else {
#pragma unroll
        for (int c = 0; c < 5; ++c) racc[c] = r[c];
      }
      if (sizeof(T) == 8) wave_priority<1>();
      const double J_fin = J_prev;
#pragma unroll
      for (int c = 0; c < 5; ++c) hz_prev[c] = hz[c];
      lz_prev = lz;
      nz_prev = nz;
      J_prev = Jn;
      // ---- shift the column queues (plane t values from LDS), before the
      // stores: the shift takes the column loads of this plane, and a wait
      // for them after the stores would wait for the stores too ----
#pragma unroll
      for (int c = 0; c < 5; ++c) {
        qm2[c] = qm1[c];
        qm1[c] = sq[c][ey][ex];
        qw[c] = qa[c];
        qa[c] = qn[c];
      }
      um1[0] = s.u[ey][ex]; um1[1] = s.v[ey][ex]; um1[2] = s.w[ey][ex]; um1[3] = s.tem[ey][ex];
      pm1 = s.p[ey][ex];
      __builtin_amdgcn_sched_barrier(0);
      wait_vm<0>();  // Q^(0); on every path, so that nothing issued before the stores is waited for after them
      if (t > kb && out_ok) {
        // stage update of plane t-1
        const int k = t - 1;
        const unsigned n = nt - sk;
        double qnv[5], Rv[5];
        const double Jr = kTwice ? 0.5 * J_fin : J_fin;
        const bool on_axis = (EXT & kExtAxis) && kq->axis && j == 0;  // advanced by the centerline condition
#pragma unroll
        for (int c = 0; c < 5; ++c) Rv[c] = Jr * (double)rs[c];
        if (kq->f && i == kq->i_f) {
#pragma unroll
          for (int c = 0; c < 5; ++c) Rv[c] -= kq->f[((long long)c * kq->L.nk + k) * kq->L.nj + j];
        }
#pragma unroll
        for (int c = 0; c < 5; ++c) {
          const double R = on_axis ? 0.0 : Rv[c];
          const double qu = q0v[c] - adt * R;
          qnv[c] = qu;
          if (sizeof(T) == 8 || Qout) sto(Qout + sb + c * fe, n, qu);
          if (sizeof(T) == 4 && Qsh) sto(Qsh + sb + c * fe, n, (float)qu);
          if (NORM) {
            n2[c] += R * R;
            const double a = fabs(R);
            nm[c] = (a > nm[c] || a != a) ? a : nm[c];  // NaN wins so that it is reported
          }
        }
        if (CFL && !on_axis) cmin = min_nan(cmin, cfl_local(qnv[0], qnv[1], qnv[2], qnv[3], qnv[4], J_fin, cm, kq->P));
      }
    }
  }

  // ---- block partial norms ----
  if (NORM) {
    norm_wave(n2, nm, red_s[wave], lane);
    __syncthreads();
    if (tid < 10) {
      const double* red = &red_s[0][0];
      double r = red[tid];
      for (int w = 1; w < NW; ++w) {
        const double o = red[w * 10 + tid];
        r = tid < 5 ? r + o : ((o > r || o != o) ? o : r);
      }
      part[(long long)v * 10 + tid] = r;
    }
  }
  // ---- block partial of the CFL bound (CFL only) ----
  if (CFL) {
    const double m = wave_min(cmin);
    double* red = &red_s[0][0];
    if (lane == 0) red[wave] = m;
    __syncthreads();
    if (tid == 0) {
      double r = red[0];
      for (int w = 1; w < NW; ++w) r = min_nan(r, red[w]);
      cpart[v] = r;
    }
  }
}

}  // namespace

int stage_kmax(const Layout& L) { return segment_kmax(L, kStageSpan); }

namespace {

// Stage kernel configuration for a layout and a schedule.
struct Config {
  int ntx, nty, grid, per_xcd;
};

Config config(const Layout& L, const Schedule& sch, int nxcd) {
  Config c;
  c.ntx = (L.ni + TX - 1) / TX;
  c.nty = (L.nj + TY - 1) / TY;
  // hardware block b runs on XCD b mod nxcd: virtual block (b mod nxcd)
  // per_xcd + b / nxcd, so consecutive virtual blocks share an XCD
  c.per_xcd = (sch.nblocks + nxcd - 1) / nxcd;
  c.grid = c.per_xcd * nxcd;
  return c;
}

template <class T, class QI, int EXT>
hipError_t launch_x(hipStream_t st, const Config& c, const KArgs& a, const QI* Qin, const double* Q0, double* Qout,
                    float* Qsh, const double* dtp, double dt, double alpha, double* part, double* cpart) {
  constexpr int M64 = sizeof(T) == 4 ? EXT | kExtM64 : EXT;
  if (cpart)
    k_stage<T, QI, false, true, EXT><<<c.grid, NT, 0, st>>>(a, Qin, Q0, Qout, Qsh, dtp, dt, alpha, part, cpart);
  else if (part && a.M32)
    k_stage<T, QI, true, false, EXT><<<c.grid, NT, 0, st>>>(a, Qin, Q0, Qout, Qsh, dtp, dt, alpha, part, cpart);
  else if (part)
    k_stage<T, QI, true, false, M64><<<c.grid, NT, 0, st>>>(a, Qin, Q0, Qout, Qsh, dtp, dt, alpha, part, cpart);
  else if (a.M32)
    k_stage<T, QI, false, false, EXT><<<c.grid, NT, 0, st>>>(a, Qin, Q0, Qout, Qsh, dtp, dt, alpha, part, cpart);
  else
    k_stage<T, QI, false, false, M64><<<c.grid, NT, 0, st>>>(a, Qin, Q0, Qout, Qsh, dtp, dt, alpha, part, cpart);
  return hipGetLastError();
}

template <class T, class QI>
hipError_t launch(hipStream_t st, const StageArgs& sa, const QI* Qin, const double* Q0, double* Qout, float* Qsh,
                  const double* dtp, double dt, double alpha, double* part, double* cpart) {
  if (part && cpart) return hipErrorInvalidValue;  // norms belong to stage 1, the CFL bound to stage 5
  const Config c = config(sa.L, sa.sch, sa.mach.xcds);
  KArgs a{sa.L, sa.sch, c.ntx, c.nty, c.per_xcd, sa.mach.xcds, sa.wrap, sa.M, sa.M32, sa.P, sa.f, sa.dyn, sa.axis, sa.i_f};
  // the optional SGS models (dynamic closure, isotropic SGS stress) and the
  // polar axis run in instantiations of their own, so that each path keeps
  // only the registers it needs
  const int x = !sa.P.alpha_half ? kExtPow | kExtSgs | kExtAxis
                                 : ((sa.P.sgs == 2 || sa.P.CI43 != 0.0) ? kExtSgs : 0) | (sa.axis ? kExtAxis : 0);
  if ((x & kExtSgs) && sa.P.sgs == 2 && !sa.dyn) return hipErrorInvalidValue;
  switch (x) {
    case 0: return launch_x<T, QI, 0>(st, c, a, Qin, Q0, Qout, Qsh, dtp, dt, alpha, part, cpart);
    case kExtSgs: return launch_x<T, QI, kExtSgs>(st, c, a, Qin, Q0, Qout, Qsh, dtp, dt, alpha, part, cpart);
    case kExtAxis: return launch_x<T, QI, kExtAxis>(st, c, a, Qin, Q0, Qout, Qsh, dtp, dt, alpha, part, cpart);
    case kExtSgs | kExtAxis:
      return launch_x<T, QI, kExtSgs | kExtAxis>(st, c, a, Qin, Q0, Qout, Qsh, dtp, dt, alpha, part, cpart);
    default:
      return launch_x<T, QI, kExtPow | kExtSgs | kExtAxis>(st, c, a, Qin, Q0, Qout, Qsh, dtp, dt, alpha, part, cpart);
  }
}

}  // namespace

Schedule segment_schedule(long long ntiles, int nk, int slots, int kmax, int halo, bool two_sizes) {
  const int start = halo + 1;
  Schedule best;
  long long cost = -1;
  for (int n = (nk + kmax - 1) / kmax; n <= nk; ++n) {
    const int kc = (nk + n - 1) / n;
    if ((nk + kc - 1) / kc != n) continue;  // the same chunks as fewer of them
    const int last = nk - (n - 1) * kc;
    const long long nseg = ntiles * n, nb = nseg < slots ? nseg : slots;
    const long long rounds = (nseg + nb - 1) / nb, full = (ntiles * (n - 1) + nb - 1) / nb;
    const long long c = full * kc + (rounds - full) * last + rounds * start;
    if (cost < 0 || c < cost) {
      cost = c;
      best.kc = kc;
      best.nblocks = (int)nb;
      best.nseg = (int)nseg;
    }
    if (rounds * start > cost) break;  // more chunks only add starts
  }
  // Chunks of two sizes: r full rounds are r slots segments, n a tile and one
  // more for the rest.  Long segments come first, so the slowest block has
  // its share of them, rounded up.  Tiles next to each other with different
  // chunks share fewer halo lines in the L2, so this has to shorten the slowest
  // block by 1/20 to pay.  Steps of 28 blocks of 2e6 to 2.5e7 nodes (between
  // 68 x 304 x 285 and 599 x 173 x 40), two sizes against equal chunks: where the
  // rule takes them, 19 blocks, 0.2 to 9.5 % less time (mixed 0.7 to 11 %);
  // where they would shorten the slowest block by less, 9 blocks, 3 % less to
  // 3 % more, 0.7 % more in the mean (mixed 1 to 4 % less).
  const long long equal = cost;
  for (long long r = (ntiles + slots - 1) / slots; two_sizes && r * start < cost; ++r) {
    const long long n = r * slots / ntiles, more = r * slots - n * ntiles, fewer = ntiles - more;
    if (n >= nk) break;
    const int kl = (int)((nk + n - 1) / n), kc = (int)((nk + n) / (n + 1));
    if (more == 0 || kl == kc || kl > kmax || (nk + kl - 1) / kl != n || (nk + kc - 1) / kc != n + 1) continue;
    const long long lg = (fewer * n + slots - 1) / slots;  // long segments of the slowest block
    const long long c = lg * kl + (r - lg) * kc + r * start;
    if (c >= cost || 20 * c > 19 * equal) continue;
    cost = c;
    best.kc = kc;
    best.kl = kl;
    best.nl = (int)fewer;
    best.nlong = (int)(fewer * n);
    best.nblocks = slots;
    best.nseg = (int)(r * slots);
  }
  return best;
}

// Segments round robin over one persistent block per CU.  (Against contiguous
// ranges of at least 8 tile-planes per block, which could straddle two tiles,
// as used before; FP64 stage: 32^3 52 -> 18 us, 64^3 49 -> 32,
// 128 x 64 x 64 49 -> 45, 256 x 128 x 128 267 -> 262, 400 x 250 x 250
// 1992 -> 1313, O-grid 256 x 128 x 361 784 -> 700, 800 x 500 x 500
// 10.95 -> 10.55 ms; mixed 75 x 61 x 47 45 -> 23 us.)
Schedule stage_schedule(const Layout& L, const Machine& m) {
  const long long ntiles = (long long)((L.ni + TX - 1) / TX) * ((L.nj + TY - 1) / TY);
  if (const char* env = getenv("LES_SEG")) {
    const int seg = atoi(env);
    if (seg > 0) {  // chunks of seg planes, one block per seg tile-planes
      Schedule s;
      s.kc = seg < L.nk ? seg : L.nk;
      if (s.kc > stage_kmax(L)) s.kc = stage_kmax(L);
      const long long nseg = ntiles * ((L.nk + s.kc - 1) / s.kc), nb = (ntiles * L.nk + seg - 1) / seg;
      s.nblocks = (int)(nseg < nb ? nseg : nb);
      s.nseg = (int)nseg;
      return s;
    }
  }
  return segment_schedule(ntiles, L.nk, m.cus * BPC, stage_kmax(L), 2);
}

hipError_t launch_stage_fp64(hipStream_t s, const StageArgs& a, const double* Qin, const double* Q0, double* Qout,
                             const double* dtp, double dt, double alpha, double* part, double* cpart) {
  return launch<double, double>(s, a, Qin, Q0, Qout, nullptr, dtp, dt, alpha, part, cpart);
}

hipError_t launch_stage_mixed(hipStream_t s, const StageArgs& a, const double* Qin64, const float* Qin32,
                              const double* Q0, double* Qout, float* Qsh, const double* dtp, double dt, double alpha,
                              double* part, double* cpart) {
  if (Qin64) return launch<float, double>(s, a, Qin64, Q0, Qout, Qsh, dtp, dt, alpha, part, cpart);
  return launch<float, float>(s, a, Qin32, Q0, Qout, Qsh, dtp, dt, alpha, part, cpart);
}

}  // namespace les
