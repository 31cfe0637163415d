// les_tile.hpp -- building blocks of the tiled gfx950 kernels that march a
// 32 x 16 patch of nodes in k (the stage kernel, the adjoint passes and the
// dynamic closure): segments and their schedule, periodic ghosts read at their
// source, asynchronous row copies, counted waits, LDS-only barriers and lane
// shifts.
#pragma once
#include "les_common.hpp"

namespace les {

// The device's compute-unit and XCD (accelerator complex die) counts: the
// persistent kernels run one block per CU and map consecutive blocks to one
// XCD (each XCD has its own L2).
struct Machine {
  int cus = 256;
  int xcds = 8;
};

// Work of the persistent blocks: (k chunk, tile) segments, taken round robin
// by nblocks blocks.  The first nl tiles have chunks of kl planes, the others
// of kc; the nlong segments of the former come first, each kind chunk by
// chunk and tile by tile within a chunk.
struct Schedule {
  int kc = 0;
  int nblocks = 0;
  int nl = 0, kl = 0, nlong = 0;
  int nseg = 0;
};

// The schedule of nk planes of ntiles tiles on `slots` resident blocks, at
// most kmax planes per segment.  A segment of n planes runs n + halo iterations
// (the planes before and after it that its kernel marches too) and about one
// more for its start, so the time of a launch is that of its slowest block,
// block 0: the sum of n + halo + 1 over its segments.  The number of chunks
// with the smallest sum is taken, the fewest on ties.  With two_sizes, some
// tiles may take one chunk fewer than the others, where no number of equal
// chunks fills the blocks' last round.
Schedule segment_schedule(long long ntiles, int nk, int slots, int kmax, int halo, bool two_sizes = true);

// The tile and planes [k0, k1) of segment x.
struct Segment {
  int tile, ch, k0, k1;
};
__device__ __forceinline__ Segment segment_at(const Schedule& s, int ntiles, int nk, int x) {
  const bool lg = x < s.nlong;
  const int y = lg ? x : x - s.nlong, n = lg ? s.nl : ntiles - s.nl, len = lg ? s.kl : s.kc;
  Segment g;
  g.ch = __builtin_amdgcn_readfirstlane(y / n);
  g.tile = __builtin_amdgcn_readfirstlane((lg ? 0 : s.nl) + y - g.ch * n);
  g.k0 = g.ch * len;
  g.k1 = min(nk, g.k0 + len);
  return g;
}

// The planes around its segment that a kernel's per-thread element offsets
// span: from `below` planes before the segment's first, where they start, to
// `ahead` planes after its last.
struct Span {
  int below, ahead;
};
constexpr Span kStageSpan{2, 2};  // the stage kernel and the adjoint's flux pass

// The most planes one segment may march: its offsets reach kc - 1 + below +
// ahead planes and, within a plane, less than three more (the two ghost planes
// before the interior, and the node), and must stay below 2^29 (32-bit byte
// offsets of doubles).  0 when even one plane is too large.
inline int segment_kmax(const Layout& L, Span s) {
  const long long k = (1LL << 29) / L.sk - (s.below + s.ahead + 2);
  return k < 1 ? 0 : (k > (1 << 30) ? (1 << 30) : (int)k);
}

// What bounds a kernel's offsets on a block (see segment_kmax): the most
// planes of its segments, the first and last plane it marches, and its span.
struct SegmentBounds {
  int planes, first, last, below, ahead;
};

// Periodic ghosts read at their source, so that nobody has to copy them: per[d]
// is the period of direction d (n, or n - 1 with superposed first and last
// nodes), 0 for a direction whose ghosts are read where they are.  A node
// outside the block along an in-plane direction with per = 0 keeps its place
// in all three (an edge ghost of a Dirichlet side holds a value of its own).
struct Wrap {
  int per[3] = {0, 0, 0};
};

// The in-plane element offset of column (i, j), both in [-2, n + 1], with the
// top bit set when its ghosts keep their place (an offset is below 2^29).
__device__ __forceinline__ unsigned wrap_column(const Layout& L, const Wrap& w, int i, int j) {
  const bool gi = i < 0 || i >= L.ni, gj = j < 0 || j >= L.nj;
  const bool own = (gi && !w.per[0]) || (gj && !w.per[1]);
  if (gi && !own) i += i < 0 ? w.per[0] : -w.per[0];
  if (gj && !own) j += j < 0 ? w.per[1] : -w.per[1];
  return (unsigned)(L.o + i + (long long)j * L.sj) | (own ? 0x80000000u : 0u);
}

// Plane k in [-2, n + 1] of the columns: element offset of the base plane and
// what columns that keep their place and columns that wrap add to it (both
// planes of a wrapped one are reached by 32-bit offsets from the lower).
struct PlaneRef {
  long long base;
  unsigned own, in;
};
__device__ __forceinline__ PlaneRef wrap_plane(const Layout& L, const Wrap& w, int k) {
  const unsigned p = (unsigned)((long long)w.per[2] * L.sk);
  const bool hi = k >= L.nk;
  return {(long long)(hi ? k - w.per[2] : k) * L.sk, hi ? p : 0, k < 0 ? p : 0};
}
__device__ __forceinline__ unsigned wrap_offset(unsigned col, const PlaneRef& p) {
  return (col & 0x7fffffffu) + ((int)col < 0 ? p.own : p.in);
}

// Global accesses use a uniform (scalar) base per field plus a 32-bit
// per-thread byte offset, so that each access needs one VGPR for its address.
template <class X>
__device__ __forceinline__ X ldo(const X* base, unsigned off) {
  return *(const X*)((const char*)base + (size_t)(off * (unsigned)sizeof(X)));
}
template <class X>
__device__ __forceinline__ void sto(X* base, unsigned off, X v) {
  *(X*)((char*)base + (size_t)(off * (unsigned)sizeof(X))) = v;
}

// One asynchronous global->LDS copy of 16 bytes (two doubles) per lane to 1 KB
// of consecutive LDS (dst uniform; lane l's 16 bytes land at dst + 16 l).
__device__ __forceinline__ void copy_to_lds(const char* src, double* dst) {
  __builtin_amdgcn_global_load_lds((const void*)src, (__attribute__((address_space(3))) void*)dst, 16, 0, 0);
}

// s_waitcnt vmcnt(N): all but the N most recent vector memory operations of
// this wave have completed (expcnt and lgkmcnt left unconstrained)
template <int N>
__device__ __forceinline__ void wait_vm() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (0x7 << 4) | (0xF << 8));
}

// Block barrier for LDS data only: release/acquire at workgroup scope for
// the local address space, so the wave waits for its own LDS operations but
// not for outstanding global loads, stores or global->LDS copies (which a
// full __syncthreads drains).
__device__ __forceinline__ void lds_barrier() {
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
  __builtin_amdgcn_s_waitcnt(0xC07F);
  __builtin_amdgcn_s_barrier();
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
}

// Priority (3 high .. 0) of this wave for its SIMD's issue slots.  Two waves
// share a SIMD; at equal priority the older one runs ahead and the younger
// finishes each phase alone, with nothing to hide its latencies behind, while
// the older waits at the barrier.  A wave that lowers its priority as it
// gets through a phase lets the one behind catch up.  (Stage kernel and
// dynamic closure; the adjoint's dissipation pass, whose phases wait more for
// LDS, lost 6 % by it.)
template <int N>
__device__ __forceinline__ void wave_priority() {
  __builtin_amdgcn_s_setprio(N);
}

// The value of the lane before / after this one (DPP wave shifts by one lane;
// the end lanes read 0).
__device__ __forceinline__ float lane_prev(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x138, 0xf, 0xf, true));
}
__device__ __forceinline__ float lane_next(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x130, 0xf, 0xf, true));
}
__device__ __forceinline__ double lane_prev(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x138, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x138, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double lane_next(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x130, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x130, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}

// Keeps the computation of x before this point (the compiler would sink it to
// the use, past a barrier, with all of its inputs alive).
__device__ __forceinline__ void pin(double& x) { asm volatile("" : "+v"(x)); }

// The ten metric values of this thread's node from its wave's copied rows
// (p = &block[0][row][column], fields 64 doubles apart).  Read by hand, with
// the wait for the reads in the same block: the compiler would wait for
// every outstanding copy, load and store of the wave before an LDS read of a
// block that copies write.  The caller has waited for the copies; the reads
// are done when this returns, so the block may be copied over.
__device__ __forceinline__ void read_metric_rows(const double* p, double m[9], double& J) {
  typedef double d2 __attribute__((ext_vector_type(2)));
  d2 m0, m1, m2, m3, m4;
  const unsigned la = (unsigned)(uintptr_t)(__attribute__((address_space(3))) const double*)p;
  asm volatile(
      "ds_read2st64_b64 %0, %5 offset0:0 offset1:1\n"
      "ds_read2st64_b64 %1, %5 offset0:2 offset1:3\n"
      "ds_read2st64_b64 %2, %5 offset0:4 offset1:5\n"
      "ds_read2st64_b64 %3, %5 offset0:6 offset1:7\n"
      "ds_read2st64_b64 %4, %5 offset0:8 offset1:9\n"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(m0), "=&v"(m1), "=&v"(m2), "=&v"(m3), "=&v"(m4)
      : "v"(la)
      : "memory");
  m[0] = m0.x; m[1] = m0.y; m[2] = m1.x; m[3] = m1.y; m[4] = m2.x;
  m[5] = m2.y; m[6] = m3.x; m[7] = m3.y; m[8] = m4.x;
  J = m4.y;
}

}  // namespace les
