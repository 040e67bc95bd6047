// Device helpers that the step kernels and the adjoint kernels share: lane moves, the kinetic
// operator along the lanes, the angles and scales of a step's substeps, and the order in which
// workgroups take tiles.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "qlg_internal.hpp"
#include "qlg_math.hpp"

namespace qlg {

// Whole-wavefront moves by one lane through DPP (wave_shl:1, wave_shr:1, both
// available on CDNA): a VALU operation that the compiler can fold into the
// arithmetic that consumes it, instead of a round trip through the LDS
// crossbar.  The end lane, always a halo lane here, reads 0.
constexpr int kDppWaveShl1 = 0x130;   // lane i reads lane i + 1
constexpr int kDppWaveShr1 = 0x138;   // lane i reads lane i - 1

template <int Ctrl>
__device__ __forceinline__ float dpp_move(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), Ctrl, 0xF, 0xF, true));
}
template <int Ctrl>
__device__ __forceinline__ double dpp_move(double v) {
  const unsigned long long u = (unsigned long long)__double_as_longlong(v);
  const unsigned lo = (unsigned)__builtin_amdgcn_mov_dpp((int)(unsigned)u, Ctrl, 0xF, 0xF, true);
  const unsigned hi = (unsigned)__builtin_amdgcn_mov_dpp((int)(unsigned)(u >> 32), Ctrl, 0xF, 0xF, true);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
template <typename T>
__device__ __forceinline__ cx<T> from_next_lane(cx<T> v) {
  return cx<T>{dpp_move<kDppWaveShl1>(v.re), dpp_move<kDppWaveShl1>(v.im)};
}
template <typename T>
__device__ __forceinline__ cx<T> from_prev_lane(cx<T> v) {
  return cx<T>{dpp_move<kDppWaveShr1>(v.re), dpp_move<kDppWaveShr1>(v.im)};
}

// Sum over the 64 lanes of a wavefront (every lane returns the total): within the rows of 16 lanes by
// shifts, then row by row, all through DPP moves.  Six dependent LDS exchanges of 64 bits took about
// three times as long.
template <int Ctrl, int RowMask>
__device__ __forceinline__ double dpp_add(double v) {
  const unsigned long long u = (unsigned long long)__double_as_longlong(v);
  const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)u, Ctrl, RowMask, 0xF, false);
  const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(u >> 32), Ctrl, RowMask, 0xF, false);
  return v + __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
__device__ __forceinline__ double wave_sum(double v) {
  v = dpp_add<0x111, 0xF>(v);   // row_shr:1, 2, 4, 8: lane 15 of each row holds its sum
  v = dpp_add<0x112, 0xF>(v);
  v = dpp_add<0x114, 0xF>(v);
  v = dpp_add<0x118, 0xF>(v);
  v = dpp_add<0x142, 0xA>(v);   // row_bcast:15 into rows 1 and 3
  v = dpp_add<0x143, 0xC>(v);   // row_bcast:31 into rows 2 and 3: lane 63 holds the total
  const unsigned long long u = (unsigned long long)__double_as_longlong(v);
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)u, kLanes - 1);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(u >> 32), kLanes - 1);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// Neighbours along the axis on the neighbouring lanes.
struct LaneShift {
  __device__ __forceinline__ bool one() const { return false; }
  template <typename T>
  __device__ __forceinline__ cx<T> next(cx<T> v) const { return from_next_lane(v); }
  template <typename T>
  __device__ __forceinline__ cx<T> prev(cx<T> v) const { return from_prev_lane(v); }
};

// 2i I'_q: S_q C S_q^T C by collide_r, with the axis along the lanes (the factor 1/(2i) is left to
// the caller).  Q = 1: qubit b (the paper's qubit 2) moves; Q = 0: qubit a (qubit 1).
template <typename T, int Q, typename Shift = LaneShift>
__device__ __forceinline__ void iprime_r_lanes(cx<T> (&a)[5], cx<T> (&b)[5], const Shift& sh = Shift{}) {
  collide_r(a, b);
#pragma unroll
  for (int m = 0; m < 5; ++m) {   // S^T: q(x) <- q(x + 1)
    if (Q) b[m] = sh.next(b[m]);
    else   a[m] = sh.next(a[m]);
  }
  collide_r(a, b);
#pragma unroll
  for (int m = 0; m < 5; ++m) {   // S: q(x) <- q(x - 1)
    if (Q) b[m] = sh.prev(b[m]);
    else   a[m] = sh.prev(a[m]);
  }
}

// The same along an axis of one site, where the streams are none.
template <typename T>
__device__ __forceinline__ void iprime_r_sites(cx<T> (&a)[5], cx<T> (&b)[5]) {
  collide_r(a, b);
  collide_r(a, b);
}

// What an interleaved substep U I' leaves the state multiplied by, in modulus: 2 from the I'
// (collide_r) times UScale from U.
template <typename T>
constexpr int kSubstepScale = 2 * UScale<T>::value;

// Angles of interleaved substep j = 0..3 of a four-I' sequence, on a state that
// carries the factor kSubstepScale^j (and i^j) of the j substeps before it: the n terms'
// angles and F's scale times kSubstepScale^-2j (exact).  Formed from the unscaled angles in
// registers, so that a run-time j reads no kernel argument inside the row loop.
template <typename T>
__device__ __forceinline__ Angles<T> substep_angles(const Angles<T>& base, int j) {
  const T f = ldexp(T(1), (kSubstepScale<T> == 4 ? -4 : -2) * j);
  Angles<T> a = base;
  a.tg0 *= f;
  a.tg25 *= f;
  a.fs = f;
  return a;
}

// The factor that brings the state back to its true value after kSubsteps (2 or 4) I', with a
// U before each of them or, in the plain split, with one U before the first (plain_u) or none.
template <typename T, int kSubsteps>
__device__ __forceinline__ T substep_unscale(bool plain, bool plain_u) {
  constexpr T i = kSubsteps == 4 ? T(1) / 16 : T(-1) / 4;   // (2i)^-kSubsteps
  constexpr T u = T(1) / UScale<T>::value;
  constexpr T un = kSubsteps == 4 ? u * u * u * u : u * u;
  return plain ? (plain_u ? i * u : i) : i * un;
}

__device__ __forceinline__ int64_t wrap64(int64_t x, int64_t n) {
  int64_t r = x % n;
  return r < 0 ? r + n : r;
}

// Workgroups are dispatched round-robin over the 8 XCDs of the chip, each with its
// own L2.  Give each XCD a contiguous range of logical workgroups, so that tiles
// that share halo rows and columns (consecutive tiles) read them through one L2.
constexpr int kXcds = 8;
__device__ __forceinline__ int xcd_contiguous_block(int b, int nblocks) {
  const int x = b % kXcds, l = b / kXcds;
  const int per = nblocks / kXcds, extra = nblocks % kXcds;
  return x * per + (x < extra ? x : extra) + l;
}

// Line passes: the lines along an axis are laid end to end, each with 4 halo slots on both sides
// (n + 8 slots), and cut into windows of 64 slots that overlap by 8: lane i of window w holds slot
// 56 w + i, and lanes 4..59 own their sites.  The halo slots between two lines of one window serve as
// those at its ends do, so a window holds the end of one line and the start of the next: nlines lines
// take (nlines (n + 8) - 8) / 56 windows, where windows that begin with each line would take
// nlines ceil(n / 56): 1.4 per line of 70 sites instead of 2, 4.7 of 256 instead of 5.  Where n is at
// or just below a multiple of 56 the latter are fewer, and the line's slots are that multiple.  Time
// per step with windows that begin with each line, and with these (us, complex128 / complex64): 64^3
// 131 / 93, 109 / 82; 50 x 70 x 90 135 / 95, 127 / 90; 128^3 785 / 525, 700 / 435; 256^3 5360 / 3365,
// 5200 / 3170; 1024^2 215 / 140, 215 / 132; the reverse step of 64^3 368 in complex64, 290.  (Those of
// complex128 before w_apply kept the state apart from its corrections; now 115, 127, 710, 5490 and 228.)
constexpr int kLineStride = kLanes - 2 * kLineHalo;
struct LineSlot {
  int line;   // its line (past the last one: any)
  int at;     // its site, periodic
  bool own;   // a site this lane computes
};
// Lines of one site have no neighbours (iprime_r_sites): a window takes 56 of them, where with halos
// of their own it held seven.
__device__ __forceinline__ LineSlot line_slot(uint32_t window, int lane, int n, int nlines) {
  if (n == 1) {
    const int line = (int)(window * kLineStride) + lane - kLineHalo;
    const bool own = lane >= kLineHalo && lane < kLanes - kLineHalo && line < nlines;
    return LineSlot{own ? line : 0, 0, own};
  }
  const uint32_t len = line_slots((uint32_t)n);
  const uint32_t slot = window * kLineStride, q = slot / len, r = slot - q * len + (uint32_t)lane;
  LineSlot s;
  uint32_t d;
  if (len != (uint32_t)n + 2 * kLineHalo) d = 0;   // whole windows: none crosses lines
  else if (len >= kLanes) d = r >= len ? 1u : 0u;
  else d = r / len;
  const bool in = q + d < (uint32_t)nlines;
  s.line = (int)(in ? q + d : q);
  const int pos = (int)(r - d * len) - kLineHalo;
  if (n < kLineHalo) s.at = (int)((uint32_t)(pos + kLineHalo * n) % (uint32_t)n);
  else s.at = pos < 0 ? pos + n : pos >= n ? pos - n : pos;   // whole windows: n > 48, pos < n + 12
  s.own = in && lane >= kLineHalo && lane < kLanes - kLineHalo && s.at == pos;
  return s;
}

// Group t of a pass along y or z over the runs of column groups (line_fold): which run and window,
// and a slot's plane and column group.
struct LineRun {
  int fold, nplanes, first, window;
  __device__ __forceinline__ LineRun(int t, int n, int planes, int ncol) {
    nplanes = planes;
    fold = (int)line_fold((uint32_t)n, (uint32_t)planes);
    const uint32_t runs = fold == 1 ? (uint32_t)ncol : (uint32_t)(ncol + fold - 1) / (uint32_t)fold;
    const uint32_t w = (uint32_t)t / runs;
    window = (int)w;
    first = (int)((uint32_t)t - w * runs) * fold;   // the run's first column group
  }
  __device__ __forceinline__ LineSlot slot(int i, int n, int* plane, int* col) const {
    const LineSlot l = line_slot(window, i, n, nplanes * fold);
    const int j = fold == 1 ? 0 : (int)((uint32_t)l.line / (uint32_t)nplanes);
    *plane = l.line - j * nplanes;
    *col = first + j;
    return l;
  }
};

}  // namespace qlg
