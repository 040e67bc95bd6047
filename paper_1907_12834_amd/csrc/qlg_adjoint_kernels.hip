// Kernels of the reverse-mode (adjoint) QLG step.
//
// The adjoint walks each step's substeps backwards.  The kinetic factors are
// linear and unitary, so their pull-back is the exact inverse I'^H = C^H S C^H S^T
// applied to the cotangent (no stored state).  The self-interaction is
// nonlinear: its pull-back (qlg_vjp.hpp, FP64) needs the substep's input
// state, which the recompute regenerates from the segment's checkpoint.
//
// Interleaved split: line passes, as the forward's (qlg_kernels.hip): the four
// substeps of one axis per launch, the axis along the lanes, 56 owned sites and
// 4 halo sites on each side per wavefront.  Plain split and objectives: one
// thread per site over 256-site chunks of each instance.

#include <algorithm>
#include <type_traits>

#include "qlg_adjoint_kernels.hpp"
#include "qlg_lanes.hpp"
#include "qlg_math.hpp"
#include "qlg_vjp.hpp"

namespace qlg {

namespace {

struct Site {
  InstDesc d;
  int c;            // the 256-site chunk this workgroup owns
  int s, x, y, z;
  bool ok;
};

// This thread's site in chunk c (thread t of the workgroup takes site t of the chunk).
__device__ __forceinline__ Site site_of_chunk(const LaunchGeom& g, int c) {
  Site r;
  r.c = c;
  r.d = g.inst[g.chunk2inst[c]];
  r.s = (c - r.d.chunk_begin) * kChunk + threadIdx.x;
  r.ok = r.s < r.d.sites;
  r.x = r.ok ? r.s % r.d.nx : 0;
  r.y = r.ok ? (r.s / r.d.nx) % r.d.ny : 0;
  r.z = r.ok ? r.s / (r.d.nx * r.d.ny) : 0;
  return r;
}

__device__ __forceinline__ Site site_here(const LaunchGeom& g) {
  return site_of_chunk(g, xcd_contiguous_block(blockIdx.x, gridDim.x));
}

// site index of the neighbour at offset dir (+1 / -1) along axis (0 = x, 1 = y, 2 = z), periodic
__device__ __forceinline__ int neighbour(const Site& r, int axis, int dir) {
  // one branch per axis: selecting the extent by a run-time axis index puts them on the stack
  if (axis == 0) {
    int x = r.x + dir;
    x = x < 0 ? x + r.d.nx : (x >= r.d.nx ? x - r.d.nx : x);
    return r.s - r.x + x;
  }
  if (axis == 1) {
    int y = r.y + dir;
    y = y < 0 ? y + r.d.ny : (y >= r.d.ny ? y - r.d.ny : y);
    return r.s + (y - r.y) * r.d.nx;
  }
  int z = r.z + dir;
  z = z < 0 ? z + r.d.nz : (z >= r.d.nz ? z - r.d.nz : z);
  return r.s + (z - r.z) * r.d.nx * r.d.ny;
}

template <typename T, typename S>
__device__ __forceinline__ void load_site(const cx<T>* __restrict__ st, const InstDesc& d, int s,
                                          cx<S> (&a)[5], cx<S> (&b)[5]) {
#pragma unroll
  for (int m = 0; m < 5; ++m) {
    const cx<T> va = st[d.off + m * d.stride + s];
    const cx<T> vb = st[d.off + (5 + m) * d.stride + s];
    a[m] = cx<S>{(S)va.re, (S)va.im};
    b[m] = cx<S>{(S)vb.re, (S)vb.im};
  }
}

template <typename T>
__device__ __forceinline__ void store_site(cx<T>* __restrict__ st, const InstDesc& d, int s, const cx<T> (&a)[5],
                                           const cx<T> (&b)[5]) {
#pragma unroll
  for (int m = 0; m < 5; ++m) {
    st[d.off + m * d.stride + s] = a[m];
    st[d.off + (5 + m) * d.stride + s] = b[m];
  }
}

// The same, with the non-temporal hint: for the recorded self-interaction
// inputs, written once per segment recompute and read back once, by the
// reverse sweep, so they need not displace lines the recompute still reads.
template <typename T>
__device__ __forceinline__ void store_site_nt(cx<T>* __restrict__ st, const InstDesc& d, int s, const cx<T> (&a)[5],
                                              const cx<T> (&b)[5]) {
#pragma unroll
  for (int m = 0; m < 5; ++m) {
    cx<T>* pa = st + d.off + m * d.stride + s;
    cx<T>* pb = st + d.off + (5 + m) * d.stride + s;
    __builtin_nontemporal_store(a[m].re, &pa->re);
    __builtin_nontemporal_store(a[m].im, &pa->im);
    __builtin_nontemporal_store(b[m].re, &pb->re);
    __builtin_nontemporal_store(b[m].im, &pb->im);
  }
}
template <typename T, typename S>
__device__ __forceinline__ void load_site_nt(const cx<T>* __restrict__ st, const InstDesc& d, int s,
                                             cx<S> (&a)[5], cx<S> (&b)[5]) {
#pragma unroll
  for (int m = 0; m < 5; ++m) {
    const cx<T>* pa = st + d.off + m * d.stride + s;
    const cx<T>* pb = st + d.off + (5 + m) * d.stride + s;
    a[m] = cx<S>{(S)__builtin_nontemporal_load(&pa->re), (S)__builtin_nontemporal_load(&pa->im)};
    b[m] = cx<S>{(S)__builtin_nontemporal_load(&pb->re), (S)__builtin_nontemporal_load(&pb->im)};
  }
}

// C^H times (1 - i), the adjoint of collide_r:  a' = a - i b,  b' = b - i a
__device__ __forceinline__ void collide_r_adj(cx<double>& a, cx<double>& b) {
  const cx<double> x = a, y = b;
  a = cx<double>{x.re + y.im, x.im - y.re};
  b = cx<double>{y.re + x.im, y.im - x.re};
}
__device__ __forceinline__ void collide_r_adj(cx<double> (&a)[5], cx<double> (&b)[5]) {
#pragma unroll
  for (int m = 0; m < 5; ++m) collide_r_adj(a[m], b[m]);
}

// lambda <- I'^H_{q} lambda with the axis along the lanes: q from the next site, C^H, q from the
// one before, C^H (the order of iprime_adj_site), the factors of the two C^H divided out.
// Q = 1: qubit b moves; Q = 0: qubit a.
template <int Q, typename Shift>
__device__ __forceinline__ void iprime_adj_lanes(const Shift& sh, cx<double> (&a)[5], cx<double> (&b)[5]) {
#pragma unroll
  for (int m = 0; m < 5; ++m) {
    if (Q) b[m] = sh.next(b[m]);
    else   a[m] = sh.next(a[m]);
  }
  collide_r_adj(a, b);
#pragma unroll
  for (int m = 0; m < 5; ++m) {
    if (Q) b[m] = sh.prev(b[m]);
    else   a[m] = sh.prev(a[m]);
  }
  collide_r_adj(a, b);
  unphase_by(a, b, -0.5);
}
// The same along an axis of one site.
__device__ __forceinline__ void iprime_adj_sites(cx<double> (&a)[5], cx<double> (&b)[5]) {
  collide_r_adj(a, b);
  collide_r_adj(a, b);
  unphase_by(a, b, -0.5);
}

// How a pass reads its neighbours along the axis: LaneShift along y and z of more than kThinAxis sites.
// one(): an axis of one site, without any.
// The same along x, of any extent.
struct LaneShiftX : LaneShift {
  int n;
  __device__ __forceinline__ bool one() const { return n == 1; }
};
// Lanes by number: the rings of a thin axis.
struct RingShift {
  int n, up, down;   // extent, lanes of the next site and of the one before, in bytes
  __device__ __forceinline__ bool one() const { return n == 1; }
  static __device__ __forceinline__ float read(float v, int lane) {
    return __int_as_float(__builtin_amdgcn_ds_bpermute(lane, __float_as_int(v)));
  }
  static __device__ __forceinline__ double read(double v, int lane) {
    const unsigned long long u = (unsigned long long)__double_as_longlong(v);
    const unsigned lo = (unsigned)__builtin_amdgcn_ds_bpermute(lane, (int)(unsigned)u);
    const unsigned hi = (unsigned)__builtin_amdgcn_ds_bpermute(lane, (int)(unsigned)(u >> 32));
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
  }
  template <typename T>
  __device__ __forceinline__ cx<T> next(cx<T> v) const { return cx<T>{read(v.re, up), read(v.im, up)}; }
  template <typename T>
  __device__ __forceinline__ cx<T> prev(cx<T> v) const { return cx<T>{read(v.re, down), read(v.im, down)}; }
};

}  // namespace

// (I' in)(x) for I'_{axis,q} = S_q C S_q^T C, from `in` at x-1, x, x+1, with the fused
// kernels' operation order: c = C(in) at x-1, x, x+1;  t(y) = (c.nonq(y), c.q(y+1));
// m(y) = C t(y) (two collides by collide_r, their exact factor 2i divided out at the end);
// out.nonq(x) = m(x).nonq, out.q(x) = m(x-1).q.
template <typename T>
__device__ __forceinline__ void iprime_site(const cx<T>* __restrict__ in, const Site& r, int axis, int qb,
                                            cx<T> (&oa)[5], cx<T> (&ob)[5]) {
  const int sm = neighbour(r, axis, -1), sp = neighbour(r, axis, +1);
  cx<T> a0[5], b0[5], a1[5], b1[5], a2[5], b2[5];   // x-1, x, x+1
  load_site(in, r.d, sm, a0, b0);
  load_site(in, r.d, r.s, a1, b1);
  load_site(in, r.d, sp, a2, b2);
  collide_r(a0, b0);
  collide_r(a1, b1);
  collide_r(a2, b2);
  cx<T> ta[5], tb[5], ua[5], ub[5];
#pragma unroll
  for (int m = 0; m < 5; ++m) {
    // t(x) = (nonq of c(x), q of c(x+1));  t(x-1) = (nonq of c(x-1), q of c(x))
    ta[m] = sel(qb != 0, a1[m], a2[m]);
    tb[m] = sel(qb != 0, b2[m], b1[m]);
    ua[m] = sel(qb != 0, a0[m], a1[m]);
    ub[m] = sel(qb != 0, b1[m], b0[m]);
  }
  collide_r(ta, tb);
  collide_r(ua, ub);
#pragma unroll
  for (int m = 0; m < 5; ++m) {
    oa[m] = sel(qb != 0, ta[m], ua[m]);   // moving qubit from m(x-1), the other from m(x)
    ob[m] = sel(qb != 0, ub[m], tb[m]);
  }
  unphase_by(oa, ob, T(0.5));
}

// One link of the recorded forward chain that regenerates a checkpoint segment:
//   z = I'_{axis,q}(in) at this site (z = in when axis < 0),  rec <- z (when rec is set),
//   out <- U(z) (out <- z when !with_u).
// Successive links walk the substeps "U_k then I'_k" of consecutive steps as
// "I'_{k-1} then U_k", so every input z of a self-interaction is written once.
// theta (V + mu) at a site, for a context with an external or chemical potential
__device__ __forceinline__ double ext_here(const Site& r, const double* pot, double mu, double theta) {
  return theta * ((pot ? pot[r.d.psi_off / 5 + r.s] : 0.0) + mu);
}

template <typename T>
__global__ __launch_bounds__(kChunk) void k_chain(const cx<T>* __restrict__ in, cx<T>* __restrict__ out,
                                                 cx<T>* __restrict__ rec, LaunchGeom g, int axis, int qb,
                                                 int with_u, Angles<T> ang, const double* __restrict__ pot,
                                                 double mu, double theta) {
  const Site r = site_here(g);
  if (!r.ok) return;
  cx<T> a[5], b[5];
  if (axis >= 0) iprime_site(in, r, axis, qb, a, b);
  else load_site(in, r.d, r.s, a, b);
  if (rec) store_site_nt(rec, r.d, r.s, a, b);
  if (with_u) {
    // the same per-site angle as the fused forward kernels: T(theta) T(V + mu)
    if (pot || mu != 0.0) potential<T, true>(a, b, ang, T(theta) * T((pot ? pot[r.d.psi_off / 5 + r.s] : 0.0) + mu));
    else potential(a, b, ang);
    scale_by(a, b, T(1) / UScale<T>::value);
  }
  store_site(out, r.d, r.s, a, b);
}

// (I'^H lambda)(x) = (C^H S_q C^H S_q^T lambda)(x) (FP64) from lambda at x-1, x, x+1:
//   w(y) = C^H(lambda.nonq(y), lambda.q(y+1));  out(x) = C^H(w(x).nonq, w(x-1).q).
__device__ __forceinline__ void iprime_adj_site(const cx<double>* __restrict__ in, const Site& r, int axis, int qb,
                                                cx<double> (&oa)[5], cx<double> (&ob)[5]) {
  const int sm = neighbour(r, axis, -1), sp = neighbour(r, axis, +1);
  // All loads of a thread are in flight before the first is used, the components one after the other: one
  // component's result waits for its six loads only.  Left to itself the compiler takes the loads in groups,
  // in 73 registers (a substep of 512^2 15.9 us, of 1024^2 82; so 13.8 and 73).
  cx<double> z[5][6];   // a and b at x-1, x, x+1
#pragma unroll
  for (int m = 0; m < 5; ++m) {
    const cx<double>* p = in + r.d.off + m * r.d.stride;
    const cx<double>* q = p + 5 * r.d.stride;
    z[m][0] = p[sm];
    z[m][1] = q[sm];
    z[m][2] = p[r.s];
    z[m][3] = q[r.s];
    z[m][4] = p[sp];
    z[m][5] = q[sp];
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int m = 0; m < 5; ++m) {
    cx<double> wa = sel(qb != 0, z[m][2], z[m][4]), wb = sel(qb != 0, z[m][5], z[m][3]);   // w(x)
    cx<double> va = sel(qb != 0, z[m][0], z[m][2]), vb = sel(qb != 0, z[m][3], z[m][1]);   // w(x-1)
    collide_r_adj(wa, wb);
    collide_r_adj(va, vb);
    oa[m] = sel(qb != 0, wa, va);
    ob[m] = sel(qb != 0, vb, wb);
    collide_r_adj(oa[m], ob[m]);
  }
  unphase_by(oa, ob, -0.5);
}

// lambda <- I'^H lambda, out of place.
__global__ __launch_bounds__(kChunk) void k_sub_iprime_adj(const cx<double>* __restrict__ in,
                                                          cx<double>* __restrict__ out, LaunchGeom g, int axis,
                                                          int qb) {
  const Site r = site_here(g);
  if (!r.ok) return;
  cx<double> oa[5], ob[5];
  iprime_adj_site(in, r, axis, qb, oa, ob);
  store_site(out, r.d, r.s, oa, ob);
}

// Block sum of three doubles into dst[0..2] (fixed order).
__device__ __forceinline__ void block_sum3(double v0, double v1, double v2, double* __restrict__ dst) {
  __shared__ double red[3][kChunk / kLanes];
  const int lane = threadIdx.x & (kLanes - 1), wv = threadIdx.x >> 6;
  double v[3] = {v0, v1, v2};
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const double s = wave_sum(v[k]);
    if (lane == 0) red[k][wv] = s;
  }
  __syncthreads();
  if (threadIdx.x < 3) {
    double s = 0.0;
#pragma unroll
    for (int j = 0; j < kChunk / kLanes; ++j) s += red[threadIdx.x][j];
    dst[threadIdx.x] = s;
  }
}

// lambda <- (dU)^H lambda at the substep input z (FP64 Jacobian); dg partials per chunk.
template <typename T>
__global__ __launch_bounds__(kChunk) void k_sub_vjp(const cx<T>* __restrict__ z, cx<double>* __restrict__ lam,
                                                   LaunchGeom g, double theta, double g0, double g1, double g2,
                                                   const double* __restrict__ pot, double mu,
                                                   double* __restrict__ part) {
  const Site r = site_here(g);
  double dg[3] = {0.0, 0.0, 0.0};
  if (r.ok) {
    cx<double> a[5], b[5], la[5], lb[5];
    load_site_nt(z, r.d, r.s, a, b);
    load_site(lam, r.d, r.s, la, lb);
    potential_vjp(a, b, la, lb, theta, g0, g1, g2, dg, ext_here(r, pot, mu, theta));
    store_site(lam, r.d, r.s, la, lb);
  }
  block_sum3(dg[0], dg[1], dg[2], part + 3 * (int64_t)r.c);
}

// ---------------------------------------------------------------------------
// Interleaved split: recompute and pull-back as line passes
// ---------------------------------------------------------------------------
// One launch per axis and step for the recompute and one for the pull-back, the state and the
// cotangent in registers through four substeps.  With a launch per y substep (each read the
// cotangent of three sites and a record and wrote the cotangent), a persistent kernel for the four x
// substeps and the derivative in the frame of F a reverse step of 512^2 took 278 us in complex64,
// 355 in complex128, of 64^2 in complex128 64; now 172, 227 and 39.  Bound by the FP64 derivative (1060
// instructions per substep; 256 registers, so two wavefronts per SIMD: 52 % of the issue rate at
// 512^2) and by the records' traffic.  Records copied to LDS a substep ahead gained nothing (512^2
// complex64 180 -> 186 us, complex128 229 -> 227).  Along y and z axes of up to kThinAxis sites the
// windows are others (ThinTile).
//
// Along x a wavefront takes one window of the lines laid end to end (line_slot); along y or z a
// workgroup takes W neighbouring columns of one window, turned in LDS (as k_line_yz).  pre[i] is the
// first window of instance i, pre[nbatch] their number; both are read through the constant address
// space (scalar loads).
struct LineTile {
  InstDesc d;
  int t;             // x: window, y and z: group of the instance
  int n;             // extent along the lines
};
__device__ __forceinline__ int line_instance(const LaunchGeom& g, const int* pre_g, int w, InstDesc* d, int* t) {
  typedef const __attribute__((address_space(4))) int32_t* CInt;
  const CInt pre = (CInt)pre_g;
  int lo = 0, hi = g.nbatch;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (pre[mid] <= w) lo = mid;
    else hi = mid;
  }
  static_assert(sizeof(InstDesc) % 4 == 0, "InstDesc is read as 32-bit words");
  constexpr int kWords = (int)(sizeof(InstDesc) / 4);
  const CInt words = (CInt)g.inst + kWords * lo;
  int32_t buf[kWords];
#pragma unroll
  for (int i = 0; i < kWords; ++i) buf[i] = words[i];
  __builtin_memcpy(d, buf, sizeof(InstDesc));
  *t = w - pre[lo];
  return lo;
}
__device__ __forceinline__ LineTile line_tile_x(const LaunchGeom& g, const int* pre, int w) {
  LineTile r;
  line_instance(g, pre, w, &r.d, &r.t);
  r.n = r.d.nx;
  return r;
}
struct LineTileYz : LineTile {
  bool zp;
  int rstride, pstride;   // sites between neighbours along the line, and between planes
};
__device__ __forceinline__ LineTileYz line_tile_yz(const LaunchGeom& g, const int* pre, int grp, bool zp) {
  LineTileYz r;
  line_instance(g, pre, grp, &r.d, &r.t);
  r.zp = zp;
  r.n = zp ? r.d.nz : r.d.ny;
  r.rstride = zp ? r.d.nx * r.d.ny : r.d.nx;
  r.pstride = zp ? r.d.nx : r.d.nx * r.d.ny;
  return r;
}
template <int W>
__device__ __forceinline__ LineRun line_run(const LineTileYz& t) {
  return LineRun(t.t, t.n, t.zp ? t.d.ny : t.d.nz, (t.d.nx + W - 1) / W);
}
// This thread's element of a group's window, 64 slots x W columns, for the loads and stores that run
// along x.
template <int W>
struct TileElem {
  int er, ec;
  int at;          // site
  bool store;
  __device__ __forceinline__ TileElem(const LineTileYz& t, const LineRun& run) {
    er = threadIdx.x / W;
    ec = threadIdx.x % W;
    int plane, col;
    const LineSlot l = run.slot(er, t.n, &plane, &col);
    const int x = col * W + ec;
    at = plane * t.pstride + l.at * t.rstride + (x < t.d.nx ? x : t.d.nx - 1);
    store = l.own && x < t.d.nx;
  }
};
// This lane's place in a record along y or z: site `at` of the line of column x and plane p, at
// (p nx + x) n + at.
template <int W>
struct LaneElem {
  bool own;
  int rec;         // place in a record
  int pot;         // site
  __device__ __forceinline__ LaneElem(const LineTileYz& t, const LineRun& run, int lane, int wv) {
    int plane, col;
    const LineSlot l = run.slot(lane, t.n, &plane, &col);
    int x = col * W + wv;
    own = l.own && x < t.d.nx;
    if (x >= t.d.nx) x = t.d.nx - 1;
    rec = (plane * t.d.nx + x) * t.n + l.at;
    pot = plane * t.pstride + l.at * t.rstride + x;
  }
};

// The recompute of one axis: z_0 = in, z_{k+1} = I'_k U(z_k) for k = 0..3 (qubits b, b, a, a),
// out = z_4.  rec + k rstep receives z_k, k >= first (along x a record is a state copy; along y
// and z it runs along the lines, site r of the line of column x and plane p at (p nx + x) n + r,
// so that the pull-back's lanes read it without a turn).
template <typename T, bool kExt, typename Shift, typename Put>
__device__ __forceinline__ void recompute_substeps(const Shift& sh, cx<T> (&a)[5], cx<T> (&b)[5], const Angles<T>& ang, T ext,
                                                  Put put) {
  constexpr T kUnscale = T(0.5) / UScale<T>::value;   // of U and of the I' after it
#pragma unroll 1
  for (int k = 0; k < 2; ++k) {
    put(k);
    potential<T, kExt>(a, b, ang, ext);
    if (sh.one()) iprime_r_sites(a, b);
    else iprime_r_lanes<T, 1>(a, b, sh);
    unphase_by(a, b, kUnscale);
  }
#pragma unroll 1
  for (int k = 2; k < 4; ++k) {
    put(k);
    potential<T, kExt>(a, b, ang, ext);
    if (sh.one()) iprime_r_sites(a, b);
    else iprime_r_lanes<T, 0>(a, b, sh);
    unphase_by(a, b, kUnscale);
  }
}

// (FP64: a budget for three wavefronts per SIMD, as k_line_yz.)
template <typename T, bool kExt>
__global__ __launch_bounds__(kChunk) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 8 ? 3 : 1)))
void k_recompute_x(const cx<T>* __restrict__ in, cx<T>* __restrict__ out,
                                                       cx<T>* __restrict__ rec, int64_t rstep, int first,
                                                       LaunchGeom g, const int* __restrict__ pre, int nwaves,
                                                       Angles<T> ang, const double* __restrict__ pot, double mu,
                                                       double theta) {
  constexpr int kWaves = kChunk / kLanes;
  const int w = xcd_contiguous_block(blockIdx.x, gridDim.x) * kWaves + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (w >= nwaves) return;
  const LineTile t = line_tile_x(g, pre, w);
  const LineSlot l = line_slot(t.t, threadIdx.x & (kLanes - 1), t.n, t.d.ny * t.d.nz);
  const int s = l.line * t.n + l.at;
  cx<T> a[5], b[5];
  load_site(in, t.d, s, a, b);
  T ext = T(0);
  if constexpr (kExt) ext = T(theta) * T((pot ? pot[t.d.psi_off / 5 + s] : 0.0) + mu);
  recompute_substeps<T, kExt>(LaneShiftX{{}, t.n}, a, b, ang, ext, [&](int k) __attribute__((always_inline)) {
    if (l.own && k >= first) store_site_nt(rec + k * rstep, t.d, s, a, b);
  });
  if (l.own) store_site(out, t.d, s, a, b);
}

// The same budget.
template <typename T, int W, bool kExt>
__global__ __launch_bounds__(kLanes * W) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 8 ? 3 : 2)))
void k_recompute_yz(const cx<T>* __restrict__ in, cx<T>* __restrict__ out,
                                                            cx<T>* __restrict__ rec, int64_t rstep, LaunchGeom g,
                                                            const int* __restrict__ pre, int zp, Angles<T> ang,
                                                            const double* __restrict__ pot, double mu, double theta) {
  __shared__ cx<T> buf[10][kLanes][W + 1];
  const int lane = threadIdx.x & (kLanes - 1), wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const LineTileYz t = line_tile_yz(g, pre, xcd_contiguous_block(blockIdx.x, gridDim.x), zp != 0);
  const LineRun run = line_run<W>(t);
  const TileElem<W> e(t, run);
  {
    cx<T> v[10];
#pragma unroll
    for (int p = 0; p < 10; ++p) v[p] = in[t.d.off + e.at + p * t.d.stride];
#pragma unroll
    for (int p = 0; p < 10; ++p) buf[p][e.er][e.ec] = v[p];
  }
  __syncthreads();
  cx<T> a[5], b[5];
#pragma unroll
  for (int m = 0; m < 5; ++m) {
    a[m] = buf[m][lane][wv];
    b[m] = buf[5 + m][lane][wv];
  }
  const LaneElem<W> le(t, run, lane, wv);
  T ext = T(0);
  if constexpr (kExt) ext = T(theta) * T((pot ? pot[t.d.psi_off / 5 + le.pot] : 0.0) + mu);
  recompute_substeps<T, kExt>(LaneShift{}, a, b, ang, ext, [&](int k) __attribute__((always_inline)) {
    if (le.own) store_site_nt(rec + k * rstep, t.d, le.rec, a, b);
  });
#pragma unroll
  for (int m = 0; m < 5; ++m) {
    buf[m][lane][wv] = a[m];
    buf[5 + m][lane][wv] = b[m];
  }
  __syncthreads();
  if (e.store) {
#pragma unroll
    for (int p = 0; p < 10; ++p) out[t.d.off + e.at + p * t.d.stride] = buf[p][e.er][e.ec];
  }
}

// The pull-back through one axis: for k = 3, ..., 0 (qubits a, a, b, b),
//   lambda <- (dU_k)^H I'^H_k lambda  at the recorded inputs z_k = rec + k rstep,
// site s of the records on this lane.  dg: the sums of this lane's site (owned lanes only).
template <typename T, typename Shift>
__device__ __forceinline__ void adjoint_substeps(const Shift& sh, cx<double> (&la)[5], cx<double> (&lb)[5],
                                                const cx<T>* __restrict__ rec, int64_t rstep, const InstDesc& d, int s,
                                                double theta, double g0, double g1, double g2, double ext,
                                                double (&dg)[3]) {
  auto substep = [&](int k, auto q) __attribute__((always_inline)) {
    cx<double> a[5], b[5];
    load_site_nt(rec + k * rstep, d, s, a, b);
    if (sh.one()) iprime_adj_sites(la, lb);
    else iprime_adj_lanes<decltype(q)::value>(sh, la, lb);
    potential_vjp(a, b, la, lb, theta, g0, g1, g2, dg, ext);
  };
#pragma unroll 1
  for (int k = 3; k >= 2; --k) substep(k, std::integral_constant<int, 0>{});
#pragma unroll 1
  for (int k = 1; k >= 0; --k) substep(k, std::integral_constant<int, 1>{});
}

// dL/dg of a wavefront's owned lanes into part[0..2].
__device__ __forceinline__ void store_dg(double (&dg)[3], bool own, int lane, double* __restrict__ part) {
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    dg[k] = wave_sum(own ? dg[k] : 0.0);
  }
  if (lane == 0) {
    part[0] = dg[0];
    part[1] = dg[1];
    part[2] = dg[2];
  }
}

template <typename T>
__global__ __launch_bounds__(kChunk) __attribute__((amdgpu_waves_per_eu(2)))
void k_adjoint_x(const cx<T>* __restrict__ rec, int64_t rstep, const cx<double>* __restrict__ lin,
                 cx<double>* __restrict__ lout, LaunchGeom g, const int* __restrict__ pre, int nwaves, double theta,
                 double g0, double g1, double g2, const double* __restrict__ pot, double mu,
                 double* __restrict__ part) {
  constexpr int kWaves = kChunk / kLanes;
  const int w = xcd_contiguous_block(blockIdx.x, gridDim.x) * kWaves + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (w >= nwaves) return;
  const int lane = threadIdx.x & (kLanes - 1);
  const LineTile t = line_tile_x(g, pre, w);
  const LineSlot l = line_slot(t.t, lane, t.n, t.d.ny * t.d.nz);
  const int s = l.line * t.n + l.at;
  cx<double> la[5], lb[5];
  load_site(lin, t.d, s, la, lb);
  const double ext = theta * ((pot ? pot[t.d.psi_off / 5 + s] : 0.0) + mu);
  double dg[3] = {0.0, 0.0, 0.0};
  adjoint_substeps(LaneShiftX{{}, t.n}, la, lb, rec, rstep, t.d, s, theta, g0, g1, g2, ext, dg);
  if (l.own) store_site(lout, t.d, s, la, lb);
  store_dg(dg, l.own, lane, part + 3 * (int64_t)w);
}

template <typename T>
__global__ __launch_bounds__(kLanes * kAdjCols) __attribute__((amdgpu_waves_per_eu(2)))
void k_adjoint_yz(const cx<T>* __restrict__ rec, int64_t rstep, const cx<double>* __restrict__ lin,
                  cx<double>* __restrict__ lout, LaunchGeom g, const int* __restrict__ pre, int zp, double theta,
                  double g0, double g1, double g2, const double* __restrict__ pot, double mu,
                  double* __restrict__ part) {
  constexpr int W = kAdjCols;
  __shared__ cx<double> buf[10][kLanes][W + 1];
  // this thread's site through the substeps, whose registers are all taken (with it and its places
  // in LDS spilled to scratch 13 registers per lane: 512^2 71 -> 68 us a launch without)
  __shared__ volatile int keep[kLanes * W];
  const int lane = threadIdx.x & (kLanes - 1), wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int grp = xcd_contiguous_block(blockIdx.x, gridDim.x);
  const LineTileYz t = line_tile_yz(g, pre, grp, zp != 0);
  const LineRun run = line_run<W>(t);
  {
    const TileElem<W> e(t, run);
    keep[threadIdx.x] = e.store ? e.at : -1;
    cx<double> v[10];
#pragma unroll
    for (int p = 0; p < 10; ++p) v[p] = lin[t.d.off + e.at + p * t.d.stride];
#pragma unroll
    for (int p = 0; p < 10; ++p) buf[p][e.er][e.ec] = v[p];
  }
  __syncthreads();
  cx<double> la[5], lb[5];
#pragma unroll
  for (int m = 0; m < 5; ++m) {
    la[m] = buf[m][lane][wv];
    lb[m] = buf[5 + m][lane][wv];
  }
  const LaneElem<W> le(t, run, lane, wv);
  const double ext = theta * ((pot ? pot[t.d.psi_off / 5 + le.pot] : 0.0) + mu);
  double dg[3] = {0.0, 0.0, 0.0};
  adjoint_substeps(LaneShift{}, la, lb, rec, rstep, t.d, le.rec, theta, g0, g1, g2, ext, dg);
#pragma unroll
  for (int m = 0; m < 5; ++m) {
    buf[m][lane][wv] = la[m];
    buf[5 + m][lane][wv] = lb[m];
  }
  store_dg(dg, le.own, lane, part + 3 * ((int64_t)grp * W + wv));
  __syncthreads();
  // the thread number made opaque, so that its ten places in LDS are not kept through the substeps
  unsigned tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  tid &= kLanes * W - 1;
  const int at = keep[tid];
  if (at >= 0) {
    cx<double>* dst = lout + t.d.off + at;
#pragma unroll
    for (int p = 0; p < 10; ++p) dst[p * t.d.stride] = buf[p][tid / W][tid % W];
  }
}

// Axes of up to kThinAxis sites along y or z: a wavefront takes 64 / n whole lines without halos, in site
// order (x, then the planes), lane at * (64 / n) + l holding site `at` of line l: loads, stores and
// records (here a state copy) run along x as they lie, without a turn in LDS, and the neighbours are the
// other lanes of a ring, read through the LDS crossbar.  In windows with halos and columns turned in LDS
// two or three sites of ten or eleven slots were their own, and lines of one site were stored one by one;
// a reverse step took (us, complex64 / complex128; in brackets with one thread per site and substep)
// 300000 x 1 496 / 536 (340 / 422), now 190 / 245; 150000 x 2 517 / 593 (367 / 461), 190 / 244;
// 100000 x 3 457 / 525 (384 / 501), 213 / 279; 400 x 400 x 2 701 / 782 (588 / 749), 301 / 388.  From four
// sites on the halos' windows are ahead of a thread per site (75000 x 4 348 / 389; 385 / 503).
struct ThinTile : LineTileYz {
  int s;
  bool own;
  RingShift ring;
  __device__ __forceinline__ ThinTile(const LineTileYz& t, int lane) : LineTileYz(t) {
    const int per = kLanes / n, at0 = lane / per, l = lane - at0 * per;
    const bool in = at0 < n;   // three sites: lane 63 holds none
    const int at = in ? at0 : 0;
    const uint32_t nlines = (uint32_t)d.sites / (uint32_t)n, line0 = (uint32_t)this->t * (uint32_t)per + (uint32_t)l;
    own = in && line0 < nlines;
    const uint32_t line = line0 < nlines ? line0 : nlines - 1u;
    const uint32_t plane = line / (uint32_t)d.nx;   // of the planes of one site along the axis
    s = zp ? (int)line + at * rstride : (int)plane * pstride + at * rstride + (int)(line - plane * (uint32_t)d.nx);
    ring.n = n;
    ring.up = 4 * (in ? (at + 1 == n ? 0 : at + 1) * per + l : lane);
    ring.down = 4 * (in ? (at == 0 ? n - 1 : at - 1) * per + l : lane);
  }
};

template <typename T, bool kExt>
__global__ __launch_bounds__(kChunk) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 8 ? 3 : 1)))
void k_recompute_thin(const cx<T>* __restrict__ in, cx<T>* __restrict__ out,
                                                          cx<T>* __restrict__ rec, int64_t rstep, LaunchGeom g,
                                                          const int* __restrict__ pre, int nwaves, int zp,
                                                          Angles<T> ang, const double* __restrict__ pot, double mu,
                                                          double theta) {
  constexpr int kWaves = kChunk / kLanes;
  const int w = xcd_contiguous_block(blockIdx.x, gridDim.x) * kWaves + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (w >= nwaves) return;
  const ThinTile t(line_tile_yz(g, pre, w, zp != 0), threadIdx.x & (kLanes - 1));
  cx<T> a[5], b[5];
  load_site(in, t.d, t.s, a, b);
  T ext = T(0);
  if constexpr (kExt) ext = T(theta) * T((pot ? pot[t.d.psi_off / 5 + t.s] : 0.0) + mu);
  recompute_substeps<T, kExt>(t.ring, a, b, ang, ext, [&](int k) __attribute__((always_inline)) {
    if (t.own) store_site_nt(rec + k * rstep, t.d, t.s, a, b);
  });
  if (t.own) store_site(out, t.d, t.s, a, b);
}

template <typename T>
__global__ __launch_bounds__(kChunk) __attribute__((amdgpu_waves_per_eu(2)))
void k_adjoint_thin(const cx<T>* __restrict__ rec, int64_t rstep, const cx<double>* __restrict__ lin,
                    cx<double>* __restrict__ lout, LaunchGeom g, const int* __restrict__ pre, int nwaves, int zp,
                    double theta, double g0, double g1, double g2, const double* __restrict__ pot, double mu,
                    double* __restrict__ part) {
  constexpr int kWaves = kChunk / kLanes;
  const int w = xcd_contiguous_block(blockIdx.x, gridDim.x) * kWaves + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (w >= nwaves) return;
  const int lane = threadIdx.x & (kLanes - 1);
  const ThinTile t(line_tile_yz(g, pre, w, zp != 0), lane);
  cx<double> la[5], lb[5];
  load_site(lin, t.d, t.s, la, lb);
  const double ext = theta * ((pot ? pot[t.d.psi_off / 5 + t.s] : 0.0) + mu);
  double dg[3] = {0.0, 0.0, 0.0};
  adjoint_substeps(t.ring, la, lb, rec, rstep, t.d, t.s, theta, g0, g1, g2, ext, dg);
  if (t.own) store_site(lout, t.d, t.s, la, lb);
  store_dg(dg, t.own, lane, part + 3 * (int64_t)w);
}

// The instance tables of the line passes, one after the other (nbatch + 1 entries each): x windows, y
// and z groups of the recompute (rec_cols columns), y and z groups of the pull-back (kAdjCols), y and z
// windows of thin axes.  Along y and z an instance has either groups or windows.
__global__ void k_line_prefix(LaunchGeom g, int rec_cols, int* __restrict__ pre) {
  const int q = threadIdx.x;
  if (q >= kLinePrefixes) return;
  int* p = pre + q * (g.nbatch + 1);
  const int cols = q <= 2 ? rec_cols : kAdjCols;
  int acc = 0;
  for (int i = 0; i < g.nbatch; ++i) {
    p[i] = acc;
    const InstDesc d = g.inst[i];
    const uint32_t nx = d.nx, ny = d.ny, nz = d.nz, ncol = (nx + cols - 1) / cols;
    const uint32_t n = q & 1 ? ny : nz, planes = q & 1 ? nz : ny;
    if (q == 0) acc += line_windows(nx, ny * nz);
    else if (n <= kThinAxis) acc += q >= 5 ? thin_windows(n, nx * planes) : 0u;
    else acc += q >= 5 ? 0u : line_groups(n, planes, ncol);
  }
  p[g.nbatch] = acc;
}

// acc[0..2] += sum over chunks of part (single block, fixed order).  Unrolling
// issues the loads of eight chunks ahead of their additions; each thread still
// adds its chunks in increasing order.
// One workgroup of 1024 threads: thread t sums the partials t, t + 1024, ... (a serial chain of
// a few dozen loads each), then the 16 wavefront sums are added in order.
constexpr int kDgThreads = 1024;
__global__ __launch_bounds__(kDgThreads) void k_dg_accumulate(const double* __restrict__ part, int nparts,
                                                            double* __restrict__ acc) {
  constexpr int kW = kDgThreads / kLanes;
  __shared__ double red[3][kW];
  const int lane = threadIdx.x & (kLanes - 1), wv = threadIdx.x >> 6;
  double v[3] = {0.0, 0.0, 0.0};
#pragma unroll 8
  for (int c = threadIdx.x; c < nparts; c += kDgThreads) {
    v[0] += part[3 * c];
    v[1] += part[3 * c + 1];
    v[2] += part[3 * c + 2];
  }
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const double s = wave_sum(v[k]);
    if (lane == 0) red[k][wv] = s;
  }
  __syncthreads();
  if (threadIdx.x < 3) {
    double t = 0.0;
#pragma unroll
    for (int j = 0; j < kW; ++j) t += red[threadIdx.x][j];
    acc[threadIdx.x] += t;
  }
}

// First stage of launch_dg_reduce: workgroup b sums the partials of its contiguous range
// [b n / G, (b + 1) n / G) (thread t: entries t, t + 256, ... of the range; then the four
// wavefront sums in order) into red[b][0..2].
__global__ __launch_bounds__(kChunk) void k_dg_blocks(const double* __restrict__ part, int64_t n,
                                                     double* __restrict__ red) {
  const int64_t G = gridDim.x;
  const int64_t lo = n * blockIdx.x / G, hi = n * (blockIdx.x + 1) / G;
  double v[3] = {0.0, 0.0, 0.0};
#pragma unroll 8
  for (int64_t c = lo + threadIdx.x; c < hi; c += kChunk) {
    v[0] += part[3 * c];
    v[1] += part[3 * c + 1];
    v[2] += part[3 * c + 2];
  }
  block_sum3(v[0], v[1], v[2], red + 3 * (int64_t)blockIdx.x);
}

// Energy objective: lambda_a = lambda_b = 2 dE/dpsi* written in the canonical
// complex128 qubits layout; per chunk partials part[6c + 0..3] of
// eps^d x (E density, n^2/2, |F|^2/2, |sigma|^2/10).
template <typename T>
__global__ __launch_bounds__(kChunk) void k_energy_grad(const cx<T>* __restrict__ st, cx<double>* __restrict__ lam,
                                                       LaunchGeom g, int ndim, double eps, double g0,
                                                       double g1, double g2, const double* __restrict__ pot,
                                                       double mu, double* __restrict__ part) {
  const Site r = site_here(g);
  double e = 0.0, en = 0.0, ef = 0.0, es = 0.0;
  if (r.ok) {
    const double meas = ndim == 1 ? eps : ndim == 2 ? eps * eps : eps * eps * eps;
    const double ie2 = 1.0 / (eps * eps);
    cx<double> a[5], b[5], p[5], lap[5];
    load_site(st, r.d, r.s, a, b);
#pragma unroll
    for (int m = 0; m < 5; ++m) {
      p[m] = a[m] + b[m];
      lap[m] = cx<double>{0.0, 0.0};
    }
    double ekin = 0.0;
    for (int axis = 0; axis < ndim; ++axis) {
      cx<double> pa[5], pb[5], ma[5], mb[5];
      load_site(st, r.d, neighbour(r, axis, +1), pa, pb);
      load_site(st, r.d, neighbour(r, axis, -1), ma, mb);
#pragma unroll
      for (int m = 0; m < 5; ++m) {
        const cx<double> pp = pa[m] + pb[m], pm = ma[m] + mb[m];
        const cx<double> df = pp - p[m];
        ekin += df.re * df.re + df.im * df.im;
        lap[m] = lap[m] + (2.0 * p[m] - pp - pm);
      }
    }
    // H_loc psi = g0 n psi + g1 (F.f) psi + (g2/5) sigma S psi*
    double q[5], n = 0.0;
#pragma unroll
    for (int m = 0; m < 5; ++m) {
      q[m] = p[m].re * p[m].re + p[m].im * p[m].im;
      n += q[m];
    }
    const double Fz = 2.0 * (q[0] - q[4]) + (q[1] - q[3]);
    const cx<double> f1 = cmulc(p[0], p[1]) + cmulc(p[3], p[4]);
    const cx<double> f2 = cmulc(p[1], p[2]) + cmulc(p[2], p[3]);
    const double Fx = 2.0 * f1.re + Consts::r6 * f2.re, Fy = 2.0 * f1.im + Consts::r6 * f2.im;
    const cx<double> sig = 2.0 * (p[0] * p[4]) - 2.0 * (p[1] * p[3]) + p[2] * p[2];
    const double cf[4] = {2.0, Consts::r6, Consts::r6, 2.0};
    cx<double> fp[5] = {}, fm[5] = {};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      fp[i] = cf[i] * p[i + 1];
      fm[i + 1] = cf[i] * p[i];
    }
    const cx<double> cpl{0.5 * Fx, -0.5 * Fy}, cmi{0.5 * Fx, 0.5 * Fy};
    const double vmu = ext_here(r, pot, mu, 1.0);   // V + mu at this site (0 without a potential)
    cx<double> Sp[5];
    {
      cx<double> pc[5];
#pragma unroll
      for (int m = 0; m < 5; ++m) pc[m] = conj(p[m]);
      Sp[0] = pc[4]; Sp[1] = -1.0 * pc[3]; Sp[2] = pc[2]; Sp[3] = -1.0 * pc[1]; Sp[4] = pc[0];
    }
#pragma unroll
    for (int m = 0; m < 5; ++m) {
      cx<double> h = (g0 * n + vmu) * p[m] + g1 * ((Fz * (2 - m)) * p[m] + cpl * fp[m] + cmi * fm[m]);
      h = h + (g2 / 5.0) * (sig * Sp[m]);
      const cx<double> l = (2.0 * meas) * (ie2 * lap[m] + h);
      const int64_t o = r.d.qb_off + (int64_t)m * r.d.sites + r.s;
      lam[o] = l;
      lam[o + 5 * (int64_t)r.d.sites] = l;
    }
    const double f2s = Fx * Fx + Fy * Fy + Fz * Fz, s2 = sig.re * sig.re + sig.im * sig.im;
    e = ekin * ie2 + 0.5 * (g0 * n * n + g1 * f2s + g2 * s2 / 5.0) + vmu * n;
    en = 0.5 * n * n;
    ef = 0.5 * f2s;
    es = 0.1 * s2;
    e *= meas; en *= meas; ef *= meas; es *= meas;
  }
  // four partials in a 6-double slot per chunk: two block sums (e, en, ef) and (es, 0, 0)
  block_sum3(e, en, ef, part + 6 * (int64_t)r.c);
  __syncthreads();
  block_sum3(es, 0.0, 0.0, part + 6 * (int64_t)r.c + 3);
}

// Fidelity objective, pass 1: chunk partials of eps^d <target|psi> (re, im).
template <typename T>
__global__ __launch_bounds__(kChunk) void k_fid_overlap(const cx<T>* __restrict__ st, const cx<T>* __restrict__ tgt,
                                                       LaunchGeom g, double meas, double* __restrict__ part) {
  const Site r = site_here(g);
  double re = 0.0, im = 0.0;
  if (r.ok) {
    cx<double> a[5], b[5];
    load_site(st, r.d, r.s, a, b);
#pragma unroll
    for (int m = 0; m < 5; ++m) {
      const cx<T> tv = tgt[r.d.psi_off + (int64_t)m * r.d.sites + r.s];
      const cx<double> t{(double)tv.re, (double)tv.im};
      const cx<double> c = cmulc(t, a[m] + b[m]);
      re += c.re;
      im += c.im;
    }
    re *= meas;
    im *= meas;
  }
  block_sum3(re, im, 0.0, part + 3 * (int64_t)r.c);
}

// Per-instance sum of the pass-1 partials into ov[inst][3].
__global__ __launch_bounds__(kChunk) void k_fid_reduce(LaunchGeom g, const double* __restrict__ part,
                                                      double* __restrict__ ov) {
  const InstDesc d = g.inst[blockIdx.x];
  double v[3] = {0.0, 0.0, 0.0};
  for (int c = threadIdx.x; c < d.nchunks; c += kChunk) {
    v[0] += part[3 * (d.chunk_begin + c)];
    v[1] += part[3 * (d.chunk_begin + c) + 1];
  }
  block_sum3(v[0], v[1], v[2], ov + 3 * (int64_t)blockIdx.x);
}

// Pass 2: lambda_a = lambda_b = 2 eps^d <target|psi> target.
template <typename T>
__global__ __launch_bounds__(kChunk) void k_fid_grad(const cx<T>* __restrict__ tgt, cx<double>* __restrict__ lam,
                                                    LaunchGeom g, double meas, const double* __restrict__ ov) {
  const Site r = site_here(g);
  if (!r.ok) return;
  const int inst = g.chunk2inst[r.c];
  const cx<double> o{ov[3 * inst], ov[3 * inst + 1]};
#pragma unroll
  for (int m = 0; m < 5; ++m) {
    const cx<T> tv = tgt[r.d.psi_off + (int64_t)m * r.d.sites + r.s];
    const cx<double> l = (2.0 * meas) * (o * cx<double>{(double)tv.re, (double)tv.im});
    const int64_t off = r.d.qb_off + (int64_t)m * r.d.sites + r.s;
    lam[off] = l;
    lam[off + 5 * (int64_t)r.d.sites] = l;
  }
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
#define QLG_GRID dim3(g.nchunks), dim3(kChunk), 0, st

hipError_t launch_chain(int dtype, const void* in, void* out, void* rec, const LaunchGeom& g, int axis, int qb,
                        bool with_u, double tg0, double tg1, double tg25, const ExtPot& ext, double theta,
                        hipStream_t st) {
  if (g.nchunks == 0) return hipSuccess;
  if (dtype == 0)
    hipLaunchKernelGGL(k_chain<float>, QLG_GRID, (const cx<float>*)in, (cx<float>*)out, (cx<float>*)rec, g, axis,
                       qb, with_u ? 1 : 0, Angles<float>{(float)tg0, (float)tg1, (float)tg25}, ext.V, ext.mu,
                       theta);
  else
    hipLaunchKernelGGL(k_chain<double>, QLG_GRID, (const cx<double>*)in, (cx<double>*)out, (cx<double>*)rec, g,
                       axis, qb, with_u ? 1 : 0, Angles<double>{tg0, tg1, tg25}, ext.V, ext.mu, theta);
  return hipGetLastError();
}

hipError_t launch_sub_iprime_adj(const void* in, void* out, const LaunchGeom& g, int axis, int qb, hipStream_t st) {
  hipLaunchKernelGGL(k_sub_iprime_adj, QLG_GRID, (const cx<double>*)in, (cx<double>*)out, g, axis, qb);
  return hipGetLastError();
}

hipError_t launch_sub_vjp(int dtype, const void* z, void* lam, const LaunchGeom& g, double theta, double g0,
                          double g1, double g2, const ExtPot& ext, double* part, double* acc, hipStream_t st) {
  if (dtype == 0)
    hipLaunchKernelGGL(k_sub_vjp<float>, QLG_GRID, (const cx<float>*)z, (cx<double>*)lam, g, theta, g0, g1, g2,
                       ext.V, ext.mu, part);
  else
    hipLaunchKernelGGL(k_sub_vjp<double>, QLG_GRID, (const cx<double>*)z, (cx<double>*)lam, g, theta, g0, g1,
                       g2, ext.V, ext.mu, part);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_dg_accumulate, dim3(1), dim3(kDgThreads), 0, st, (const double*)part, g.nchunks, acc);
  return hipGetLastError();
}

hipError_t launch_recompute(int dtype, int axis, const void* in, void* out, void* rec, size_t rec_bytes, int first,
                            const LaunchGeom& g, const LineCounts& n, const int* pre, double tg0, double tg1,
                            double tg25, const ExtPot& ext, double theta, hipStream_t st) {
  constexpr int kWaves = kChunk / kLanes;
  const int* p = pre + axis * (g.nbatch + 1);
  auto go = [&](auto tag, auto cols) {
    using T = decltype(tag);
    constexpr int W = decltype(cols)::value;
    const Angles<T> ang{(T)tg0, (T)tg1, (T)tg25};
    const int64_t rstep = (int64_t)(rec_bytes / sizeof(cx<T>));
    if (axis == 0) {
      const dim3 grid((n.x + kWaves - 1) / kWaves), block(kChunk);
      if (ext.on())
        hipLaunchKernelGGL((k_recompute_x<T, true>), grid, block, 0, st, (const cx<T>*)in, (cx<T>*)out, (cx<T>*)rec, rstep,
                           first, g, p, n.x, ang, ext.V, ext.mu, theta);
      else
        hipLaunchKernelGGL((k_recompute_x<T, false>), grid, block, 0, st, (const cx<T>*)in, (cx<T>*)out, (cx<T>*)rec,
                           rstep, first, g, p, n.x, ang, ext.V, ext.mu, theta);
      return;
    }
    if (const int nt = n.thin[axis - 1]) {
      const dim3 grid((nt + kWaves - 1) / kWaves), block(kChunk);
      const int* pt = pre + (4 + axis) * (g.nbatch + 1);
      if (ext.on())
        hipLaunchKernelGGL((k_recompute_thin<T, true>), grid, block, 0, st, (const cx<T>*)in, (cx<T>*)out, (cx<T>*)rec,
                           rstep, g, pt, nt, axis == 2 ? 1 : 0, ang, ext.V, ext.mu, theta);
      else
        hipLaunchKernelGGL((k_recompute_thin<T, false>), grid, block, 0, st, (const cx<T>*)in, (cx<T>*)out, (cx<T>*)rec,
                           rstep, g, pt, nt, axis == 2 ? 1 : 0, ang, ext.V, ext.mu, theta);
    }
    if (n.rec[axis - 1] == 0) return;
    const dim3 grid(n.rec[axis - 1]), block(kLanes * W);
    if (ext.on())
      hipLaunchKernelGGL((k_recompute_yz<T, W, true>), grid, block, 0, st, (const cx<T>*)in, (cx<T>*)out, (cx<T>*)rec,
                         rstep, g, p, axis == 2 ? 1 : 0, ang, ext.V, ext.mu, theta);
    else
      hipLaunchKernelGGL((k_recompute_yz<T, W, false>), grid, block, 0, st, (const cx<T>*)in, (cx<T>*)out, (cx<T>*)rec,
                         rstep, g, p, axis == 2 ? 1 : 0, ang, ext.V, ext.mu, theta);
  };
  if (dtype == 0) go(0.0f, std::integral_constant<int, line_cols(0)>{});
  else go(0.0, std::integral_constant<int, line_cols(1)>{});
  return hipGetLastError();
}

hipError_t launch_adjoint(int dtype, int axis, const void* rec, size_t rec_bytes, const void* lam_in, void* lam_out,
                          const LaunchGeom& g, const LineCounts& n, const int* pre, double theta, double g0, double g1,
                          double g2, const ExtPot& ext, double* part, hipStream_t st) {
  constexpr int kWaves = kChunk / kLanes;
  auto go = [&](auto tag) {
    using T = decltype(tag);
    const int64_t rstep = (int64_t)(rec_bytes / sizeof(cx<T>));
    if (axis == 0) {
      hipLaunchKernelGGL(k_adjoint_x<T>, dim3((n.x + kWaves - 1) / kWaves), dim3(kChunk), 0, st, (const cx<T>*)rec, rstep,
                         (const cx<double>*)lam_in, (cx<double>*)lam_out, g, pre, n.x, theta, g0, g1, g2, ext.V, ext.mu,
                         part);
      return;
    }
    const int nt = n.thin[axis - 1], zp = axis == 2 ? 1 : 0;
    if (nt)
      hipLaunchKernelGGL(k_adjoint_thin<T>, dim3((nt + kWaves - 1) / kWaves), dim3(kChunk), 0, st, (const cx<T>*)rec, rstep,
                         (const cx<double>*)lam_in, (cx<double>*)lam_out, g, pre + (4 + axis) * (g.nbatch + 1), nt, zp,
                         theta, g0, g1, g2, ext.V, ext.mu, part);
    if (n.adj[axis - 1])
      hipLaunchKernelGGL(k_adjoint_yz<T>, dim3(n.adj[axis - 1]), dim3(kLanes * kAdjCols), 0, st, (const cx<T>*)rec, rstep,
                         (const cx<double>*)lam_in, (cx<double>*)lam_out, g, pre + (2 + axis) * (g.nbatch + 1), zp, theta,
                         g0, g1, g2, ext.V, ext.mu, part + 3 * (int64_t)nt);
  };
  if (dtype == 0) go(0.0f);
  else go(0.0);
  return hipGetLastError();
}

hipError_t launch_line_prefix(int dtype, const LaunchGeom& g, int* pre, hipStream_t st) {
  hipLaunchKernelGGL(k_line_prefix, dim3(1), dim3(64), 0, st, g, line_cols(dtype), pre);
  return hipGetLastError();
}

hipError_t launch_dg_reduce(const double* part, int64_t nparts, double* red, double* acc, hipStream_t st) {
  hipLaunchKernelGGL(k_dg_blocks, dim3(kDgBlocks), dim3(kChunk), 0, st, part, nparts, red);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_dg_accumulate(red, kDgBlocks, acc, st);
}

hipError_t launch_dg_accumulate(const double* part, int nparts, double* acc, hipStream_t st) {
  hipLaunchKernelGGL(k_dg_accumulate, dim3(1), dim3(kDgThreads), 0, st, part, nparts, acc);
  return hipGetLastError();
}

hipError_t launch_energy_grad(int dtype, int ndim, const void* state, void* lam, const LaunchGeom& g, double eps,
                              double g0, double g1, double g2, const ExtPot& ext, double* part, hipStream_t st) {
  if (dtype == 0)
    hipLaunchKernelGGL(k_energy_grad<float>, QLG_GRID, (const cx<float>*)state, (cx<double>*)lam, g, ndim, eps,
                       g0, g1, g2, ext.V, ext.mu, part);
  else
    hipLaunchKernelGGL(k_energy_grad<double>, QLG_GRID, (const cx<double>*)state, (cx<double>*)lam, g, ndim,
                       eps, g0, g1, g2, ext.V, ext.mu, part);
  return hipGetLastError();
}

hipError_t launch_fidelity_grad(int dtype, const void* state, const void* target, void* lam, const LaunchGeom& g,
                                double meas, double* part, double* ov, hipStream_t st) {
  if (dtype == 0)
    hipLaunchKernelGGL(k_fid_overlap<float>, QLG_GRID, (const cx<float>*)state, (const cx<float>*)target, g, meas,
                       part);
  else
    hipLaunchKernelGGL(k_fid_overlap<double>, QLG_GRID, (const cx<double>*)state, (const cx<double>*)target, g,
                       meas, part);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_fid_reduce, dim3(g.nbatch), dim3(kChunk), 0, st, g, (const double*)part, ov);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (dtype == 0)
    hipLaunchKernelGGL(k_fid_grad<float>, QLG_GRID, (const cx<float>*)target, (cx<double>*)lam, g, meas,
                       (const double*)ov);
  else
    hipLaunchKernelGGL(k_fid_grad<double>, QLG_GRID, (const cx<double>*)target, (cx<double>*)lam, g, meas,
                       (const double*)ov);
  return hipGetLastError();
}

// complex128 cotangent: canonical qubits layout <-> padded planes
__global__ __launch_bounds__(kChunk) void k_lam_in(const cx<double>* __restrict__ qb, cx<double>* __restrict__ st,
                                                  LaunchGeom g) {
  const Site r = site_here(g);
  if (!r.ok) return;
#pragma unroll
  for (int p = 0; p < 10; ++p) st[r.d.off + p * r.d.stride + r.s] = qb[r.d.qb_off + (int64_t)p * r.d.sites + r.s];
}
__global__ __launch_bounds__(kChunk) void k_lam_out(const cx<double>* __restrict__ st, cx<double>* __restrict__ qb,
                                                   LaunchGeom g) {
  const Site r = site_here(g);
  if (!r.ok) return;
#pragma unroll
  for (int p = 0; p < 10; ++p) qb[r.d.qb_off + (int64_t)p * r.d.sites + r.s] = st[r.d.off + p * r.d.stride + r.s];
}

// Adjoint of the encoding a = b = psi / 2 (Sec. III, two qubits per m_f level): psi enters
// both qubits with weight 1/2, so dL/dpsi_m = (lambda_a,m + lambda_b,m) / 2.  Canonical
// qubits layout in, canonical psi layout out, both complex128.
__global__ __launch_bounds__(kChunk) void k_encode_adj(const cx<double>* __restrict__ qb,
                                                      cx<double>* __restrict__ dpsi, LaunchGeom g) {
  const Site r = site_here(g);
  if (!r.ok) return;
#pragma unroll
  for (int m = 0; m < 5; ++m) {
    const cx<double> la = qb[r.d.qb_off + (int64_t)m * r.d.sites + r.s];
    const cx<double> lb = qb[r.d.qb_off + (int64_t)(5 + m) * r.d.sites + r.s];
    dpsi[r.d.psi_off + (int64_t)m * r.d.sites + r.s] = 0.5 * (la + lb);
  }
}

hipError_t launch_encode_adj(const void* lam, void* dpsi, const LaunchGeom& g, hipStream_t st) {
  hipLaunchKernelGGL(k_encode_adj, QLG_GRID, (const cx<double>*)lam, (cx<double>*)dpsi, g);
  return hipGetLastError();
}

hipError_t launch_lam_layout(bool to_planes, const void* src, void* dst, const LaunchGeom& g, hipStream_t st) {
  if (to_planes)
    hipLaunchKernelGGL(k_lam_in, QLG_GRID, (const cx<double>*)src, (cx<double>*)dst, g);
  else
    hipLaunchKernelGGL(k_lam_out, QLG_GRID, (const cx<double>*)src, (cx<double>*)dst, g);
  return hipGetLastError();
}

__global__ void k_zero(double* p, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0.0;
}

hipError_t launch_zero(double* p, int n, hipStream_t st) {
  hipLaunchKernelGGL(k_zero, dim3((n + 255) / 256), dim3(256), 0, st, p, n);
  return hipGetLastError();
}

}  // namespace qlg
