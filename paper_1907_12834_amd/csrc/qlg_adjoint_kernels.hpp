// Launchers of the adjoint kernels (qlg_adjoint_kernels.hip).
#pragma once

#include "qlg_internal.hpp"

namespace qlg {

// One link of the recorded forward chain: z = I'_{axis,qb}(in) (z = in when axis < 0),
// rec <- z when rec is not null, out <- U(z) with angles (tg0, tg1, tg25) when with_u, else z.
// ext (V, mu) with theta: the potential's per-site phase theta (V + mu) inside U.
hipError_t launch_chain(int dtype, const void* in, void* out, void* rec, const LaunchGeom& g, int axis, int qb,
                        bool with_u, double tg0, double tg1, double tg25, const ExtPot& ext, double theta,
                        hipStream_t st);
hipError_t launch_sub_iprime_adj(const void* in, void* out, const LaunchGeom& g, int axis, int qb, hipStream_t st);
// lam <- (dU)^H lam at z; acc[0..2] += dL/dg (part: nchunks x 3 doubles of scratch)
hipError_t launch_sub_vjp(int dtype, const void* z, void* lam, const LaunchGeom& g, double theta, double g0,
                          double g1, double g2, const ExtPot& ext, double* part, double* acc, hipStream_t st);
// Interleaved split: line passes (one axis, 0 = x, 1 = y, 2 = z, of one step per launch).
constexpr int kAdjCols = 4;        // columns per y or z group of the pull-back (complex128: 64 bytes)
constexpr int kLinePrefixes = 7;   // instance tables of nbatch + 1 ints each (launch_line_prefix)
struct LineCounts {
  int x;         // x windows (wavefronts)
  int rec[2];    // y, z groups of the recompute (line_cols(dtype) columns of a window)
  int adj[2];    // y, z groups of the pull-back (kAdjCols columns)
  int thin[2];   // y, z windows of the instances whose axis has at most kThinAxis sites (no groups)
};
// The recompute of one axis: z_0 = in, z_{k+1} = I'_k U(z_k), out = z_4; rec + k rec_bytes receives
// z_k for k >= first (x, and y and z of up to kThinAxis sites: as a state copy; other y and z: along
// the lines; first = 0 but for x).
hipError_t launch_recompute(int dtype, int axis, const void* in, void* out, void* rec, size_t rec_bytes, int first,
                            const LaunchGeom& g, const LineCounts& n, const int* pre, double tg0, double tg1,
                            double tg25, const ExtPot& ext, double theta, hipStream_t st);
// The pull-back through one axis at the records of the same layout; dg partials per wavefront into
// part[n.x][3] (x) or part[n.thin[axis - 1] + kAdjCols n.adj[axis - 1]][3] (no accumulation).
hipError_t launch_adjoint(int dtype, int axis, const void* rec, size_t rec_bytes, const void* lam_in, void* lam_out,
                          const LaunchGeom& g, const LineCounts& n, const int* pre, double theta, double g0, double g1,
                          double g2, const ExtPot& ext, double* part, hipStream_t st);
// pre[kLinePrefixes][nbatch + 1]: the instances' first x window, y and z groups and thin windows
// (device table)
hipError_t launch_line_prefix(int dtype, const LaunchGeom& g, int* pre, hipStream_t st);
// acc[0..2] += sum of nparts consecutive 3-vectors of part (fixed order)
hipError_t launch_dg_accumulate(const double* part, int nparts, double* acc, hipStream_t st);
// The same for many partials: kDgBlocks workgroups sum contiguous ranges of part into
// red[kDgBlocks][3] (fixed order), then one workgroup adds those to acc in order.
constexpr int kDgBlocks = 256;
hipError_t launch_dg_reduce(const double* part, int64_t nparts, double* red, double* acc, hipStream_t st);
// energy objective: canonical complex128 cotangent + chunk partials [nchunks][4]
hipError_t launch_energy_grad(int dtype, int ndim, const void* state, void* lam, const LaunchGeom& g, double eps,
                              double g0, double g1, double g2, const ExtPot& ext, double* part, hipStream_t st);
// fidelity objective: partials [nchunks][3], per-instance overlaps ov[nbatch][3]
hipError_t launch_fidelity_grad(int dtype, const void* state, const void* target, void* lam, const LaunchGeom& g,
                                double meas, double* part, double* ov, hipStream_t st);
hipError_t launch_lam_layout(bool to_planes, const void* src, void* dst, const LaunchGeom& g, hipStream_t st);
// dpsi = (lambda_a + lambda_b) / 2: adjoint of the encoding, complex128 canonical layouts
hipError_t launch_encode_adj(const void* lam, void* dpsi, const LaunchGeom& g, hipStream_t st);
hipError_t launch_zero(double* p, int n, hipStream_t st);

}  // namespace qlg
