// Internal declarations shared by the kernels (qlg_kernels.hip) and the C ABI
// implementation (qlg_api.cpp).  Not part of the public interface.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/qlg.h"

namespace qlg {

// One lattice instance inside a batch.  Offsets are in complex elements.
struct InstDesc {
  int64_t off;        // first element of the instance's 10 qubit planes in one state copy
  int64_t psi_off;    // first element of the instance in the canonical psi layout
  int64_t qb_off;     // first element of the instance in the canonical qubits layout
  int64_t stride;     // plane stride (>= sites, multiple of 64)
  int32_t nx, ny, nz; // extents (ny = 1 in 1D, nz = 1 in 1D and 2D)
  int32_t sites;      // nx * ny * nz
  int32_t tile_begin; // first global wave tile of the fused step (3D: of its y-x pass)
  int32_t ntx, nty;   // tiles along x and bands along y (nty = 1 in 1D); 3D: ntx * nty * nz tiles
  // The band form's 3D z pass: first tile, 64-column tiles along x, bands along z (ntx_z * ntz * ny
  // tiles).  A plan of line passes has no such pass and keeps there the first group of the
  // instance in its x, y and z launches.
  union {
    struct { int32_t tile_begin_z, ntx_z, ntz; };
    struct { int32_t line[3]; };
  };
  int32_t chunk_begin;// first 256-site chunk for elementwise / reduction kernels
  int32_t nchunks;
};

constexpr int kChunk = 256;      // sites per chunk of the elementwise / reduction kernels
constexpr int kNObs = 10;        // norm_q, norm_psi, pop[5], e_kin, e_pot, spare
constexpr int kRecord = 16;      // doubles per instance in an observables record
constexpr int kLanes = 64;       // wavefront width on gfx950
constexpr int kHalo2D = 4;       // x halo of the 2D kernel (4 I' per axis per step)
constexpr int kValid2D = kLanes - 2 * kHalo2D;
constexpr int kLineHalo = 4;     // halo slots at each end of a line of the line passes
// The slots a line of n sites takes in a line pass, n + 8 with its halos, or whole 56-site windows
// where those are fewer (line_slot in qlg_lanes.hpp), and the windows (wavefronts) of nlines lines.
template <typename I>
constexpr I line_slots(I n) {
  const I v = kLanes - 2 * kLineHalo, tiles = (n + v - 1) / v * v;
  return n + 2 * kLineHalo < tiles ? n + 2 * kLineHalo : tiles;
}
template <typename I>
constexpr I line_windows(I n, I nlines) {
  const I v = kLanes - 2 * kLineHalo;
  if (n == 1) return (nlines + v - 1) / v;   // no halos: a shift along one site is none
  return (nlines * line_slots(n) - 2 * kLineHalo + v - 1) / v;
}
// Along y and z a column group's lines (one per plane) are one run of lines.  Where that run leaves
// more than half of a window empty, several neighbouring column groups share a run: how many, and the
// launch's groups for ncol column groups.  (Step of 40000 x 8 complex128 202 -> 85 us.)
template <typename I>
constexpr I line_fold(I n, I nplanes) {
  if (n == 1) return nplanes > 28 ? 1 : (kLanes - 2 * kLineHalo) / nplanes;
  return nplanes > 32 || nplanes * line_slots(n) > 32 ? 1 : kLanes / (nplanes * line_slots(n));
}
template <typename I>
constexpr I line_groups(I n, I nplanes, I ncol) {
  const I f = line_fold(n, nplanes);
  return (ncol + f - 1) / f * line_windows<I>(n, nplanes * f);
}

// The groups of one instance's x, y and z line launches: kLineTileRows windows along x, one window of
// `cols` columns along y and z.
constexpr int kLineTileRows = 8;
inline void line_launch_groups(int64_t nx, int64_t ny, int64_t nz, int cols, int64_t (&groups)[3]) {
  const int64_t ncol = (nx + cols - 1) / cols;
  groups[0] = (line_windows<int64_t>(nx, ny * nz) + kLineTileRows - 1) / kLineTileRows;
  groups[1] = line_groups<int64_t>(ny, nz, ncol);
  groups[2] = line_groups<int64_t>(nz, ny, ncol);
}
// A launch holds fewer than 2^32 threads.  (A y group's columns past a lattice of one to three columns
// are threads too: 1 x 24000 x 24000 would take 5.3e9 in complex64.)
constexpr bool launch_fits(int64_t workgroups, int threads) { return workgroups <= int64_t(UINT32_MAX) / threads; }

// The adjoint's passes along y and z over axes of up to kThinAxis sites hold whole lines, without halos,
// as rings of lanes: the windows (wavefronts) of nlines lines of n sites.
constexpr int kThinAxis = 3;
template <typename I>
constexpr I thin_windows(I n, I nlines) {
  const I lines = kLanes / n;
  return (nlines + lines - 1) / lines;
}

struct LaunchGeom {
  const InstDesc* inst;        // device [nbatch]
  const int32_t* tile2inst;    // device [ntiles]
  const int32_t* chunk2inst;   // device [nchunks]
  const int32_t* tile2inst_z;  // device [ntiles_z], 3D z pass
  int32_t ntiles, nchunks, nbatch, ntiles_z;
  int32_t nline[3];            // groups of the x, y and z line launches (0: not a plan of line passes)
};

// The psi-independent diagonal term (V(x) + mu) psi_m of the equation of motion
// (Sec. II, "Additional terms"): V per site in the canonical scalar layout (FP64,
// [instance][y][x]; nullptr: none) and a uniform mu.  theta is the interleaved
// angle eps^2 / (4 d); the plain split uses eps^2.
struct ExtPot {
  const double* V = nullptr;
  double mu = 0.0;
  double theta = 0.0;
  bool on() const { return V != nullptr || mu != 0.0; }
};

// Kernel launchers (qlg_kernels.hip).  All return the hipError_t of the launch.
// dtype: 0 = complex64, 1 = complex128.  Angles are theta*g0, theta*g1, theta*g2/5.
// ev0/ev1 (optional): events the dispatch packet itself stamps at kernel start/end.
// split: where the two qubit amplitudes of a site live: 0 = one lane holds both
// (k_step1d, 64-site tiles, steps <= 7); 1 = two wavefronts (k_step1d_pair, 64-site
// tiles, steps <= 7); 2 = two neighbouring lanes (k_step1d_lanes, 32-site tiles, steps <= 3).
constexpr int kLaneTileSites = 32;
hipError_t launch_step1d(int dtype, int steps, int split, bool plain, bool overlap, const void* in, void* out,
                         const LaunchGeom& g, double tg0, double tg1, double tg25, const ExtPot& ext,
                         double* ovpart, hipStream_t st, hipEvent_t ev0 = nullptr, hipEvent_t ev1 = nullptr);
// Part of a step that one launch of the 2D kernel runs: all four y (or z) stages, then
// the x half unless it is a z pass (kWhole); or the y half over two launches, kYFirst (the
// two stages that move qubit b) and kYSecond (the two that move qubit a, then the x half),
// each with a two-stage row pipeline: half the LDS per wavefront.
enum StepPart : int { kWhole = 0, kYFirst = 1, kYSecond = 2 };
// 2D step, or one pass of a 3D step: zpass = the four z substeps only (rows along z,
// 64-column tiles, the 3D z-pass tile table); otherwise the y and x substeps of each
// z plane.  full_factor: theta of the plain split's single U over the interleaved theta
// (4 ndim); plain_u: this pass applies that U (2D, 3D z pass).  prev (may equal out):
// the state before the step, for the overlap partials.
hipError_t launch_step2d(int dtype, bool plain, bool overlap, int tile_rows, bool zpass, bool plain_u, int part,
                         double full_factor, const void* in, void* out, const void* prev, const LaunchGeom& g,
                         double tg0, double tg1, double tg25, const ExtPot& ext, double* ovpart,
                         hipStream_t st, hipEvent_t ev0 = nullptr, hipEvent_t ev1 = nullptr);
// One axis of a 2D or 3D step as a line pass (axis 0 = x, 1 = y, 2 = z): the four substeps along
// it, from in to out (not in place).  Needs the groups of the plan of line passes and, for the
// overlap, the tile table of 8-row bands.  plain_u: this pass applies the plain split's U; prev (may
// equal out): as above, for an x pass that records the overlap.
constexpr int line_cols(int dtype) { return dtype == 0 ? 8 : 4; }            // columns of a y or z group
hipError_t launch_line(int dtype, int axis, bool plain, bool overlap, bool plain_u, double full_factor, const void* in,
                       void* out, const void* prev, const LaunchGeom& g, double tg0, double tg1, double tg25,
                       const ExtPot& ext, double* ovpart, hipStream_t st, hipEvent_t ev0 = nullptr,
                       hipEvent_t ev1 = nullptr);
hipError_t launch_set_psi(int dtype, const void* psi, void* state, const LaunchGeom& g, hipStream_t st);
hipError_t launch_get_psi(int dtype, const void* state, void* psi, const LaunchGeom& g, hipStream_t st);
hipError_t launch_set_qubits(int dtype, const void* qb, void* state, const LaunchGeom& g, hipStream_t st);
hipError_t launch_get_qubits(int dtype, const void* state, void* qb, const LaunchGeom& g, hipStream_t st);
// Per-chunk partial sums of the kNObs observables into part[nchunks][kNObs]; the
// potential energy density includes (V + mu) n.
hipError_t launch_observables(int dtype, int ndim, const void* state, const LaunchGeom& g, double g0,
                              double g1, double g2, const ExtPot& ext, double* part, hipStream_t st);
// Per-instance record rec[nbatch][kRecord] from the chunk partials, the per-tile
// overlap partials (ovpart may be null; ov_tiles > 0: of one instance's first tiles only) and a
// reference record (ref may be null).
hipError_t launch_record(const LaunchGeom& g, const double* part, const double* ovpart, int ov_tiles,
                         const double* ref, double* rec, int64_t step, hipStream_t st);

// Host checks of a parameter block shared by every entry point that takes one (no
// device call, no allocation); *msg receives a static description of the failure.
qlg_status validate_params(const qlg_params* p, const char** msg);
// Observables records (kRecord doubles per instance, written by k_reduce_record) to
// qlg_obs values; false if a record is non-finite or drifted (no allocation).
bool decode_record_values(const qlg_params& p, const double* rec, int64_t nrec, qlg_obs* out);

}  // namespace qlg
