// lbm_runtime.hpp -- host-side pieces shared by the single-jet and batch
// runtimes: validation, descriptor setup, kernel tables, small helpers.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <utility>
#include <vector>

#include "../../include/lbm.h"
#include "lbm_device.hpp"

namespace lbmx {

#define LBM_HIP(expr)                              \
  do {                                             \
    if ((expr) != hipSuccess) return LBM_EDEVICE;  \
  } while (0)

constexpr int64_t NO_TARGET = INT64_MAX / 4;

inline int storage_bytes(int prec) { return prec == LBM_PREC_FP32 ? 4 : 2; }
inline size_t align256(size_t b) { return (b + 255) & ~size_t(255); }

// Bytes of one population buffer (13 planes with their ghost rings).
inline size_t buffer_bytes(const lbm_config *c, int prec) {
  return align256((size_t)NPOP * (size_t)layout_plane(c->nx, c->nr) * storage_bytes(prec));
}

// Buffers per jet: two, or one in place.
inline int n_buffers(int layout) { return layout == LBM_LAYOUT_SINGLE ? 1 : 2; }

// The view (see State in lbm_device.hpp) of the state after `step` steps.
inline int32_t state_view_of(int layout, int64_t step, int32_t flip) {
  if (layout == LBM_LAYOUT_SINGLE) return 2 + (int32_t)(step & 1);
  return (int32_t)((step + flip) & 1);
}

int validate_config(const lbm_config *c, bool check_precision);

// Host copy of the property tables as (M, dM) pairs at each grid point.
std::vector<float4> make_table(const lbm_config *c);

// Fill the physics fields of a descriptor (no buffers, table or inlet).
void fill_desc(JetDesc &d, const lbm_config *c);

// Inlet rows as float4 (ux, ur, T, 0); n_t == 0 gives one ambient row.
int make_inlet(const lbm_config *c, int32_t n_t, const double *ux, const double *ur,
               const double *T, std::vector<float4> &out);

// ---- kernel tables ---------------------------------------------------------
// A launch variant: block (bx, by), tile (bx * nx) x (by * ny) nodes, the
// occupancy target, the cache policy, and the steps one launch advances
// (2: the LDS-blocked two-step kernel; more: the marching kernel, with
// strips of 64 - 2 (steps - 1) columns and by tiles of march_rows() rows).
struct TileShape {
  int bx, by, ny, nx, waves, cache, steps, lds;
  const void *fn[4];  // FP32, FP16-dev, BF16-dev, FP16-dev rounded stochastically
  const void *big[4]; // instances for larger property tables (more than two steps)
  int stack_rows;     // rows of a stacked tile (0: not the stacked-row kernel)
};
const TileShape *tile_shapes(int *count);
extern const TileShape kMarch4, kMarch5, kStack[4];
// A jet of a launch.  plain: its edges are in line in the marching kernel (no
// equilibrium side, no wall at column -1).
struct LaunchJet {
  int32_t nx, nr;
  bool plain;
};
typedef std::vector<LaunchJet> LaunchJets;
template <class D>  // lbm_config or JetDesc
LaunchJet launch_jet(const D &d) {
  bool plain = d.bc[0] != LBM_BC_WALL;
  for (int s = 0; s < 4; ++s) plain = plain && d.bc[s] != LBM_BC_EQ;
  return {d.nx, d.nr, plain};
}
// The shapes of a group of launches: `shape` for as many steps as its launches
// hold, and `rest` (if any) for what is left, if that is at most rest_max
// steps; rows of a wave's tile where `shape` marches.
struct LaunchPlan {
  int shape = 0, rest = -1;
  int32_t rest_max = 0, rows = 0;
};
// The plan for jets of one storage form, and the plan of one given shape.
LaunchPlan default_plan(int prec, const LaunchJets &jets);
LaunchPlan plan_of(int shape, const LaunchJets &jets);
// Steps per launch of what a group of k steps leaves after its full launches.
int32_t rest_steps(const LaunchPlan &p, int32_t k);
// A jet's tiles in the plan's launches.
void fill_tiles(JetDesc &d, const LaunchPlan &p);
// launch(shape, offset in the group, flip toggles before it, steps) for every
// launch of a group of k steps, up to the first that fails.
template <class F>
int for_launches(const LaunchPlan &p, int32_t k, const F &launch) {
  int n, rc = 0;
  const TileShape *s = tile_shapes(&n);
  const int32_t spl = s[p.shape].steps, rest_spl = rest_steps(p, k);
  for (int32_t q = 0, m = 0; q < k && !rc; q += m) {
    const int shape = k - q < spl && k - q <= p.rest_max ? p.rest : p.shape;
    m = std::min(s[shape].steps, k - q);
    rc = launch(shape, q, group_toggles(q, k, spl, rest_spl), m);
  }
  return rc;
}
inline bool marches(const TileShape &s) { return s.big[0] != nullptr && s.stack_rows == 0; }

inline int codec_index(int prec) { return prec - LBM_PREC_FP32; }

// One launch of tile shape `shape`: the step (or pair) at step0 + koff, with
// `tog` the parity of flip toggles since the last advance and nsteps the
// steps it may take (at most the shape's); big_table: a jet's property table
// has more entries than the marching kernel holds in LDS.
int launch_step(int shape, int prec, bool big_table, int grid, hipStream_t st, const JetDesc *jets,
                const TileStart *tiles, const BatchHdr *hdr, int32_t koff, int32_t tog,
                int32_t nsteps, int32_t *flags);
// Advance after a group of delta steps in launches of spl steps and, of the
// rest, rest_spl (spl = 0: one jet, its flip toggled by `flip`).
int launch_advance(hipStream_t st, JetDesc *jets, const BatchHdr *hdr, int32_t njets_max,
                   int32_t delta, int32_t spl, int32_t rest_spl, int32_t flip = 0);
// Single-buffer step over shape 0's tile list.
int launch_aa_step(int prec, int grid, hipStream_t st, const JetDesc *jets, const TileStart *tiles,
                   const BatchHdr *hdr, int32_t koff, int32_t *flags);
// Helpers on the state after `step` steps, seen through `view`
// (state_view_of).
// Inlet entries (ux, ur, T) on the device, made the populations that enter.
int launch_inlet(hipStream_t st, float4 *rows, size_t n);
int launch_init(int prec, hipStream_t st, const JetDesc *d, const lbm_config *c, int64_t step,
                int32_t view, const float4 *state, float4 u0);
int launch_ghost_fill(int prec, hipStream_t st, const JetDesc *d, const lbm_config *c,
                      int64_t step, int32_t view);
int launch_moments(int prec, hipStream_t st, const JetDesc *d, int64_t step, int32_t view,
                   int64_t n0, int64_t n, double *out, int32_t *flags);
int launch_profiles(int prec, hipStream_t st, const JetDesc *d, const lbm_config *c,
                    int64_t step, int32_t view, double *out);
int launch_conservation(int prec, hipStream_t st, const JetDesc *d, int64_t nodes, int64_t step,
                        int32_t view, RedPartial *partial, int nblocks, RedPartial *out);
int launch_decode(int prec, hipStream_t st, const JetDesc *d, int64_t step, int32_t view,
                  int64_t e0, int64_t n, double *out);
int launch_narrow(hipStream_t st, const double *in, float *out, int64_t n, int32_t *bad);
int launch_encode(int prec, hipStream_t st, const JetDesc *d, const lbm_config *c, int64_t step,
                  int32_t view, const float *in);

// Tiles of a jet, per row in *tiles_x; rows: the marching kernel's tile_rows.
int tiles_of(int32_t nx, int32_t nr, int shape, int32_t rows, int32_t *tiles_x);
// Rows of a wave's tile for jets marched in one launch, and the time the
// marching is expected to take.
int32_t march_rows(const LaunchJets &jets, int shape, double *us = nullptr);
int device_cus();  // of the current device
bool big_table(const lbm_config *c);

// Workgroups of the step kernel of `shape` (or of the single-buffer kernel)
// that the current device holds at once: one full wave of a persistent grid.
int resident_workgroups(int shape, int prec, bool single_buffer);

// Results are written as the doubles the caller takes.  Up to PINNED_RESULT
// bytes the kernel writes them straight into pinned host memory: one launch
// and one wait (profiles of a 128 x 32 jet 20 us with the binding; device
// memory, two copies back and a conversion on the host took 48).  Larger ones
// go through device memory in pieces of at most PIECE_BYTES (any run of nodes
// or values, so that no grid needs more) and are copied to the caller's arrays at the copy engine's rate, with no pass over them on the
// host (populations out and in and fields of a 1024 x 256 jet: 3.6 ms, with
// host conversions 7.4).
constexpr size_t PINNED_RESULT = size_t(1) << 20;
constexpr size_t PIECE_BYTES = size_t(64) << 20;

// Pinned host memory that kernels write to; grows on demand.
struct Pinned {
  void *p = nullptr;
  size_t bytes = 0;
  int get(size_t need, void **out) {
    if (need > bytes) {
      release();
      if (hipHostMalloc(&p, need, hipHostMallocDefault) != hipSuccess) {
        p = nullptr;
        (void)hipGetLastError();
        return LBM_ENOMEM;
      }
      bytes = need;
    }
    *out = p;
    return LBM_OK;
  }
  void release() {
    if (p) (void)hipHostFree(p);
    p = nullptr;
    bytes = 0;
  }
};

// Simple device scratch that grows on demand.
struct Scratch {
  void *p = nullptr;
  size_t bytes = 0;
  int get(size_t need, void **out) {
    if (need > bytes) {
      if (p) (void)hipFree(p);
      p = nullptr;
      bytes = 0;
      if (hipMalloc(&p, need) != hipSuccess) {
        p = nullptr;
        (void)hipGetLastError();  // (the caller's code says it; no later call shall)
        return LBM_ENOMEM;
      }
      bytes = need;
    }
    *out = p;
    return LBM_OK;
  }
  // Room for a piece of `total` items of `item` bytes: all of them, at most
  // PIECE_BYTES, and down to 1 MiB where the device has no more to give.
  int piece(int64_t total, size_t item, void **out, int64_t *n) {
    size_t room = std::min((size_t)total * item, PIECE_BYTES);
    int rc;
    while ((rc = get(room, out)) == LBM_ENOMEM && room > PINNED_RESULT) room /= 2;
    *n = (int64_t)(room / item);
    return rc;
  }
  void release() {
    if (p) (void)hipFree(p);
    p = nullptr;
    bytes = 0;
  }
};

}  // namespace lbmx
