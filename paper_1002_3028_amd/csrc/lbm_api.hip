// lbm_api.hip -- single-jet C-ABI (include/lbm.h) on one HIP device.
//
// A handle owns (or borrows) two population buffers and a stream, plus a few
// small device arrays (the descriptor, the property table, the inlet rows) and
// pinned memory for small results.  Steps are enqueued as launches of its
// plan's shapes, or as HIP graphs of the launches of k steps followed by the
// descriptor advance.
#include <algorithm>
#include <mutex>

#include "lbm_runtime.hpp"

using namespace lbmx;

namespace {
// Workgroups of the FP64 conservation reduction at most (each strides over
// nodes, so every grid fits).
constexpr int kMaxRedBlocks = 1024;
}  // namespace

// Partial sums of the no-allocation FP64 conservation reduction
// (lbm_conservation_noalloc): one per reduction workgroup, 32 KB.  Each device
// holds its own copy until the process ends.  In host code the name stands for
// no device address: host code reaches the array only through the pointer that
// hipGetSymbolAddress returns for the current device (scratch_on).
static __device__ __align__(256) RedPartial scratch[kMaxRedBlocks];

namespace {
// The handle's small results, in pinned host memory that kernels write to
// directly; the profiles (2 (nx + nr) doubles) of a jet of up to 4096 columns
// and rows together follow (larger ones get memory when they are asked for:
// pinning 320 KB took a third of a handle's creation).
struct HostBlock {
  RedPartial total;   // of the conservation reduction
  int32_t unstable;   // the steps' instability flag
  int32_t bad_input;  // a value handed in was not finite
};
constexpr size_t kProfilesAt = 256;
constexpr size_t kProfilesHeld = size_t(64) << 10;
size_t profile_bytes(const lbm_config &c) { return 2 * sizeof(double) * ((size_t)c.nx + c.nr); }
static_assert(sizeof(HostBlock) <= kProfilesAt, "host block");
}  // namespace

struct lbm_handle {
  int device = 0;
  lbm_config cfg{};
  std::vector<double> nu_tab, al_tab;
  int prec = LBM_PREC_FP32;
  int layout = LBM_LAYOUT_TWO_BUFFERS;
  void *buf = nullptr;
  bool own_buf = false;
  hipStream_t stream = nullptr;
  bool own_stream = false;
  // device arrays
  JetDesc *d_desc = nullptr;
  int32_t *d_flag = nullptr;  // host->unstable
  float4 *d_table = nullptr;
  float4 *d_inlet = nullptr;
  Scratch scratch, piece;
  HostBlock *host = nullptr;
  Pinned result;  // fields and populations of up to PINNED_RESULT bytes
  JetDesc desc{};
  int64_t step = 0;  // steps done
  int32_t flip = 0;  // state after s steps in buf[(s + flip) & 1]
  // step0 and flip held by the device descriptor: they may lag step and flip
  // (directly launched steps pass the difference as koff and tog; a graph,
  // whose arguments are fixed, first brings them up to date)
  int64_t base = 0;
  int32_t dflip = 0;
  LaunchPlan plan;
  bool unstable = false;
  int32_t graph_k = 0;
  hipGraphExec_t gexec = nullptr;
  int32_t gexec_k = 0, gexec_shape = -1;
};

namespace {

int32_t view_of(const lbm_handle *h, int64_t step) {
  return state_view_of(h->layout, step, h->flip);
}

int upload_desc(lbm_handle *h) {
  h->base = h->step;
  h->dflip = h->flip;
  h->desc.step0 = h->base;
  h->desc.flip = h->flip;
  LBM_HIP(hipMemcpyAsync(h->d_desc, &h->desc, sizeof(JetDesc), hipMemcpyHostToDevice, h->stream));
  LBM_HIP(hipStreamSynchronize(h->stream));
  return LBM_OK;
}

int set_plan(lbm_handle *h, const LaunchPlan &plan) {
  h->plan = plan;
  fill_tiles(h->desc, plan);
  return upload_desc(h);
}

// Workgroups of a launch of one of the plan's shapes: one per tile.
int grid_of(const lbm_handle *h, int shape) {
  int n;
  const int32_t tiles = tile_shapes(&n)[shape].steps > 2 ? h->desc.mtiles : h->desc.ntiles;
  return (tiles + 7) / 8 * 8;
}

void drop_graph(lbm_handle *h) {
  if (h->gexec) (void)hipGraphExecDestroy(h->gexec);
  h->gexec = nullptr;
  h->gexec_k = 0;
  h->gexec_shape = -1;
}

// Sync, then fold the device instability flag into the sticky state.
int sync_and_check(lbm_handle *h) {
  LBM_HIP(hipStreamSynchronize(h->stream));
  LBM_HIP(hipGetLastError());
  if (h->host->unstable) h->unstable = true;
  return h->unstable ? LBM_EUNSTABLE : LBM_OK;
}

// (the caller has synchronised the stream)
int clear_flag(lbm_handle *h) {
  h->host->unstable = 0;
  h->unstable = false;
  return LBM_OK;
}

void release(lbm_handle *h) {
  if (!h) return;
  if (h->stream) (void)hipStreamSynchronize(h->stream);
  drop_graph(h);
  h->scratch.release();
  h->piece.release();
  h->result.release();
  if (h->host) (void)hipHostFree(h->host);
  if (h->d_desc) (void)hipFree(h->d_desc);
  if (h->d_table) (void)hipFree(h->d_table);
  if (h->d_inlet) (void)hipFree(h->d_inlet);
  if (h->own_buf && h->buf) (void)hipFree(h->buf);
  if (h->own_stream && h->stream) (void)hipStreamDestroy(h->stream);
  delete h;
}

int upload_inlet(lbm_handle *h, const std::vector<float4> &rows, int32_t n_t) {
  float4 *p = nullptr;
  LBM_HIP(hipStreamSynchronize(h->stream));
  if (hipMalloc(&p, rows.size() * sizeof(float4)) != hipSuccess) return LBM_ENOMEM;
  if (hipMemcpy(p, rows.data(), rows.size() * sizeof(float4), hipMemcpyHostToDevice) !=
      hipSuccess) {
    (void)hipFree(p);
    return LBM_EDEVICE;
  }
  if (h->d_inlet) (void)hipFree(h->d_inlet);
  h->d_inlet = p;
  h->desc.inlet = p;
  h->desc.n_t = n_t;
  int rc = launch_inlet(h->stream, p, rows.size());
  if (!rc) rc = upload_desc(h);
  if (rc) return rc;
  // the inlet ghosts of the current buffer follow the new rows
  if ((rc = launch_ghost_fill(h->prec, h->stream, h->d_desc, &h->cfg, h->step, view_of(h, h->step)))) return rc;
  LBM_HIP(hipStreamSynchronize(h->stream));
  return LBM_OK;
}

int create_common(const lbm_config *cfg, void *dev_buf, size_t bytes, void *stream,
                  lbm_handle **out) {
  if (!out) return LBM_EINVAL;
  *out = nullptr;
  int rc = validate_config(cfg, true);
  if (rc) return rc;
  lbm_handle *h = new (std::nothrow) lbm_handle();
  if (!h) return LBM_ENOMEM;
  h->cfg = *cfg;
  if (cfg->table_n > 0) {
    h->nu_tab.assign(cfg->nu_mult, cfg->nu_mult + cfg->table_n);
    h->al_tab.assign(cfg->alpha_mult, cfg->alpha_mult + cfg->table_n);
    h->cfg.nu_mult = h->nu_tab.data();
    h->cfg.alpha_mult = h->al_tab.data();
  }
  h->prec = cfg->precision;
  h->layout = cfg->layout;
  if (hipGetDevice(&h->device) != hipSuccess) {
    release(h);
    return LBM_EDEVICE;
  }
  const size_t one = buffer_bytes(cfg, h->prec);
  const size_t total = n_buffers(h->layout) * one;
  if (dev_buf) {
    if (bytes < total || ((uintptr_t)dev_buf & 255)) {
      release(h);
      return LBM_EINVAL;
    }
    h->buf = dev_buf;
    h->stream = (hipStream_t)stream;
  } else {
    if (hipMalloc(&h->buf, total) != hipSuccess) {
      release(h);
      return LBM_ENOMEM;
    }
    h->own_buf = true;
    if (hipStreamCreateWithFlags(&h->stream, hipStreamNonBlocking) != hipSuccess) {
      release(h);
      return LBM_EDEVICE;
    }
    h->own_stream = true;
  }
  std::vector<float4> table = make_table(&h->cfg);
  bool ok = hipMalloc(&h->d_desc, sizeof(JetDesc)) == hipSuccess &&
            hipHostMalloc((void **)&h->host,
                          kProfilesAt + (profile_bytes(*cfg) <= kProfilesHeld ? profile_bytes(*cfg) : 0),
                          hipHostMallocDefault) == hipSuccess &&
            hipHostGetDevicePointer((void **)&h->d_flag, &h->host->unstable, 0) == hipSuccess &&
            hipMalloc(&h->d_table, table.size() * sizeof(float4)) == hipSuccess;
  if (!ok) {
    release(h);
    return LBM_ENOMEM;
  }
  *h->host = HostBlock{};
  ok = hipMemcpy(h->d_table, table.data(), table.size() * sizeof(float4),
                 hipMemcpyHostToDevice) == hipSuccess;
  if (!ok) {
    release(h);
    return LBM_EDEVICE;
  }
  JetDesc &d = h->desc;
  fill_desc(d, &h->cfg);
  d.buf[0] = h->buf;
  d.buf[1] = h->layout == LBM_LAYOUT_SINGLE ? h->buf : (char *)h->buf + one;
  d.table = h->d_table;
  d.target = NO_TARGET;
  d.slot = 0;
  std::vector<float4> rows;
  make_inlet(&h->cfg, 0, nullptr, nullptr, nullptr, rows);
  if ((rc = upload_inlet(h, rows, 1)) ||
      (rc = set_plan(h, h->layout == LBM_LAYOUT_SINGLE
                            ? LaunchPlan{0}
                            : default_plan(h->prec, {launch_jet(*cfg)})))) {
    release(h);
    return rc;
  }
  // both buffers at the initial equilibrium, each with its ghost ring (the
  // constant ghosts of equilibrium sides are only ever written here; the
  // single buffer's step rewrites them itself)
  const float4 u0 =
      make_float4((float)cfg->rho0, (float)cfg->ux0, (float)cfg->ur0, (float)cfg->T0);
  for (int64_t q = n_buffers(h->layout) - 1; q >= 0 && !rc; --q) {
    const int32_t v = view_of(h, q);
    rc = launch_init(h->prec, h->stream, h->d_desc, &h->cfg, q, v, nullptr, u0);
    if (!rc) rc = launch_ghost_fill(h->prec, h->stream, h->d_desc, &h->cfg, q, v);
  }
  if (rc || hipStreamSynchronize(h->stream) != hipSuccess) {
    release(h);
    return rc ? rc : LBM_EDEVICE;
  }
  *out = h;
  return LBM_OK;
}

// Steps one launch of the handle's shape advances (the one shape of a single
// buffer takes one).
int32_t steps_per_launch(const lbm_handle *h) {
  int nsh;
  return tile_shapes(&nsh)[h->plan.shape].steps;
}

// Flip toggles of a group of k steps.
int32_t toggles_of(const lbm_handle *h, int32_t k) {
  return group_toggles(k, k, steps_per_launch(h), rest_steps(h->plan, k));
}

// The launches of a group of k steps on `st`, starting koff0 steps past the
// descriptor's step0 with its flip toggled by tog0; then, if `advance`, the
// descriptor advance (koff0 = tog0 = 0 then).
int enqueue_group(lbm_handle *h, int32_t k, hipStream_t st, int32_t koff0 = 0, int32_t tog0 = 0,
                  bool advance = true) {
  int rc = for_launches(h->plan, k, [&](int shape, int32_t q, int32_t tog, int32_t m) {
    if (h->layout == LBM_LAYOUT_SINGLE)
      return launch_aa_step(h->prec, grid_of(h, shape), st, h->d_desc, nullptr, nullptr, koff0 + q,
                            h->d_flag);
    return launch_step(shape, h->prec, big_table(&h->cfg), grid_of(h, shape), st, h->d_desc,
                       nullptr, nullptr, koff0 + q, tog0 ^ tog, m, h->d_flag);
  });
  if (!rc && advance)
    rc = launch_advance(st, h->d_desc, nullptr, 1, k, steps_per_launch(h), rest_steps(h->plan, k));
  return rc;
}

// Capture k steps as one graph (enqueue_group's launches).
int capture_group(lbm_handle *h, int32_t k) {
  hipGraph_t g;
  LBM_HIP(hipStreamBeginCapture(h->stream, hipStreamCaptureModeThreadLocal));
  const int crc = enqueue_group(h, k, h->stream);
  const hipError_t e = hipStreamEndCapture(h->stream, &g);
  if (crc || e != hipSuccess) return crc ? crc : LBM_EDEVICE;
  const hipError_t ei = hipGraphInstantiate(&h->gexec, g, nullptr, nullptr, 0);
  (void)hipGraphDestroy(g);
  if (ei != hipSuccess) {
    h->gexec = nullptr;
    return LBM_EDEVICE;
  }
  h->gexec_k = k;
  h->gexec_shape = h->plan.shape;
  return LBM_OK;
}

// Capture and upload the graph of the handle's group size and shape now, so
// that the first lbm_step that replays it pays no capture or instantiation.
int prepare_graph(lbm_handle *h) {
  if (h->graph_k <= 0) return LBM_OK;
  if (h->gexec && h->gexec_k == h->graph_k && h->gexec_shape == h->plan.shape) return LBM_OK;
  drop_graph(h);
  const int rc = capture_group(h, h->graph_k);
  if (rc) return rc;
  // (an optimisation only: the graph also uploads itself at its first launch)
  (void)hipGraphUpload(h->gexec, h->stream);
  // One dry replay, so that the first lbm_step does not pay the graph's
  // first launch: with the descriptor's target at its step0 every tile is
  // skipped and the advance leaves step0 and flip as they are, so the state
  // does not change.
  h->desc.target = h->step;  // (upload_desc sets step0 to the step count)
  int rc2 = upload_desc(h);
  if (!rc2 && hipGraphLaunch(h->gexec, h->stream) != hipSuccess) rc2 = LBM_EDEVICE;
  if (!rc2 && hipStreamSynchronize(h->stream) != hipSuccess) rc2 = LBM_EDEVICE;
  h->desc.target = NO_TARGET;
  const int rc3 = upload_desc(h);
  return rc2 ? rc2 : rc3;
}

// Brings the device descriptor's step0 and flip to the host's.
int catch_up(lbm_handle *h) {
  if (h->base == h->step && h->dflip == h->flip) return LBM_OK;
  const int rc = launch_advance(h->stream, h->d_desc, nullptr, 1, (int32_t)(h->step - h->base), 0,
                                0, h->flip ^ h->dflip);
  if (rc) return rc;
  h->base = h->step;
  h->dflip = h->flip;
  return LBM_OK;
}

int launch_steps(lbm_handle *h, int64_t n) {
  const int32_t spl = steps_per_launch(h);
  int rc;
  while (n > 0) {
    const bool graph = h->graph_k > 0 && n >= h->graph_k;
    // (the lag is kept below 2^30 steps, so koff fits its 32 bits)
    if ((graph || h->step - h->base > (1 << 30)) && (rc = catch_up(h))) return rc;
    if (graph) {
      if (!h->gexec || h->gexec_k != h->graph_k || h->gexec_shape != h->plan.shape) {
        drop_graph(h);
        if ((rc = capture_group(h, h->graph_k))) return rc;
      }
      LBM_HIP(hipGraphLaunch(h->gexec, h->stream));
      h->step += h->graph_k;
      h->base += h->graph_k;
      h->flip ^= toggles_of(h, h->graph_k);
      h->dflip ^= toggles_of(h, h->graph_k);
      n -= h->graph_k;
    } else {
      // the rest (fewer steps than a graph holds) as directly launched
      // steps: a graph's launches, offset from the descriptor, and no
      // advance (the device starts on the first kernel while the host
      // enqueues the rest)
      const int32_t m = (int32_t)std::min<int64_t>(n, (1 << 20) / spl * spl);
      if ((rc = enqueue_group(h, m, h->stream, (int32_t)(h->step - h->base),
                              h->flip ^ h->dflip, false)))
        return rc;
      h->step += m;
      h->flip ^= toggles_of(h, m);
      n -= m;
    }
  }
  return LBM_OK;
}

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
RedPartial *g_scratch_ptr[kMaxDevices] = {};

// The device address of `scratch` on `device`, resolved once per device with
// that device current.
int scratch_on(int device, RedPartial **out) {
  if (device < 0 || device >= kMaxDevices) return LBM_EDEVICE;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[device]) {
    int cur = -1;
    LBM_HIP(hipGetDevice(&cur));
    if (cur != device) LBM_HIP(hipSetDevice(device));
    void *p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (cur != device) (void)hipSetDevice(cur);
    if (e != hipSuccess || !p) return LBM_EDEVICE;
    g_scratch_ptr[device] = (RedPartial *)p;
  }
  *out = g_scratch_ptr[device];
  return LBM_OK;
}

// Reduction workgroups of the conservation kernels for a grid (the same
// count in both conservation entry points, so their sums agree bit for bit).
int red_blocks(const lbm_handle *h) {
  const int64_t nodes = (int64_t)h->cfg.nx * h->cfg.nr;
  return (int)std::min<int64_t>(kMaxRedBlocks, (nodes + RED_THREADS - 1) / RED_THREADS);
}

// Of the values e0 .. e0 + n - 1 of all populations: how many are f's (the
// first nine planes; g's follow).
int64_t f_part(int64_t e0, int64_t n, int64_t nodes) {
  return std::max<int64_t>(0, std::min(9 * nodes, e0 + n) - e0);
}

// Both conservation entry points: reduce into `part` (nblocks partials), the
// total into the host block, and wait.
int conservation_into(lbm_handle *h, RedPartial *part, int nblocks, double *mass3d,
                      double *energy3d) {
  const int64_t nodes = (int64_t)h->cfg.nx * h->cfg.nr;
  int rc;
  if ((rc = launch_conservation(h->prec, h->stream, h->d_desc, nodes, h->step,
                                view_of(h, h->step), part, nblocks, &h->host->total)))
    return rc;
  const int st = sync_and_check(h);
  if (st == LBM_EDEVICE) return st;
  const RedPartial r = h->host->total;
  *mass3d = r.mass;
  *energy3d = r.energy;
  if (r.bad != 0.0) h->unstable = true;
  return h->unstable ? LBM_EUNSTABLE : LBM_OK;
}

}  // namespace

extern "C" {

int lbm_bytes_required(const lbm_config *cfg, size_t *bytes) {
  if (!bytes) return LBM_EINVAL;
  const int rc = validate_config(cfg, true);
  if (rc) return rc;
  *bytes = n_buffers(cfg->layout) * buffer_bytes(cfg, cfg->precision);
  return LBM_OK;
}

int lbm_create(const lbm_config *cfg, lbm_handle **out) {
  return create_common(cfg, nullptr, 0, nullptr, out);
}

int lbm_create_in(const lbm_config *cfg, void *dev_buf, size_t bytes, void *hip_stream,
                  lbm_handle **out) {
  if (!dev_buf) return out ? (*out = nullptr, LBM_EINVAL) : LBM_EINVAL;
  return create_common(cfg, dev_buf, bytes, hip_stream, out);
}

void lbm_destroy(lbm_handle *h) { release(h); }

int lbm_set_inlet(lbm_handle *h, int32_t n_t, const double *ux, const double *ur,
                  const double *T) {
  if (!h || n_t < 1) return LBM_EINVAL;
  std::vector<float4> rows;
  const int rc = make_inlet(&h->cfg, n_t, ux, ur, T, rows);
  if (rc) return rc;
  return upload_inlet(h, rows, n_t);
}

int lbm_step(lbm_handle *h, int64_t n_steps) {
  if (!h || n_steps < 0) return LBM_EINVAL;
  if (h->unstable) return LBM_EUNSTABLE;
  return launch_steps(h, n_steps);
}

int64_t lbm_step_count(const lbm_handle *h) { return h ? h->step : -1; }

void *lbm_stream(const lbm_handle *h) { return h ? (void *)h->stream : nullptr; }

int lbm_sync(lbm_handle *h) {
  if (!h) return LBM_EINVAL;
  return sync_and_check(h);
}

int lbm_set_graph_steps(lbm_handle *h, int32_t k) {
  if (!h || k < 0) return LBM_EINVAL;
  LBM_HIP(hipStreamSynchronize(h->stream));
  h->graph_k = k;
  if (k == 0) drop_graph(h);
  return prepare_graph(h);
}

int lbm_set_tile_shape(lbm_handle *h, int32_t index) {
  if (!h) return LBM_EINVAL;
  LBM_HIP(hipStreamSynchronize(h->stream));
  // (a refused index leaves the handle as it is: the device's descriptor may
  // lag behind the step count, and base and dflip say by how much)
  int n;
  tile_shapes(&n);
  if (index < 0 || index >= n || (h->layout == LBM_LAYOUT_SINGLE && index != 0)) return LBM_EINVAL;
  const int rc = set_plan(h, plan_of(index, {launch_jet(h->cfg)}));
  if (rc) return rc;
  drop_graph(h);
  return prepare_graph(h);
}

int lbm_moments(lbm_handle *h, double *rho, double *ux, double *ur, double *T) {
  if (!h) return LBM_EINVAL;
  const int64_t nodes = (int64_t)h->cfg.nx * h->cfg.nr;
  double *const to[4] = {rho, ux, ur, T};
  const int32_t view = view_of(h, h->step);
  int rc;
  void *p;
  if (4 * nodes * sizeof(double) <= PINNED_RESULT) {
    if ((rc = h->result.get(4 * nodes * sizeof(double), &p))) return rc;
    if ((rc = launch_moments(h->prec, h->stream, h->d_desc, h->step, view, 0, nodes, (double *)p,
                             h->d_flag)))
      return rc;
    const int st = sync_and_check(h);
    if (st == LBM_EDEVICE) return st;
    for (int q = 0; q < 4; ++q)
      if (to[q]) std::memcpy(to[q], (double *)p + q * nodes, nodes * sizeof(double));
    return st;
  }
  int64_t most;
  if ((rc = h->piece.piece(nodes, 4 * sizeof(double), &p, &most))) return rc;
  for (int64_t n0 = 0; n0 < nodes; n0 += most) {
    const int64_t n = std::min(most, nodes - n0);
    if ((rc = launch_moments(h->prec, h->stream, h->d_desc, h->step, view, n0, n, (double *)p,
                             h->d_flag)))
      return rc;
    LBM_HIP(hipStreamSynchronize(h->stream));
    for (int q = 0; q < 4; ++q)
      if (to[q])
        LBM_HIP(hipMemcpy(to[q] + n0, (double *)p + q * n, n * sizeof(double),
                          hipMemcpyDeviceToHost));
  }
  return sync_and_check(h);
}

int lbm_profiles(lbm_handle *h, double *ux_axis, double *T_axis, double *ux_exit,
                 double *T_exit) {
  if (!h) return LBM_EINVAL;
  const size_t nx = h->cfg.nx, nr = h->cfg.nr;
  void *v = (char *)h->host + kProfilesAt;
  int rc = profile_bytes(h->cfg) <= kProfilesHeld ? LBM_OK : h->result.get(profile_bytes(h->cfg), &v);
  if (rc) return rc;
  if ((rc = launch_profiles(h->prec, h->stream, h->d_desc, &h->cfg, h->step, view_of(h, h->step),
                            (double *)v)))
    return rc;
  const double *p = (const double *)v;
  const int st = sync_and_check(h);
  if (st == LBM_EDEVICE) return st;
  if (ux_axis) std::memcpy(ux_axis, p, nx * sizeof(double));
  if (T_axis) std::memcpy(T_axis, p + nx, nx * sizeof(double));
  if (ux_exit) std::memcpy(ux_exit, p + 2 * nx, nr * sizeof(double));
  if (T_exit) std::memcpy(T_exit, p + 2 * nx + nr, nr * sizeof(double));
  return st;
}

int lbm_conservation(lbm_handle *h, double *mass3d, double *energy3d) {
  if (!h || !mass3d || !energy3d) return LBM_EINVAL;
  const int nblocks = red_blocks(h);
  void *p;
  const int rc = h->scratch.get(nblocks * sizeof(RedPartial), &p);
  if (rc) return rc;
  return conservation_into(h, (RedPartial *)p, nblocks, mass3d, energy3d);
}

int lbm_conservation_noalloc(lbm_handle *h, double *mass3d, double *energy3d) {
  if (!h || !mass3d || !energy3d) return LBM_EINVAL;
  const int nblocks = red_blocks(h);
  if (nblocks > kMaxRedBlocks) return LBM_EINVAL;
  RedPartial *part;
  const int rc = scratch_on(h->device, &part);
  if (rc) return rc;
  return conservation_into(h, part, nblocks, mass3d, energy3d);
}

int lbm_set_state(lbm_handle *h, const double *rho, const double *ux, const double *ur,
                  const double *T) {
  if (!h || !rho || !ux || !ur || !T) return LBM_EINVAL;
  const int64_t nodes = (int64_t)h->cfg.nx * h->cfg.nr;
  std::vector<float4> s((size_t)nodes);
  for (int64_t n = 0; n < nodes; ++n) {
    if (!(rho[n] > 0.0) || !std::isfinite(rho[n]) || !std::isfinite(ux[n]) ||
        !std::isfinite(ur[n]) || !std::isfinite(T[n]))
      return LBM_EINVAL;
    s[n] = make_float4((float)rho[n], (float)ux[n], (float)ur[n], (float)T[n]);
  }
  void *p;
  int rc = h->scratch.get(nodes * sizeof(float4), &p);
  if (rc) return rc;
  LBM_HIP(hipStreamSynchronize(h->stream));
  LBM_HIP(hipMemcpy(p, s.data(), nodes * sizeof(float4), hipMemcpyHostToDevice));
  if ((rc = launch_init(h->prec, h->stream, h->d_desc, &h->cfg, h->step, view_of(h, h->step),
                        (const float4 *)p, make_float4(0, 0, 0, 0))))
    return rc;
  if ((rc = launch_ghost_fill(h->prec, h->stream, h->d_desc, &h->cfg, h->step, view_of(h, h->step)))) return rc;
  LBM_HIP(hipStreamSynchronize(h->stream));
  return clear_flag(h);
}

int lbm_get_populations(lbm_handle *h, double *f, double *g) {
  if (!h) return LBM_EINVAL;
  const int64_t nodes = (int64_t)h->cfg.nx * h->cfg.nr;
  const size_t one = nodes * sizeof(double);
  const int32_t view = view_of(h, h->step);
  int rc;
  void *p;
  if (NPOP * one <= PINNED_RESULT) {
    if ((rc = h->result.get(NPOP * one, &p))) return rc;
    if ((rc = launch_decode(h->prec, h->stream, h->d_desc, h->step, view, 0, NPOP * nodes,
                            (double *)p)))
      return rc;
    const int st = sync_and_check(h);
    if (st == LBM_EDEVICE) return st;
    if (f) std::memcpy(f, p, 9 * one);
    if (g) std::memcpy(g, (double *)p + 9 * nodes, 4 * one);
    return st;
  }
  int64_t most;
  if ((rc = h->piece.piece(NPOP * nodes, sizeof(double), &p, &most))) return rc;
  for (int64_t e0 = 0; e0 < NPOP * nodes; e0 += most) {
    const int64_t n = std::min(most, NPOP * nodes - e0);
    if ((rc = launch_decode(h->prec, h->stream, h->d_desc, h->step, view, e0, n, (double *)p)))
      return rc;
    LBM_HIP(hipStreamSynchronize(h->stream));
    const int64_t nf = f_part(e0, n, nodes);
    if (nf > 0 && f)
      LBM_HIP(hipMemcpy(f + e0, p, nf * sizeof(double), hipMemcpyDeviceToHost));
    if (n > nf && g)
      LBM_HIP(hipMemcpy(g + (e0 + nf - 9 * nodes), (double *)p + nf, (n - nf) * sizeof(double),
                        hipMemcpyDeviceToHost));
  }
  return sync_and_check(h);
}

int lbm_set_populations(lbm_handle *h, const double *f, const double *g, int64_t step) {
  if (!h || !f || !g || step < 0) return LBM_EINVAL;
  const int64_t nodes = (int64_t)h->cfg.nx * h->cfg.nr;
  const size_t one = nodes * sizeof(double);
  // the values as floats in device memory, checked on the way; the state is
  // touched only if all are finite
  void *v, *p;
  int rc = h->scratch.get(NPOP * nodes * sizeof(float), &v);
  if (rc) return rc;
  LBM_HIP(hipStreamSynchronize(h->stream));
  h->host->bad_input = 0;
  if (NPOP * one <= PINNED_RESULT) {
    if ((rc = h->result.get(NPOP * one, &p))) return rc;
    std::memcpy(p, f, 9 * one);
    std::memcpy((double *)p + 9 * nodes, g, 4 * one);
    if ((rc = launch_narrow(h->stream, (const double *)p, (float *)v, NPOP * nodes,
                            &h->host->bad_input)))
      return rc;
  } else {
    int64_t most;
    if ((rc = h->piece.piece(NPOP * nodes, sizeof(double), &p, &most))) return rc;
    for (int64_t e0 = 0; e0 < NPOP * nodes; e0 += most) {
      const int64_t n = std::min(most, NPOP * nodes - e0), nf = f_part(e0, n, nodes);
      LBM_HIP(hipStreamSynchronize(h->stream));  // (the last piece has been read)
      if (nf > 0) LBM_HIP(hipMemcpy(p, f + e0, nf * sizeof(double), hipMemcpyHostToDevice));
      if (n > nf)
        LBM_HIP(hipMemcpy((double *)p + nf, g + (e0 + nf - 9 * nodes), (n - nf) * sizeof(double),
                          hipMemcpyHostToDevice));
      if ((rc = launch_narrow(h->stream, (const double *)p, (float *)v + e0, n,
                              &h->host->bad_input)))
        return rc;
    }
  }
  LBM_HIP(hipStreamSynchronize(h->stream));
  if (h->host->bad_input) return LBM_EINVAL;
  h->step = step;
  h->base = step;
  if ((rc = upload_desc(h))) return rc;
  if ((rc = launch_encode(h->prec, h->stream, h->d_desc, &h->cfg, step, view_of(h, step),
                           (const float *)v)))
    return rc;
  if ((rc = launch_ghost_fill(h->prec, h->stream, h->d_desc, &h->cfg, step, view_of(h, step)))) return rc;
  LBM_HIP(hipStreamSynchronize(h->stream));
  return clear_flag(h);
}

const char *lbm_strerror(int code) {
  switch (code) {
    case LBM_OK: return "ok";
    case LBM_EINVAL: return "invalid argument or configuration";
    case LBM_ENOMEM: return "out of memory or budget";
    case LBM_EUNSTABLE: return "unstable: non-finite value or non-positive density";
    case LBM_EDEVICE: return "HIP runtime error";
    case LBM_ESTATE: return "call not valid in the current state";
    default: return "unknown error";
  }
}

}  // extern "C"
