// lbm_kernels.hip -- kernel instantiations, launch helpers and the host-side
// configuration checks shared by the single-jet and batch runtimes.
#include "lbm_kernels.hpp"
#include "lbm_runtime.hpp"

namespace lbmx {

// ---- kernels of no storage form ----------------------------------------------
// Moves every jet's step0 by delta (clamped at the target); ends a captured
// group of steps so that the same graph serves the next group.  The group's
// launches took spl steps each and the last ones up to rest_spl:
// group_toggles of them swapped the roles of a jet's buffers.  spl = 0: one
// jet, whose flip is toggled by `flip`.
__global__ void advance_kernel(JetDesc *__restrict__ jets, const BatchHdr *__restrict__ hdr,
                               int32_t delta, int32_t spl, int32_t rest_spl, int32_t flip) {
  const int32_t q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q < (hdr ? hdr->njets : 1)) {
    const int64_t s0 = jets[q].step0, tg = jets[q].target;
    const int64_t s = s0 + delta < tg ? s0 + delta : tg;
    jets[q].flip ^= spl > 0 ? group_toggles(s - s0, delta, spl, rest_spl) : flip;
    jets[q].step0 = s;
  }
}

// Inlet entries (ux, ur, T, 0) made the populations that enter the domain
// there: the equilibria of links 1, 5, 8 and +x at density 1.
__global__ void inlet_kernel(float4 *__restrict__ rows, int64_t n) {
  const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= n) return;
  const float4 v = rows[q];
  rows[q] = make_float4(feq_link(1, 1.0f, v.x, v.y), feq_link(5, 1.0f, v.x, v.y),
                        feq_link(8, 1.0f, v.x, v.y), geq_link(0, v.z, v.x, v.y));
}

// Reduces the conservation kernel's partial sums the same way.
__global__ __launch_bounds__(RED_THREADS) void reduce_partials_kernel(
    const RedPartial *__restrict__ partial, int32_t n, RedPartial *__restrict__ out) {
  double m = 0.0, e = 0.0, bad = 0.0;
  for (int q = threadIdx.x; q < n; q += RED_THREADS) {
    m += partial[q].mass;
    e += partial[q].energy;
    bad += partial[q].bad;
  }
  __shared__ double sm[RED_THREADS], se[RED_THREADS], sb[RED_THREADS];
  sm[threadIdx.x] = m;
  se[threadIdx.x] = e;
  sb[threadIdx.x] = bad;
  __syncthreads();
  for (int w = RED_THREADS / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) {
      sm[threadIdx.x] += sm[threadIdx.x + w];
      se[threadIdx.x] += se[threadIdx.x + w];
      sb[threadIdx.x] += sb[threadIdx.x + w];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) out[0] = RedPartial{sm[0], se[0], sb[0], 0.0};
}

// Plain streaming copy, 16 B per lane per iteration.
__global__ __launch_bounds__(256) void copy_kernel(const float4 *__restrict__ src,
                                                   float4 *__restrict__ dst, int64_t n) {
  for (int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x; q < n; q += (int64_t)gridDim.x * 256)
    dst[q] = src[q];
}

// Doubles as floats; *bad is set if one is not finite.
__global__ __launch_bounds__(256) void narrow_kernel(const double *__restrict__ in,
                                                     float *__restrict__ out, int64_t n,
                                                     int32_t *__restrict__ bad) {
  bool ok = true;
  for (int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x; q < n; q += (int64_t)gridDim.x * 256) {
    const double v = in[q];
    out[q] = (float)v;
    ok &= fabs(v) < __builtin_inf();
  }
  if (!ok) *bad = 1;
}

// ---- validation (same rules the paper's setting implies: tau > 1/2 so that
// nu, alpha > 0; Pr_t > 0; a symmetry axis only at r = 0) ------------------
static bool side_ok(int side, int bc) {
  switch (side) {
    case 0: return bc == BC_INLET || bc == BC_PERIODIC || bc == BC_WALL || bc == BC_EQ;
    case 1: return bc == BC_OUTFLOW || bc == BC_PERIODIC || bc == BC_WALL || bc == BC_EQ;
    case 2: return bc == BC_AXIS || bc == BC_FREESLIP || bc == BC_WALL || bc == BC_EQ;
    default: return bc == BC_FREESLIP || bc == BC_WALL || bc == BC_EQ;
  }
}

int validate_config(const lbm_config *c, bool check_precision) {
  if (!c || c->abi_version != LBM_ABI_VERSION) return LBM_EINVAL;
  if (c->nx < 2 || c->nr < 2) return LBM_EINVAL;
  // every byte offset inside a buffer must fit the 32-bit buffer offsets
  if ((int64_t)NPOP * layout_plane(c->nx, c->nr) * 4 >= ((int64_t)1 << 31)) return LBM_EINVAL;
  if (!(c->tau_nu > 0.5) || !(c->tau_alpha > 0.5) || !std::isfinite(c->tau_nu) ||
      !std::isfinite(c->tau_alpha))
    return LBM_EINVAL;
  if (!(c->pr_t > 0.0) || !(c->cs >= 0.0) || !(c->delta > 0.0) || !std::isfinite(c->cs) ||
      !std::isfinite(c->delta) || !std::isfinite(c->pr_t))
    return LBM_EINVAL;
  if (!std::isfinite(c->r0) || c->r0 < 0.0 || !std::isfinite(c->body_force_x)) return LBM_EINVAL;
  if (c->table_n != 0) {
    if (c->table_n < 2 || !c->nu_mult || !c->alpha_mult || !(c->t_hi > c->t_lo) ||
        !std::isfinite(c->t_lo) || !std::isfinite(c->t_hi))
      return LBM_EINVAL;
    for (int q = 0; q < c->table_n; ++q)
      if (!(c->nu_mult[q] > 0.0) || !(c->alpha_mult[q] > 0.0) || !std::isfinite(c->nu_mult[q]) ||
          !std::isfinite(c->alpha_mult[q]))
        return LBM_EINVAL;
  }
  for (int s = 0; s < 4; ++s)
    if (!side_ok(s, c->bc[s])) return LBM_EINVAL;
  if ((c->bc[0] == BC_PERIODIC) != (c->bc[1] == BC_PERIODIC)) return LBM_EINVAL;
  if (c->bc[2] == BC_AXIS && c->r0 != 0.0) return LBM_EINVAL;
  for (int s = 0; s < 4; ++s)
    if (c->bc[s] == BC_EQ &&
        (!(c->eq_state[s][0] > 0.0) || !std::isfinite(c->eq_state[s][0]) ||
         !std::isfinite(c->eq_state[s][1]) || !std::isfinite(c->eq_state[s][2]) ||
         !std::isfinite(c->eq_state[s][3])))
      return LBM_EINVAL;
  if (c->hoop != 0 && c->hoop != 1) return LBM_EINVAL;
  if (c->layout != LBM_LAYOUT_TWO_BUFFERS && c->layout != LBM_LAYOUT_SINGLE) return LBM_EINVAL;
  if (!(c->rho0 > 0.0) || !std::isfinite(c->rho0) || !std::isfinite(c->ux0) ||
      !std::isfinite(c->ur0) || !std::isfinite(c->T0))
    return LBM_EINVAL;
  if (check_precision) {
    if (c->precision != LBM_PREC_FP32 && c->precision != LBM_PREC_FP16DEV &&
        c->precision != LBM_PREC_BF16DEV && c->precision != LBM_PREC_FP16SR)
      return LBM_EINVAL;
    if (c->precision != LBM_PREC_FP32 &&
        (!std::isfinite(c->rho_ref) || !std::isfinite(c->g_ref)))
      return LBM_EINVAL;
  }
  return LBM_OK;
}

std::vector<float4> make_table(const lbm_config *c) {
  std::vector<float4> t;
  if (c->table_n == 0) {
    t.assign(2, make_float4(1.f, 0.f, 1.f, 0.f));
    return t;
  }
  const int n = c->table_n;
  t.resize(n);
  for (int q = 0; q < n; ++q) {
    const double a = c->nu_mult[q], b = c->alpha_mult[q];
    const double da = q + 1 < n ? c->nu_mult[q + 1] - a : 0.0;
    const double db = q + 1 < n ? c->alpha_mult[q + 1] - b : 0.0;
    t[q] = make_float4((float)a, (float)da, (float)b, (float)db);
  }
  return t;
}

void fill_desc(JetDesc &d, const lbm_config *c) {
  d.nx = c->nx;
  d.nr = c->nr;
  d.pitch = layout_pitch(c->nx);
  d.plane = layout_plane(c->nx, c->nr);
  d.table_n = c->table_n == 0 ? 2 : c->table_n;
  d.hoop = c->hoop;
  for (int s = 0; s < 4; ++s) {
    d.bc[s] = c->bc[s];
    d.wallT[s] = (float)c->wall_T[s];
    for (int q = 0; q < 4; ++q) d.eq[s][q] = (float)c->eq_state[s][q];
  }
  d.r0 = (float)c->r0;
  d.nu0 = (float)((c->tau_nu - 0.5) / 3.0);
  d.alpha0 = (float)((c->tau_alpha - 0.5) / 2.0);
  const double csd = c->cs * c->delta;
  d.c18 = (float)(18.0 * csd * csd);
  d.inv_prt = (float)(1.0 / c->pr_t);
  d.G = (float)c->body_force_x;
  d.t_lo = c->table_n == 0 ? 0.f : (float)c->t_lo;
  d.t_scale = c->table_n == 0 ? 0.f : (float)((c->table_n - 1) / (c->t_hi - c->t_lo));
  d.rho_ref = (float)c->rho_ref;
  d.g4_ref = (float)(0.25 * c->g_ref);
  d.flip = 0;
  d.tiles_x = d.mtiles_x = 1;
  d.ntiles = d.mtiles = 0;
  d.tile_rows = 0;
  d.tile_steps = 1;
  d.cus = device_cus();
}

int make_inlet(const lbm_config *c, int32_t n_t, const double *ux, const double *ur,
               const double *T, std::vector<float4> &out) {
  if (n_t < 0) return LBM_EINVAL;
  if (n_t == 0) {
    out.assign((size_t)c->nr, make_float4(0.f, 0.f, (float)c->T0, 0.f));
    return LBM_OK;
  }
  if (!ux || !ur || !T) return LBM_EINVAL;
  const size_t n = (size_t)n_t * (size_t)c->nr;
  out.resize(n);
  for (size_t q = 0; q < n; ++q) {
    if (!std::isfinite(ux[q]) || !std::isfinite(ur[q]) || !std::isfinite(T[q])) return LBM_EINVAL;
    out[q] = make_float4((float)ux[q], (float)ur[q], (float)T[q], 0.f);
  }
  return LBM_OK;
}

// ---- tile shapes -------------------------------------------------------------
#define LBM_SHAPE(BX, BY, NY, NX, W, CP)                                         \
  {BX, BY, NY, NX, W, CP, 1, 0,                                                  \
   {(const void *)&step_kernel<CodecF32, BX, BY, NY, NX, W, CP>,                 \
    (const void *)&step_kernel<CodecF16, BX, BY, NY, NX, W, CP>,                 \
    (const void *)&step_kernel<CodecBF16, BX, BY, NY, NX, W, CP>,                \
    (const void *)&step_kernel<CodecF16SR, BX, BY, NY, NX, W, CP>}, {}}
// two steps per launch: 64 x TY tiles, block 64 x NW (lds: the LDS image of
// FP32 storage; the 16-bit forms keep theirs in the storage type, half that)
#define LBM_PAIR(TY, NW, W, CP)                                                  \
  {64, NW, (TY) / (NW), 1, W, CP, 2, (NPOP - ((CP) & 8 ? 1 : 0)) * ((TY) + 2) * PAIR_W * 4, \
   {(const void *)&pair_kernel<CodecF32, TY, NW, W, CP>,                         \
    (const void *)&pair_kernel<CodecF16, TY, NW, W, CP>,                         \
    (const void *)&pair_kernel<CodecBF16, TY, NW, W, CP>,                        \
    (const void *)&pair_kernel<CodecF16SR, TY, NW, W, CP>}, {}}

static const std::vector<TileShape> &shapes() {
  static const std::vector<TileShape> table = {
    LBM_SHAPE(64, 4, 1, 1, 1, 0),  LBM_SHAPE(128, 2, 1, 1, 1, 0), LBM_SHAPE(256, 1, 1, 1, 1, 0),
    LBM_SHAPE(64, 8, 1, 1, 1, 0),  LBM_SHAPE(64, 4, 2, 1, 1, 0),  LBM_SHAPE(64, 4, 1, 2, 1, 0),
    LBM_SHAPE(128, 2, 1, 2, 1, 0), LBM_SHAPE(64, 4, 1, 1, 1, 1),  LBM_SHAPE(64, 4, 1, 1, 1, 2),
    LBM_SHAPE(64, 4, 1, 1, 1, 3),  LBM_SHAPE(64, 4, 2, 1, 1, 1),  LBM_SHAPE(64, 4, 2, 1, 1, 3),
    LBM_SHAPE(128, 2, 1, 1, 1, 1), LBM_SHAPE(64, 8, 2, 1, 1, 0),
    LBM_PAIR(8, 4, 4, 0),          LBM_PAIR(12, 4, 3, 0),         LBM_PAIR(16, 4, 2, 0),
    LBM_PAIR(8, 4, 4, 1),          LBM_PAIR(12, 4, 3, 1),         LBM_PAIR(8, 4, 4, 4),
    LBM_PAIR(12, 4, 3, 4),         LBM_PAIR(8, 4, 4, 5),          LBM_PAIR(16, 4, 2, 4),
    LBM_PAIR(8, 4, 5, 8),          LBM_PAIR(8, 4, 5, 9),          LBM_PAIR(8, 4, 5, 12),
    LBM_PAIR(12, 4, 3, 8),
    // 16-bit storage: a 64 x 16 tile's image (28.5 KB) leaves room for five
    // workgroups per CU, and the 1 024 tiles of a 2048 x 512 jet then fit
    // the resident workgroups at once (no second, partly idle round)
    LBM_PAIR(16, 4, 5, 8),         LBM_PAIR(16, 4, 5, 12),
    // up to four steps per launch, waves marching up strips
    kMarch4,
    // four to eight steps per launch, a wave per row
    kStack[0], kStack[1], kStack[2], kStack[3],
    // up to five steps per launch, for states that the caches do not hold
    kMarch5,
  };
  return table;
}
#undef LBM_SHAPE
#undef LBM_PAIR

constexpr int TWO_STEP = 23;  // the 64 x 8 tile with f_0 in registers: the fastest in FP32

const TileShape *tile_shapes(int *count) {
  *count = (int)shapes().size();
  return shapes().data();
}
// The default shape, by the time a launch is expected to take per step (us,
// measured; LaunchJets are the jets of one launch).
//
// Few nodes: stacked rows, as many steps per launch as leave one workgroup a
// CU (a launch of one round takes 9.1, 10.0, 10.8 and 12.1 us for 4, 5, 6
// and 8 steps in FP32, so 2.3 to 1.5 us per step, 16-bit forms 2.6 to 1.8
// and, with stochastic rounding, 3.1 to 2.2; the one-step kernel takes 3.6
// to 4.4 on the same grids).  A second round costs as much again: in FP32
// that still pays (1024 x 256: 4.5 us per step, marching 5.5, one step 6.1),
// in 16-bit storage it does not (768 x 192: FP16 4.4 against 4.45, with
// stochastic rounding 5.1 against 4.7).
// Many nodes: FP32 marches (against the two-step kernel 7.3 / 9.0 on 1500 x
// 375, 9.4 / 13.1 on 2048 x 512, 32 / 57 on 4096 x 1024).  FP16 and BF16
// move half the bytes and pay a rounding per level: a march takes 1.19 and
// 1.25 times FP32's, and the line to the one-step kernel lies where its time,
// fitted over the node count, is longer, from half a million nodes (FP16, one
// step / march: 7.4 / 8.2 on 1400 x 350, 8.2 / 8.4 on 1536 x 384, 8.1 / 7.6 on
// 1024 x 512, 12.1 / 10.9 on 2048 x 512, 33 / 29.6 on 4096 x 1024, 97 / 62 on
// 6000 x 1500; BF16 8.3 / 8.9, 8.1 / 8.0, 12.2 /
// 11.5, 33 / 31.7 and 98 / 66).  Cohorts of several jets run two at a time
// and hide each other's launches, which is what a march saves in 16 bits: they
// keep one step per launch (64 uneven jets: FP16 130 against 130 GLUPS, BF16
// 128 against 121).
// Stochastic rounding also needs a key per level (1.55 times FP32's march):
// it marches only where one step per launch waits for HBM (2048 x 512 12.9 /
// 14.3, 4096 x 1024 33.5 / 40.6, 6000 x 1500 97 / 84).
// Both buffers of a jet in the 256 MiB of the Infinity Cache: four steps per
// launch; beyond, FP32 takes five, since a launch then waits for HBM (four /
// five steps: 15.1 / 15.8 us per step on 3000 x 700, 32.1 / 29.9 on 4096 x
// 1024, 70 / 58 on 6000 x 1500; six 17.4, 34.3 and 64; FP16 62 / 63 on the
// last).
// A march waits for its slowest wave, and the strips of an equilibrium side
// or of a wall at column -1 read or write the ring row by row: such jets take
// the two-step kernel in FP32 (2048 x 512 with four equilibrium sides: 13.7
// against 17.0 us per step, 1024 x 512 between two walls: 8.6 against 8.8)
// and one step in 16 bits (12.4 / 17.6, 7.7 / 10.1).
//
// Property tables that LDS does not hold (more than 256 entries) make a march
// wait for its gathers: 9.6 us per step against 8.8 on 2048 x 512, 15.5
// against 14.1 on 3000 x 700, 37.9 against 28.7 on 4096 x 1024 (FP16 11.0
// against 10.5, 18.3 against 17.2, 30.2 against 28.5).  That is still less
// than any other shape takes on such a jet (the two-step kernel 12.7, 20.6 and
// 56.2, FP16 one step 12.0, 18.7 and 32.1; small grids take the same time with
// either), so the table's size does not enter the rule.  One such jet among 16
// of 512 x 128 takes its cohort from 11.6 to 12.9 us per step (two steps per
// launch 14.8).
//
// A launch of fewer steps than its shape holds costs more than its share (a
// march of one step on 2048 x 512 takes 23.4 us, of two 30.3), so that a
// group's last steps, or a caller's single ones, take another shape where that
// is faster: after a march in FP32 one or two steps the two-step kernel (18.3
// and 25.7 us; 4096 x 1024: 87 and 113 against 114 and 140; three steps 44.0
// against 40.1, so they stay), in 16 bits the one-step kernel (FP16, one to
// three steps on 2048 x 512: 11.9, 23.6, 35.5 against 23.5, 33.2, 46.1; beyond
// the Infinity Cache two: 6000 x 1500, three steps 294 against 274); after
// stacked rows one step the one-step kernel (128 x 32: 4.2 against 4.7; two
// steps 7.7 against 5.7), after two rounds of them the two-step kernel (768 x
// 192, one and two steps: 6.5 and 9.7 against 8.2 and 10.1).
LaunchPlan default_plan(int prec, const LaunchJets &jets) {
  const bool fp32 = prec == LBM_PREC_FP32;
  const int cus = device_cus();
  int n, best = 0;
  const TileShape *s = tile_shapes(&n);
  double best_t = 1e30;
  int64_t nodes = 0, best_rounds = 0;
  int32_t best_rows = 0;
  bool plain = true;
  for (const auto &j : jets) nodes += (int64_t)j.nx * j.nr, plain = plain && j.plain;
  const bool cached = 2 * NPOP * (fp32 ? 4 : 2) * nodes <= int64_t(256) << 20;
  // (what a march of 16-bit storage has to stay below, and its weight)
  const double one_step =
      fp32 ? 1e30
      : jets.size() > 1 || nodes < 500000 ? 0.0
      : cached ? std::min(3.4 + 7.8e-6 * nodes, 5.0 + 6.6e-6 * nodes)
               : 10.7e-6 * nodes;
  const double weight = fp32                       ? 1.0
                        : prec == LBM_PREC_FP16DEV ? 1.19
                        : prec == LBM_PREC_BF16DEV ? 1.25
                                                   : 1.55;
  for (int q = 0; q < n; ++q) {
    const int k = s[q].steps;
    int64_t rounds = 0;
    int32_t rows = 0;
    double t;
    if (s[q].stack_rows) {
      int64_t wg = 0;
      for (const auto &j : jets) wg += tiles_of(j.nx, j.nr, q, 0, nullptr);
      rounds = (wg + cus - 1) / cus;
      if (!fp32 && rounds > 1) continue;
      t = (2.3 + rounds * (k <= 6 ? 3.0 + k : 10.5)) / k;
    } else if (fp32 && !plain && q == TWO_STEP) {
      t = 4.3 + 8.9e-6 * nodes;
    } else if (marches(s[q]) && plain && one_step > 0.0 && k == (fp32 && !cached ? 5 : 4)) {
      double us;
      rows = march_rows(jets, q, &us);
      t = (5.5 + weight * us) / k;
      if (t >= one_step) continue;
    } else {
      continue;
    }
    if (t < best_t) best = q, best_t = t, best_rounds = rounds, best_rows = rows;
  }
  LaunchPlan plan{best, -1, 0, best_rows};
  if (s[best].steps > 2) {
    const bool pair = fp32 && best_rounds != 1;
    plan.rest = pair ? TWO_STEP : 0;
    plan.rest_max = pair ? 2 : best_rounds ? 1 : cached || prec == LBM_PREC_FP16SR ? 3 : 2;
  }
  return plan;
}

int32_t rest_steps(const LaunchPlan &p, int32_t k) {
  const int32_t spl = shapes()[p.shape].steps, rest = k % spl;
  return rest > 0 && rest <= p.rest_max ? shapes()[p.rest].steps : spl;
}

LaunchPlan plan_of(int shape, const LaunchJets &jets) {
  return {shape, -1, 0, marches(shapes()[shape]) ? march_rows(jets, shape) : 0};
}

void fill_tiles(JetDesc &d, const LaunchPlan &p) {
  d.tile_rows = p.rows;
  d.tile_steps = shapes()[p.shape].steps;
  d.tiles_x = d.mtiles_x = 1;
  d.ntiles = d.mtiles = 0;
  for (const int q : {p.rest, p.shape}) {
    if (q < 0) continue;
    if (shapes()[q].steps > 2) d.mtiles = tiles_of(d.nx, d.nr, q, p.rows, &d.mtiles_x);
    else d.ntiles = tiles_of(d.nx, d.nr, q, 0, &d.tiles_x);
  }
}

int tiles_of(int32_t nx, int32_t nr, int shape, int32_t rows, int32_t *tiles_x) {
  const TileShape &s = shapes()[shape];
  const int w = s.steps > 2 ? s.bx - 2 * (s.steps - 1) : s.bx * s.nx;
  const int h = s.stack_rows ? s.stack_rows : s.by * (marches(s) ? rows : s.ny);
  const int tx = (nx + w - 1) / w;
  const int ty = (nr + h - 1) / h;
  if (tiles_x) *tiles_x = tx;
  return tx * ty;
}

// Rows of a wave's tile, for jets marched in one launch.  A wave of R rows
// does K R + K (K - 1) collisions per column (its own and the halo rows that
// its neighbours compute too), so tall tiles waste less, but the launch lasts
// as long as the busiest CU: two workgroups of four waves share a CU (one
// wave per SIMD leaves a third of the issue slots empty: 0.41 us per
// collision of a wave alone, 0.31 us with two on the SIMD), and a third has
// to wait.  The height with the least work on the busiest CU wins: on
// 2048 x 512 ten rows (468 workgroups, 9.4 us per step), not nine (540
// workgroups, 12.4) or nineteen (252 workgroups, 11.4).
int32_t march_rows(const LaunchJets &jets, int shape, double *us) {
  const TileShape &s = shapes()[shape];
  const int w = s.bx - 2 * (s.steps - 1), k = s.steps;
  const int cus = device_cus();
  int32_t nr_max = 0;
  for (const auto &j : jets) nr_max = std::max(nr_max, j.nr);
  int32_t best = 1;
  double best_t = 0.0;
  for (int32_t r = 1; r <= (nr_max + s.by - 1) / s.by; ++r) {
    const int32_t h = s.by * r;
    int64_t wg = 0;
    for (const auto &j : jets) wg += (int64_t)((j.nx + w - 1) / w) * ((j.nr + h - 1) / h);
    const int64_t per_cu = (wg + cus - 1) / cus;
    const double t = (double)(k * r + k * (k - 1)) * (0.62 * (per_cu / 2) + 0.41 * (per_cu % 2));
    if (r == 1 || t < best_t) best = r, best_t = t;
    if (per_cu == 1) break;  // (taller tiles only take longer)
  }
  if (us) *us = best_t;
  return best;
}

int device_cus() {
  int cus = 0, dev = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      cus <= 0)
    return 256;
  return cus;
}

int launch_step(int shape, int prec, bool big_table, int grid, hipStream_t st,
                const JetDesc *jets, const TileStart *tiles, const BatchHdr *hdr, int32_t koff,
                int32_t tog, int32_t nsteps, int32_t *flags) {
  const TileShape &s = shapes()[shape];
  const void *fn = (big_table && s.big[0] ? s.big : s.fn)[codec_index(prec)];
  void *args[] = {(void *)&jets, (void *)&tiles, (void *)&hdr,   (void *)&koff,
                  (void *)&tog,  (void *)&nsteps, (void *)&flags};
  LBM_HIP(hipLaunchKernel(fn, dim3(grid), dim3(s.bx, s.by), args, 0, st));
  return LBM_OK;
}

static const void *aa_fn(int prec) {
  static const void *fn[4] = {(const void *)&aa_kernel<CodecF32>,
                              (const void *)&aa_kernel<CodecF16>,
                              (const void *)&aa_kernel<CodecBF16>,
                              (const void *)&aa_kernel<CodecF16SR>};
  return fn[codec_index(prec)];
}

int resident_workgroups(int shape, int prec, bool single_buffer) {
  const TileShape &s = shapes()[shape];
  const void *fn = single_buffer ? aa_fn(prec) : s.fn[codec_index(prec)];
  const int threads = single_buffer ? 256 : s.bx * s.by;
  int per_cu = 0, cus = 0, dev = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, threads, 0) != hipSuccess ||
      hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      per_cu <= 0 || cus <= 0)
    return 2048;
  return (per_cu * cus + 7) / 8 * 8;
}

int launch_aa_step(int prec, int grid, hipStream_t st, const JetDesc *jets, const TileStart *tiles,
                   const BatchHdr *hdr, int32_t koff, int32_t *flags) {
  int32_t tog = 0, nsteps = 1;
  void *args[] = {(void *)&jets, (void *)&tiles, (void *)&hdr,   (void *)&koff,
                  (void *)&tog,  (void *)&nsteps, (void *)&flags};
  LBM_HIP(hipLaunchKernel(aa_fn(prec), dim3(grid), dim3(64, 4), args, 0, st));
  return LBM_OK;
}

int launch_advance(hipStream_t st, JetDesc *jets, const BatchHdr *hdr, int32_t njets_max,
                   int32_t delta, int32_t spl, int32_t rest_spl, int32_t flip) {
  const int blocks = (njets_max + 63) / 64;
  hipLaunchKernelGGL(advance_kernel, dim3(blocks), dim3(64), 0, st, jets, hdr, delta, spl,
                     rest_spl, flip);
  LBM_HIP(hipGetLastError());
  return LBM_OK;
}

int launch_inlet(hipStream_t st, float4 *rows, size_t n) {
  hipLaunchKernelGGL(inlet_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, rows,
                     (int64_t)n);
  LBM_HIP(hipGetLastError());
  return LBM_OK;
}

template <class C>
static void init_t(hipStream_t st, const JetDesc *d, const lbm_config *c, int64_t step, int32_t view,
                   const float4 *state, float4 u0) {
  hipLaunchKernelGGL(init_kernel<C>, dim3((c->nx + 255) / 256, c->nr), dim3(256), 0, st, d,
                     step, view, state, u0);
}
int launch_init(int prec, hipStream_t st, const JetDesc *d, const lbm_config *c, int64_t step, int32_t view,
                const float4 *state, float4 u0) {
  if (prec == LBM_PREC_FP32) init_t<CodecF32>(st, d, c, step, view, state, u0);
  else if (prec == LBM_PREC_FP16DEV) init_t<CodecF16>(st, d, c, step, view, state, u0);
  else if (prec == LBM_PREC_FP16SR) init_t<CodecF16SR>(st, d, c, step, view, state, u0);
  else init_t<CodecBF16>(st, d, c, step, view, state, u0);
  LBM_HIP(hipGetLastError());
  return LBM_OK;
}

template <class C>
static void ghost_t(hipStream_t st, const JetDesc *d, const lbm_config *c, int64_t step, int32_t view) {
  const int n = 2 * (c->nx + 2) + 2 * c->nr;
  hipLaunchKernelGGL(ghost_fill_kernel<C>, dim3((n + 255) / 256), dim3(256), 0, st, d, step, view);
}
int launch_ghost_fill(int prec, hipStream_t st, const JetDesc *d, const lbm_config *c,
                      int64_t step, int32_t view) {
  if (prec == LBM_PREC_FP32) ghost_t<CodecF32>(st, d, c, step, view);
  else if (prec == LBM_PREC_FP16DEV) ghost_t<CodecF16>(st, d, c, step, view);
  else if (prec == LBM_PREC_FP16SR) ghost_t<CodecF16SR>(st, d, c, step, view);
  else ghost_t<CodecBF16>(st, d, c, step, view);
  LBM_HIP(hipGetLastError());
  return LBM_OK;
}

int launch_moments(int prec, hipStream_t st, const JetDesc *d,
                   int64_t step, int32_t view, int64_t n0, int64_t n, double *out,
                   int32_t *flags) {
  const auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, d, step, view,
                       (int32_t)n0, (int32_t)n, out, flags);
  };
  if (prec == LBM_PREC_FP32) go(moments_kernel<CodecF32>);
  else if (prec == LBM_PREC_FP16DEV) go(moments_kernel<CodecF16>);
  else if (prec == LBM_PREC_FP16SR) go(moments_kernel<CodecF16SR>);
  else go(moments_kernel<CodecBF16>);
  LBM_HIP(hipGetLastError());
  return LBM_OK;
}

template <class C>
static void profiles_t(hipStream_t st, const JetDesc *d, const lbm_config *c, int64_t step, int32_t view,
                       double *out) {
  const int n = c->nx + c->nr;
  hipLaunchKernelGGL(profiles_kernel<C>, dim3((n + 255) / 256), dim3(256), 0, st, d, step, view, out);
}
int launch_profiles(int prec, hipStream_t st, const JetDesc *d, const lbm_config *c,
                    int64_t step, int32_t view, double *out) {
  if (prec == LBM_PREC_FP32) profiles_t<CodecF32>(st, d, c, step, view, out);
  else if (prec == LBM_PREC_FP16DEV) profiles_t<CodecF16>(st, d, c, step, view, out);
  else if (prec == LBM_PREC_FP16SR) profiles_t<CodecF16SR>(st, d, c, step, view, out);
  else profiles_t<CodecBF16>(st, d, c, step, view, out);
  LBM_HIP(hipGetLastError());
  return LBM_OK;
}

template <class C>
static void cons_t(hipStream_t st, const JetDesc *d, int64_t step, int32_t view, RedPartial *partial,
                   int nblocks) {
  hipLaunchKernelGGL(conservation_kernel<C>, dim3(nblocks), dim3(RED_THREADS), 0, st, d, step, view,
                     partial);
}
int launch_conservation(int prec, hipStream_t st, const JetDesc *d, int64_t nodes, int64_t step, int32_t view,
                        RedPartial *partial, int nblocks, RedPartial *out) {
  (void)nodes;
  if (prec == LBM_PREC_FP32) cons_t<CodecF32>(st, d, step, view, partial, nblocks);
  else if (prec == LBM_PREC_FP16DEV) cons_t<CodecF16>(st, d, step, view, partial, nblocks);
  else if (prec == LBM_PREC_FP16SR) cons_t<CodecF16SR>(st, d, step, view, partial, nblocks);
  else cons_t<CodecBF16>(st, d, step, view, partial, nblocks);
  LBM_HIP(hipGetLastError());
  hipLaunchKernelGGL(reduce_partials_kernel, dim3(1), dim3(RED_THREADS), 0, st, partial, nblocks,
                     out);
  LBM_HIP(hipGetLastError());
  return LBM_OK;
}

int launch_decode(int prec, hipStream_t st, const JetDesc *d, int64_t step, int32_t view,
                  int64_t e0, int64_t n, double *out) {
  const auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, d, step, view,
                       (int32_t)e0, (int32_t)n, out);
  };
  if (prec == LBM_PREC_FP32) go(decode_kernel<CodecF32>);
  else if (prec == LBM_PREC_FP16DEV) go(decode_kernel<CodecF16>);
  else if (prec == LBM_PREC_FP16SR) go(decode_kernel<CodecF16SR>);
  else go(decode_kernel<CodecBF16>);
  LBM_HIP(hipGetLastError());
  return LBM_OK;
}

int launch_narrow(hipStream_t st, const double *in, float *out, int64_t n, int32_t *bad) {
  const int blocks = (int)std::min<int64_t>((n + 255) / 256, 256 * 16);
  hipLaunchKernelGGL(narrow_kernel, dim3(blocks), dim3(256), 0, st, in, out, n, bad);
  LBM_HIP(hipGetLastError());
  return LBM_OK;
}

template <class C>
static void encode_t(hipStream_t st, const JetDesc *d, const lbm_config *c, int64_t step, int32_t view,
                     const float *in) {
  hipLaunchKernelGGL(encode_kernel<C>, dim3((c->nx + 255) / 256, c->nr, NPOP), dim3(256), 0, st,
                     d, step, view, in);
}
int launch_encode(int prec, hipStream_t st, const JetDesc *d, const lbm_config *c, int64_t step, int32_t view,
                  const float *in) {
  if (prec == LBM_PREC_FP32) encode_t<CodecF32>(st, d, c, step, view, in);
  else if (prec == LBM_PREC_FP16DEV) encode_t<CodecF16>(st, d, c, step, view, in);
  else if (prec == LBM_PREC_FP16SR) encode_t<CodecF16SR>(st, d, c, step, view, in);
  else encode_t<CodecBF16>(st, d, c, step, view, in);
  LBM_HIP(hipGetLastError());
  return LBM_OK;
}

}  // namespace lbmx

extern "C" int lbm_probe_copy(void *dst, const void *src, size_t bytes, void *hip_stream) {
  if (!dst || !src || bytes % 16 != 0) return LBM_EINVAL;
  const int64_t n = (int64_t)(bytes / 16);
  const int blocks = (int)std::min<int64_t>((n + 255) / 256, 256 * 32);
  if (n == 0) return LBM_OK;
  hipLaunchKernelGGL(lbmx::copy_kernel, dim3(blocks), dim3(256), 0, (hipStream_t)hip_stream,
                     (const float4 *)src, (float4 *)dst, n);
  return hipGetLastError() == hipSuccess ? LBM_OK : LBM_EDEVICE;
}

extern "C" int lbm_tile_shape_count(void) {
  int n;
  lbmx::tile_shapes(&n);
  return n;
}

extern "C" int lbm_tile_shape(int32_t index, int32_t *bx, int32_t *by, int32_t *ny,
                              int32_t *nx) {
  int n;
  const lbmx::TileShape *s = lbmx::tile_shapes(&n);
  if (index < 0 || index >= n || !bx || !by || !ny || !nx) return LBM_EINVAL;
  *bx = s[index].bx;
  *by = s[index].by;
  *ny = s[index].ny;
  *nx = s[index].nx;
  return LBM_OK;
}

extern "C" int lbm_tile_shape_info(int32_t index, int32_t *info, int32_t n) {
  int count;
  const lbmx::TileShape *s = lbmx::tile_shapes(&count);
  if (index < 0 || index >= count || !info || n < 0) return LBM_EINVAL;
  const lbmx::TileShape &t = s[index];
  const int32_t v[8] = {t.bx, t.by, t.ny, t.nx, t.waves, t.cache, t.steps, t.lds};
  for (int32_t q = 0; q < n && q < 8; ++q) info[q] = v[q];
  return LBM_OK;
}
