// lbm_stack.hpp -- several steps per launch on grids that fill the device
// only thinly: a wave per row, the rows of a tile stacked in one workgroup.
#pragma once

#include "lbm_march.hpp"

namespace lbmx {

constexpr int STACK_ROWS = 16;  // waves of a workgroup, one row each
constexpr int STACK_STEPS = 8;  // most steps of a launch

// The populations that leave a tile's rows upward (f_2, f_5, f_6, g_1) and
// downward (f_4, f_7, f_8, g_3), two buffers, one column of padding on
// either side so that the neighbour's shift along x is part of the address.
struct StackRows {
  float v[2][STACK_ROWS][8][66];
};

// The domain's edges within a tile's frame: none; only those of a jet (inlet,
// outflow, symmetry axis or free slip), whose rules are a few selects in
// straight line; others.
enum : int { TILE_INNER = 0, TILE_JET = 1, TILE_ANY = 2 };

// ---------------------------------------------------------------------------
// Up to tile_steps (K) steps per launch for grids of few tiles.  A workgroup
// of 16 waves holds 16 rows of 64 columns, a wave a row, a lane a column, in
// registers; K - 1 halo rows and columns on every side are computed and not
// stored.  Between steps a population moves along x by a lane shift, or, if
// it also moves along r, through an exchange in LDS (eight of the thirteen,
// double-buffered: one barrier per step); rows that no later step needs go
// idle.  Edge rules and rounding are the marching kernel's: the lanes of
// columns -1 and nx hold the ghost ring's values, rows 0 and nr - 1 pull from
// their own populations; the result is bit-identical to one-step launches.
//
// Bound: latency.  On a 128 x 32 jet a one-step launch takes 3.6 us however
// little it does and a two-step launch 9.3; here eight steps take 12.1 us
// (4.6 for the first, 0.7 while few rows are left, 1.5 with all 16: then the
// CU's four SIMDs are busy issuing).  1.5 us per step on 128 x 32 and
// 200 x 96, 1.8 on 1001 x 77 (K = 6), against 4.6 to 5.1 with two steps per
// launch.  The marching kernel cannot shorten this chain: its wave does the
// halo rows one after another.
// ---------------------------------------------------------------------------
template <class C, bool LT>
__global__ __launch_bounds__(64 * STACK_ROWS) void stack_kernel(
    const JetDesc *__restrict__ jets, const TileStart *__restrict__ tile_start,
    const BatchHdr *__restrict__ hdr, int32_t koff, int32_t tog, int32_t nsteps,
    int32_t *__restrict__ flags) {
  using T = typename C::T;
  using Word = typename Raw<sizeof(T)>::type;
  constexpr int ES = (int)sizeof(T);
  __shared__ float4 table[LT ? MARCH_TABLE : 1];
  __shared__ StackRows rows;
  const int lane = (int)threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.y);
  const int tid = lane + 64 * wave;
  const TileList<true> list(jets, tile_start, hdr);
  const TileWalk tw = tile_walk(list.ntiles);
  int32_t table_of = -1;
  for (int32_t t = tw.first; t < tw.end; t += tw.stride) {
    int32_t lt = t;
    const int32_t jid = list.find(lt);
    const JetDesc &d = jets[jid];
    const int64_t step = d.step0 + koff;
    if (step >= d.target) continue;
    const int64_t left = d.target - step;
    const int halo = d.tile_steps - 1;
    int m = min(d.tile_steps, nsteps);
    if (left < m) m = (int)left;
    const Physics ph(d);
    const int nx = d.nx, nr = d.nr;
    const int32_t ty = lt / d.mtiles_x;
    const int32_t tx = lt - ty * d.mtiles_x;
    const int sw = 64 - 2 * halo, sh = STACK_ROWS - 2 * halo;
    const int i0 = tx * sw, j0 = ty * sh, j1 = min(j0 + sh, nr);
    const int i = i0 - halo + lane, j = j0 - halo + wave;
    const int x0 = d.bc[0], x1 = d.bc[1], r0 = d.bc[2], r1 = d.bc[3];
    const bool px = x0 == BC_PERIODIC;
    int il = min(max(i, 0), nx - 1);  // the column loaded (clamped, or wrapped)
    if (px) {
      il = i % nx;
      il += il < 0 ? nx : 0;
    }
    const int jl = min(max(j, 0), nr - 1);
    const bool own = (lane >= halo) & (lane < halo + sw) & (i < nx);
    const bool edge_l = !px & (i0 == 0), edge_r = !px & (nx <= i0 - halo + 63);
    const bool ghost_l = !px & (i == -1), ghost_r = !px & (i == nx);
    const bool first = !px & (i == 0), last = !px & (i == nx - 1);
    const int64_t sel = step + (d.flip ^ tog);
    T *src_raw = static_cast<T *>(d.buf[sel & 1]);
    T *dst_raw = static_cast<T *>(d.buf[(sel + 1) & 1]);
    const uint32_t pitch_b = (uint32_t)d.pitch * ES, plane_b = (uint32_t)d.plane * ES;
    const uint32_t span = (uint32_t)NPOP * plane_b;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(src_raw, 0, (int)span, BUF_WORD3);
    const __amdgpu_buffer_rsrc_t rd = __builtin_amdgcn_make_buffer_rsrc(dst_raw, 0, (int)span, BUF_WORD3);
    const Src<C> src{as_global(static_cast<const T *>(src_raw)), d.plane, d.pitch};
    Word raw[NPOP];
    load_raw<C, 0>(rs, (uint32_t)node_index(d.pitch, il, jl) * ES, plane_b, pitch_b, raw);
    // inlet entries of this row: lane l holds what the state after l + 1
    // steps takes
    const bool inlet = edge_l & (x0 == BC_INLET);
    const bool ghost_in = ghost_l & inlet, row0 = j == 0, rown = j == nr - 1;
    float4 qv = make_float4(0.f, 0.f, 0.f, 0.f);
    if (inlet) {
      // (a 64-bit remainder takes 150 instructions)
      const int64_t s1 = step + 1;
      const int32_t row = s1 < (1 << 30) ? (int32_t)((uint32_t)s1 % (uint32_t)d.n_t)
                                         : (int32_t)(s1 % d.n_t);
      const int32_t at = (row + min(lane, halo)) % d.n_t;
      qv = inlet_at(d.inlet + (int64_t)at * nr, jl);
    }
    const auto entry = [&](int l) {
      return make_float4(lane_value(qv.x, l), lane_value(qv.y, l), lane_value(qv.z, l),
                         lane_value(qv.w, l));
    };
    if (LT && jid != table_of) {  // (the last tile's gathers are done: see the loop's end)
      if (tid < d.table_n) table[tid] = GlobalTable{d.table}(tid);
      __syncthreads();
    }
    table_of = jid;
    const float rr = d.r0 + (float)jl + 0.5f;
    const float rinv = fast_rcp(rr), rsq = rr * rr;
    float f[9], g[4], ug[4];
    decode_raw<C>(d, raw, f, g);
    bool ok = true;
    uint32_t key = 0;
    const auto rnd = [&](int p, float v) { return storage_round<C>(d, p, v, plane_key(key, p)); };
    const auto put = [](bool at, float v, float &to) { to = at ? v : to; };
    const auto ring = [&](int p, int gi, int gj) {
      return src.load(d, p, min(max(gi, -1), nx), gj);
    };
    const int iw = px ? il : i;
    // The levels; E: the edges the tile's rows may meet.
    const auto levels = [&](auto edges) {
      constexpr int E = decltype(edges)::value;
      for (int l = 0; l < m; ++l) {
        const int more = m - 1 - l;  // steps after this one: rows of the frame needed
        const bool act = (j >= max(j0 - more, 0)) & (j <= min(j1 - 1 + more, nr - 1));
        float(*const out)[8][66] = rows.v[l & 1];
        float(*const in)[8][66] = rows.v[(l & 1) ^ 1];
        if (act) {
          if (l > 0) {  // pull: along x by a lane shift, along r from the rows' exchange
            float o[9], og[4];
#pragma unroll
            for (int k = 0; k < 9; ++k) o[k] = f[k];
#pragma unroll
            for (int k = 0; k < 4; ++k) og[k] = g[k];
            float(*const lo)[66] = in[max(wave - 1, 0)];
            float(*const hi)[66] = in[min(wave + 1, STACK_ROWS - 1)];
            f[2] = lo[0][lane + 1];
            g[1] = lo[3][lane + 1];
            f[4] = hi[4][lane + 1];
            g[3] = hi[7][lane + 1];
            f[5] = lo[1][lane];
            f[6] = lo[2][lane + 2];
            f[7] = hi[5][lane + 2];
            f[8] = hi[6][lane];
            f[1] = from_left(o[1]);
            f[3] = from_right(o[3]);
            g[0] = from_left(og[0]);
            g[2] = from_right(og[2]);
            if constexpr (E == TILE_JET) {
              // mirrored rows (corners: the inlet's own value, rounded as the
              // link that pulls it)
              float a = o[8], b = o[5];
              if constexpr (C::dev) {
                put(ghost_in, rnd(5, entry(l - 1).z), a);
                put(ghost_in, rnd(8, entry(l - 1).y), b);
              }
              put(row0, o[4], f[2]);
              put(row0, from_left(a), f[5]);
              put(row0, from_right(o[7]), f[6]);
              put(row0, og[3], g[1]);
              put(rown, o[2], f[4]);
              put(rown, from_right(o[6]), f[7]);
              put(rown, from_left(b), f[8]);
              put(rown, og[1], g[3]);
            } else if constexpr (E == TILE_ANY) {
              if (j == 0) {  // nothing below: the r-side rule
                if (r0 == BC_AXIS || r0 == BC_FREESLIP) {
                  // (corners: the mirrored link through the x rule at the edge row)
                  float a = o[8], b = o[7];
                  if (inlet) put(ghost_l, rnd(5, entry(l - 1).z), a);
                  if (edge_l & (x0 == BC_EQ)) put(ghost_l, ring(5, -1, -1), a);
                  if (edge_r & (x1 == BC_EQ)) put(ghost_r, ring(6, nx, -1), b);
                  f[2] = o[4];
                  f[5] = from_left(a);
                  f[6] = from_right(b);
                  g[1] = og[3];
                  if (edge_l & (x0 == BC_WALL)) put(first, o[6], f[5]);
                  if (edge_r & (x1 == BC_WALL)) put(last, o[5], f[6]);
                } else if (r0 == BC_WALL) {
                  f[2] = o[4];
                  f[5] = o[7];
                  f[6] = o[8];
                  g[1] = rnd(10, wall_g(d, 2, ug[3]));
                } else {  // BC_EQ
                  f[2] = ring(2, iw, -1);
                  f[5] = ring(5, iw - 1, -1);
                  f[6] = ring(6, iw + 1, -1);
                  g[1] = ring(10, iw, -1);
                }
              }
              if (j == nr - 1) {  // nothing above
                if (r1 == BC_FREESLIP) {
                  float a = o[5], b = o[6];
                  if (inlet) put(ghost_l, rnd(8, entry(l - 1).y), a);
                  if (edge_l & (x0 == BC_EQ)) put(ghost_l, ring(8, -1, nr), a);
                  if (edge_r & (x1 == BC_EQ)) put(ghost_r, ring(7, nx, nr), b);
                  f[4] = o[2];
                  f[8] = from_left(a);
                  f[7] = from_right(b);
                  g[3] = og[1];
                  if (edge_l & (x0 == BC_WALL)) put(first, o[7], f[8]);
                  if (edge_r & (x1 == BC_WALL)) put(last, o[8], f[7]);
                } else if (r1 == BC_WALL) {
                  f[4] = o[2];
                  f[7] = o[5];
                  f[8] = o[6];
                  g[3] = rnd(12, wall_g(d, 3, ug[1]));
                } else {  // BC_EQ
                  f[4] = ring(4, iw, nr);
                  f[7] = ring(7, iw + 1, nr);
                  f[8] = ring(8, iw - 1, nr);
                  g[3] = ring(12, iw, nr);
                }
              }
              // x walls give a node its own opposite populations (r rules first)
              if (edge_l & (x0 == BC_WALL)) {
                put(first, o[3], f[1]);
                if (j > 0) put(first, o[7], f[5]);
                if (j < nr - 1) put(first, o[6], f[8]);
                put(first, rnd(9, wall_g(d, 0, ug[2])), g[0]);
              }
              if (edge_r & (x1 == BC_WALL)) {
                put(last, o[1], f[3]);
                if (j > 0) put(last, o[8], f[6]);
                if (j < nr - 1) put(last, o[5], f[7]);
                put(last, rnd(11, wall_g(d, 1, ug[0])), g[2]);
              }
            }
          }
          bool okn;
          if constexpr (LT) okn = collide(ph, rinv, rsq, f, g, NoHook(), LdsTable{table});
          else okn = collide(ph, rinv, rsq, f, g, NoHook(), GlobalTable{d.table});
          ok &= okn | !own;  // (every fluid node belongs to one wave, which reports it)
          key = sr_key(il, j, step + l + 1);
        }
        if (more > 0) {
          if (act) {
#pragma unroll
            for (int k = 0; k < 4; ++k) ug[k] = g[k];
            if constexpr (C::dev) {
#pragma unroll
              for (int p = 0; p < NPOP; ++p) {
                float &x = p < 9 ? f[p] : g[p - 9];
                x = rnd(p, x);
              }
            }
            // the lanes of columns -1 and nx hold the ghost ring's values
            if ((E == TILE_JET) | (E == TILE_ANY && inlet)) {
              const float4 q = entry(l);
              put(ghost_in, rnd(1, q.x), f[1]);
              put(ghost_in, rnd(5, q.y), f[5]);
              put(ghost_in, rnd(8, q.z), f[8]);
              put(ghost_in, rnd(9, q.w), g[0]);
            }
            if ((E == TILE_JET) | (E == TILE_ANY && edge_r && x1 == BC_OUTFLOW)) {
              put(ghost_r, from_left(f[3]), f[3]);
              put(ghost_r, from_left(f[6]), f[6]);
              put(ghost_r, from_left(f[7]), f[7]);
              put(ghost_r, from_left(g[2]), g[2]);
            }
            if constexpr (E == TILE_ANY) {
              if (edge_l & (x0 == BC_EQ)) {
                put(ghost_l, ring(1, -1, j), f[1]);
                put(ghost_l, ring(5, -1, j), f[5]);
                put(ghost_l, ring(8, -1, j), f[8]);
                put(ghost_l, ring(9, -1, j), g[0]);
              }
              if (edge_r & (x1 == BC_EQ)) {
                put(ghost_r, ring(3, nx, j), f[3]);
                put(ghost_r, ring(6, nx, j), f[6]);
                put(ghost_r, ring(7, nx, j), f[7]);
                put(ghost_r, ring(11, nx, j), g[2]);
              }
            }
            float(*const to)[66] = out[wave];
            to[0][lane + 1] = f[2];
            to[1][lane + 1] = f[5];
            to[2][lane + 1] = f[6];
            to[3][lane + 1] = g[1];
            to[4][lane + 1] = f[4];
            to[5][lane + 1] = f[7];
            to[6][lane + 1] = f[8];
            to[7][lane + 1] = g[3];
          }
          __syncthreads();
        }
      }
    };
    // rows that the tile's frame shares with the domain's edges
    const bool edge_0 = j0 - halo <= 0, edge_n = j0 + sh + halo >= nr;
    const bool jet = (!edge_l | inlet) & (!edge_r | (x1 == BC_OUTFLOW)) &
                     (!edge_0 | (r0 == BC_AXIS) | (r0 == BC_FREESLIP)) &
                     (!edge_n | (r1 == BC_FREESLIP));
    if (!(edge_l | edge_r | edge_0 | edge_n)) levels(Int<TILE_INNER>());
    else if (jet) levels(Int<TILE_JET>());
    else levels(Int<TILE_ANY>());
    if ((j >= j0) & (j < j1) & own) {
      store_node<C, 0>(d, rd, (uint32_t)node_index(d.pitch, i, j) * ES, plane_b, f, g, key);
      if (((i0 == 0) | (i0 + sw >= nx) | row0 | rown) && is_edge(d, i, j)) {
        const Dst<C> out{as_global(dst_raw), d.plane, d.pitch};
        ghost_epilogue<C>(d, out, i, j, f, g, entry(m - 1), key);
      }
    }
    if (!ok) flags[d.slot] = 1;
    if (t + tw.stride < tw.end) __syncthreads();  // the exchange is reused by the next tile
  }
}

}  // namespace lbmx
