// lbm_march.hpp -- several steps per launch with the intermediate states in
// registers (temporal blocking by a marching wave).
#pragma once

#include "lbm_kernels.hpp"

namespace lbmx {

// A column's value from the lane on its left (column i - 1) or right (i + 1).
// The lane at the wave's end gets 0: it lies in the halo, where the value is
// not used.
__device__ __forceinline__ float from_left(float v) {
  return __builtin_bit_cast(
      float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x138, 0xf, 0xf, true));
}
__device__ __forceinline__ float from_right(float v) {
  return __builtin_bit_cast(
      float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x130, 0xf, 0xf, true));
}

constexpr int MARCH_TABLE = 256;  // property-table entries held in LDS

struct LdsTable {
  static constexpr bool in_lds = true;
  const float4 *p;
  __device__ __forceinline__ float4 operator()(int i) const { return p[i]; }
};

// What a level keeps of its last rows for the next level (see march_kernel):
// the populations that move up (f_2, f_5, f_6, g_1) of its last two rows and
// those that stay in their row (f_0, f_1, f_3, g_0, g_2) of its last.
struct LevelRows {
  float u1[4], u2[4], h[5];
};

// What the edge rules of one wave's strip need.
template <class C>
struct MarchEdge {
  Src<C> src;        // the launch's source buffer (constant ring values)
  bool left, right;  // column -1 / column nx is one of the wave's lanes
  bool at_left, at_right;  // this lane is that column
  int i;             // this lane's column (wrapped with periodic x edges)
};

// The post-collision values (f, g: rounded as stored; ug: g before rounding)
// of row j of an intermediate state, made what the next level pulls: the
// lanes of columns -1 and nx take the values that a step's epilogue would
// write to the ghost ring (XE: the strip has such a lane), and up / u1 become
// the ghost rows above row nr - 1 and below row 0.  up: the populations the
// row passes upward; q: the inlet row's entry; RE: row j may be 0 or nr - 1.  Copies keep the key they were
// rounded with, computed values take the key of the plane they are written
// to, as in ghost_epilogue.
template <class C, bool XE, bool RE>
__device__ __forceinline__ void march_edges(const JetDesc &d, const MarchEdge<C> &w, int j,
                                            float (&f)[9], float (&g)[4], const float (&ug)[4],
                                            float (&u1)[4], float (&up)[4], float4 q,
                                            uint32_t key) {
  const int nr = d.nr;
  const int x0 = d.bc[0], x1 = d.bc[1], r0 = d.bc[2], r1 = d.bc[3];
  const auto rnd = [&](int p, float v) { return storage_round<C>(d, p, v, plane_key(key, p)); };
  const auto put = [](bool at, float v, float &dst) { dst = at ? v : dst; };
  const auto ring = [&](int p, int i, int jj) { return w.src.load(d, p, i, jj); };
  const bool L = w.at_left, R = w.at_right;
  if (XE && w.left) {
    if (x0 == BC_INLET) {
      put(L, rnd(1, q.x), f[1]);
      put(L, rnd(5, q.y), f[5]);
      put(L, rnd(8, q.z), f[8]);
      put(L, rnd(9, q.w), g[0]);
    } else if (x0 == BC_WALL) {
      put(L, from_right(f[3]), f[1]);
      if (!RE || j > 0) {
        put(L, from_right(f[7]), u1[1]);  // f_5 of (-1, j - 1)
        put(L, from_right(u1[2]), f[8]);  // f_6 of (0, j - 1)
      }
      put(L, rnd(9, wall_g(d, 0, from_right(ug[2]))), g[0]);
    } else {  // BC_EQ
      put(L, ring(1, -1, j), f[1]);
      put(L, ring(5, -1, j), f[5]);
      put(L, ring(8, -1, j), f[8]);
      put(L, ring(9, -1, j), g[0]);
    }
  }
  if (XE && w.right) {
    if (x1 == BC_OUTFLOW) {
      put(R, from_left(f[3]), f[3]);
      put(R, from_left(f[6]), f[6]);
      put(R, from_left(f[7]), f[7]);
      put(R, from_left(g[2]), g[2]);
    } else if (x1 == BC_WALL) {
      put(R, from_left(f[1]), f[3]);
      if (!RE || j > 0) {
        put(R, from_left(f[8]), u1[2]);  // f_6 of (nx, j - 1)
        put(R, from_left(u1[1]), f[7]);  // f_5 of (nx - 1, j - 1)
      }
      put(R, rnd(11, wall_g(d, 1, from_left(ug[0]))), g[2]);
    } else {  // BC_EQ
      put(R, ring(3, d.nx, j), f[3]);
      put(R, ring(6, d.nx, j), f[6]);
      put(R, ring(7, d.nx, j), f[7]);
      put(R, ring(11, d.nx, j), g[2]);
    }
  }
  up[0] = f[2];
  up[1] = f[5];
  up[2] = f[6];
  up[3] = g[1];
  // (a lane's column on the ring: lanes past the ring read its ends)
  const int ic = min(max(w.i, -1), d.nx);
  if (RE && j == 0) {  // ghost row -1 in place of the row below
    if (r0 == BC_AXIS || r0 == BC_FREESLIP) {
      u1[0] = f[4];
      u1[1] = f[8];
      u1[2] = f[7];
      u1[3] = g[3];
      // corners: the mirrored link through the x rule at the edge row
      if (XE && w.left) {
        if (x0 == BC_WALL) put(L, from_right(f[6]), u1[1]);
        else if (x0 == BC_INLET) put(L, rnd(5, q.z), u1[1]);
        else put(L, ring(5, -1, -1), u1[1]);
      }
      if (XE && w.right && x1 != BC_OUTFLOW)
        put(R, x1 == BC_WALL ? from_left(f[5]) : ring(6, d.nx, -1), u1[2]);
    } else if (r0 == BC_WALL) {
      u1[0] = f[4];
      u1[1] = from_right(f[7]);
      u1[2] = from_left(f[8]);
      u1[3] = rnd(10, wall_g(d, 2, ug[3]));
    } else {  // BC_EQ
      u1[0] = ring(2, ic, -1);
      u1[1] = ring(5, ic, -1);
      u1[2] = ring(6, ic, -1);
      u1[3] = ring(10, ic, -1);
    }
  }
  if (RE && j == nr - 1) {  // what is passed on is the ghost row's f_4, f_7, f_8, g_3
    if (r1 == BC_FREESLIP) {
      up[0] = f[2];
      up[1] = f[6];
      up[2] = f[5];
      up[3] = g[1];
      if (XE && w.left) {
        if (x0 == BC_WALL) put(L, from_right(f[7]), up[2]);
        else if (x0 == BC_INLET) put(L, rnd(8, q.y), up[2]);
        else put(L, ring(8, -1, nr), up[2]);
      }
      if (XE && w.right && x1 != BC_OUTFLOW)
        put(R, x1 == BC_WALL ? from_left(f[8]) : ring(7, d.nx, nr), up[1]);
    } else if (r1 == BC_WALL) {
      up[0] = f[2];
      up[1] = from_left(f[5]);
      up[2] = from_right(f[6]);
      up[3] = rnd(12, wall_g(d, 3, ug[1]));
    } else {  // BC_EQ
      up[0] = ring(4, ic, nr);
      up[1] = ring(7, ic, nr);
      up[2] = ring(8, ic, nr);
      up[3] = ring(12, ic, nr);
    }
  }
}

__device__ __forceinline__ float uniform(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, v)));
}
__device__ __forceinline__ float lane_value(float v, int l) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), l));
}

// A level's row f, g takes its place among the rows kept for the next level.
__device__ __forceinline__ void march_keep(LevelRows &v, const float (&f)[9], const float (&g)[4],
                                           const float (&up)[4]) {
#pragma unroll
  for (int k = 0; k < 4; ++k) v.u2[k] = v.u1[k], v.u1[k] = up[k];
  v.h[0] = f[0];
  v.h[1] = f[1];
  v.h[2] = f[3];
  v.h[3] = g[0];
  v.h[4] = g[2];
}

// The same, and f, g become what the next level pulls at the row below: its
// populations that move down with those of the kept rows.
__device__ __forceinline__ void march_pull(LevelRows &v, float (&f)[9], float (&g)[4],
                                           const float (&up)[4]) {
  const LevelRows o = v;
  march_keep(v, f, g, up);
  f[0] = o.h[0];
  f[1] = from_left(o.h[1]);
  f[2] = o.u2[0];
  f[3] = from_right(o.h[2]);
  f[5] = from_left(o.u2[1]);
  f[6] = from_right(o.u2[2]);
  f[7] = from_right(f[7]);
  f[8] = from_left(f[8]);
  g[0] = from_left(o.h[3]);
  g[1] = o.u2[3];
  g[2] = from_right(o.h[4]);
}

template <int N>
struct Int {
  static constexpr int value = N;
};
// f(Int<1>()), f(Int<2>()), .. f(Int<K - 1>())
template <int K, int N = 1, class F>
__device__ __forceinline__ void below(const F &f) {
  if constexpr (N < K) {
    f(Int<N>());
    below<K, N + 1>(f);
  }
}

// Where a strip's ghost columns lie: none, column -1 with an inlet, column nx
// with an outflow or a wall (the edges of a free and of an impinging jet, whose
// rows cost little more than an inner strip's), or any other rule or both.
enum : int { STRIP_INNER = 0, STRIP_INLET, STRIP_OUTFLOW, STRIP_WALL, STRIP_EDGE };

// One wave's tile: strip i0 (of kind EK), rows j0 .. j1 - 1.  ready() is
// called between the first row's loads and their use: the table in LDS is
// complete after it.  late: the wave goes first for most of its rows (see
// march_kernel).
template <class C, int K, int CP, bool LT, int EK, class Ready>
__device__ __forceinline__ bool march_tile(const JetDesc &jd, int64_t step, int32_t tog, int m,
                                           int i0, int j0, int j1, bool late,
                                           const float4 *table, const Ready &ready) {
  using T = typename C::T;
  using Word = typename Raw<sizeof(T)>::type;
  constexpr int ES = (int)sizeof(T);
  constexpr int HALO = K - 1, SW = 64 - 2 * HALO;
  constexpr int AUX_L = (CP & 2) ? CACHE_NT : 0, AUX_S = (CP & 1) ? CACHE_NT : 0;
  constexpr bool XE = EK != STRIP_INNER;
  const JetDesc &d = jd;
  const Physics ph(jd);  // (in registers: no reloads between the rows' stores)
  const int lane = (int)threadIdx.x;
  const int nx = d.nx, nr = d.nr;
  const bool px = d.bc[0] == BC_PERIODIC;
  const int i = i0 - HALO + lane;
  // the fluid column whose populations this lane loads (and whose rounding
  // key it uses): clamped into the domain, or wrapped
  int il = min(max(i, 0), nx - 1);
  if (px) {
    il = i % nx;
    il += il < 0 ? nx : 0;
  }
  const bool own = (lane >= HALO) & (lane < HALO + SW) & (i < nx);
  const int64_t sel = step + (d.flip ^ tog);
  T *src_raw = static_cast<T *>(jd.buf[sel & 1]);
  T *dst_raw = static_cast<T *>(jd.buf[(sel + 1) & 1]);
  const uint32_t pitch_b = (uint32_t)d.pitch * ES, plane_b = (uint32_t)d.plane * ES;
  const uint32_t span = (uint32_t)NPOP * plane_b;
  const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(src_raw, 0, (int)span, BUF_WORD3);
  const __amdgpu_buffer_rsrc_t rd = __builtin_amdgcn_make_buffer_rsrc(dst_raw, 0, (int)span, BUF_WORD3);
  const MarchEdge<C> edge{{as_global(static_cast<const T *>(src_raw)), d.plane, d.pitch},
                          EK == STRIP_INLET || (EK == STRIP_EDGE && i0 == 0),
                          EK == STRIP_OUTFLOW || EK == STRIP_WALL || (EK == STRIP_EDGE && nx <= i0 - HALO + 63),
                          XE && i == -1, XE && i == nx, px ? il : i};
  const bool xcol = (i0 == 0) | (i0 + SW >= nx);  // owns a column that writes ring values
  // Inlet entries: lane l < K loads what the state after l + 1 steps takes at
  // level l + 1's row, a row ahead like the populations.
  const bool inlet = EK == STRIP_INLET || (EK == STRIP_EDGE && i0 == 0 && d.bc[0] == BC_INLET);
  const int ll = min(lane, K - 1);
  const float4 *in_row = d.inlet + (inlet ? (int64_t)((step + 1 + ll) % d.n_t) * nr : 0);
  const auto in_load = [&](int t) { return inlet_at(in_row, min(max(t - ll, 0), nr - 1)); };
  const auto in_entry = [&](const float4 &q, int l) {
    return make_float4(lane_value(q.x, l), lane_value(q.y, l), lane_value(q.z, l),
                       lane_value(q.w, l));
  };
  // byte offset of this lane's column in a buffer's first row (less one
  // element, so that the loads' shifts along x are small positive constants)
  const uint32_t vload = (uint32_t)(XOFF + il - 1) * ES;
  const uint32_t vown = (uint32_t)(XOFF + i) * ES;
  Word raw[NPOP];
  const auto load_row = [&](int t) {  // the populations that row min(t, nr - 1) pulls
    const uint32_t mid = vload + (uint32_t)(min(t, nr - 1) + 1) * pitch_b;
    const uint32_t below = mid - pitch_b, above = mid + pitch_b;
#pragma unroll
    for (int p = 0; p < NPOP; ++p)
      raw[p] = buf_load<ES, AUX_L>(
          rs, (per(p) > 0 ? below : per(p) < 0 ? above : mid) + (uint32_t)((1 - pex(p)) * ES),
          (uint32_t)p * plane_b);
  };
  LevelRows lev[K - 1];
#pragma unroll
  for (int l = 0; l < K - 1; ++l) {
#pragma unroll
    for (int k = 0; k < 4; ++k) lev[l].u1[k] = lev[l].u2[k] = 0.0f;
#pragma unroll
    for (int k = 0; k < 5; ++k) lev[l].h[k] = 0.0f;
  }
  float rinv[K], rsq[K];  // 1 / r and r^2 of each level's row
#pragma unroll
  for (int l = 0; l < K; ++l) rinv[l] = rsq[l] = 1.0f;
  bool ok = true;
  float f[9], g[4];
  uint32_t key = 0;
  const float tw = EK == STRIP_WALL ? d.wallT[1] : 0.0f;  // (NaN: adiabatic)
  const auto next_row = [&](int t) {  // takes row t's loads, issues row t + 1's
#pragma unroll
    for (int l = K - 1; l > 0; --l) rinv[l] = rinv[l - 1], rsq[l] = rsq[l - 1];
    const float r = d.r0 + (float)t + 0.5f;
    rinv[0] = uniform(fast_rcp(r));
    rsq[0] = uniform(r * r);
    decode_raw<C>(d, raw, f, g);
    load_row(t + 1);
  };
  const auto level = [&](int l, int j) {  // the collision of level l + 1 at row j
    bool okn;
    if constexpr (LT) okn = collide(ph, rinv[l], rsq[l], f, g, NoHook(), LdsTable{table});
    else okn = collide(ph, rinv[l], rsq[l], f, g, NoHook(), GlobalTable{d.table});
    key = sr_key(il, j, step + l + 1);
    ok &= okn | !own;  // (every fluid node belongs to one wave, which reports it)
  };
  const auto stored = [&](float (&ug)[4]) {  // f, g as the storage form rounds them
#pragma unroll
    for (int k = 0; k < 4; ++k) ug[k] = g[k];
    if constexpr (C::dev) {
#pragma unroll
      for (int p = 0; p < NPOP; ++p) {
        float &x = p < 9 ? f[p] : g[p - 9];
        x = storage_round<C>(d, p, x, plane_key(key, p));
      }
    }
  };
  const auto store = [&](int j, const float4 &q, int l, bool ring) {
    if (own) {
      store_node<C, AUX_S>(d, rd, vown + (uint32_t)(j + 1) * pitch_b, plane_b, f, g, key);
      if (ring) {
        const Dst<C> out{as_global(dst_raw), d.plane, d.pitch};
        if (is_edge(d, i, j)) ghost_epilogue<C>(d, out, i, j, f, g, in_entry(q, l), key);
      }
    }
  };
  // the fast rows' edge rules and ring values (see march_edges, ghost_epilogue)
  const auto fast_edges = [&](int l, int j, const float (&ug)[4], float (&up)[4], const float4 &q) {
    const auto put = [](bool at, float v, float &dst) { dst = at ? v : dst; };
    if constexpr (EK == STRIP_INLET) {
      const float4 e = in_entry(q, l);
      const auto rnd = [&](int p, float v) { return storage_round<C>(d, p, v, plane_key(key, p)); };
      put(edge.at_left, rnd(1, e.x), f[1]);
      put(edge.at_left, rnd(5, e.y), f[5]);
      put(edge.at_left, rnd(8, e.z), f[8]);
      put(edge.at_left, rnd(9, e.w), g[0]);
      up[1] = f[5];
    } else if constexpr (EK == STRIP_OUTFLOW) {
      put(edge.at_right, from_left(f[3]), f[3]);
      put(edge.at_right, from_left(f[6]), f[6]);
      put(edge.at_right, from_left(f[7]), f[7]);
      put(edge.at_right, from_left(g[2]), g[2]);
      up[2] = f[6];
    } else if constexpr (EK == STRIP_WALL) {
      const float tg = tw == tw ? 0.5f * tw - from_left(ug[0]) : from_left(ug[0]);
      put(edge.at_right, from_left(f[1]), f[3]);
      put(edge.at_right, from_left(f[8]), lev[l].u1[2]);
      put(edge.at_right, from_left(lev[l].u1[1]), f[7]);
      put(edge.at_right, storage_round<C>(d, 11, tg, plane_key(key, 11)), g[2]);
    } else if constexpr (EK == STRIP_EDGE) {
      march_edges<C, true, false>(d, edge, j, f, g, ug, lev[l].u1, up, in_entry(q, l), key);
    }
  };
  const auto fast_store = [&](int j, const float4 &q) {
    if constexpr (EK == STRIP_INLET || EK == STRIP_OUTFLOW || EK == STRIP_WALL) {
      const uint32_t at = vown + (uint32_t)(j + 1) * pitch_b;
      const auto put = [&](int p, float v, uint32_t off, int kp = -1) {
        const T x = C::enc(v, pop_offset<C>(d, p), plane_key(key, kp < 0 ? p : kp));
        buf_store<ES, AUX_S>(__builtin_bit_cast(Word, x), rd, off, (uint32_t)p * plane_b);
      };
      const float4 e = in_entry(q, K - 1);
      if (own) {
        store_node<C, AUX_S>(d, rd, at, plane_b, f, g, key);
        if (EK == STRIP_INLET && i == 0) {
          put(1, e.x, at - ES);
          put(5, e.y, at - ES);
          put(8, e.z, at - ES);
          put(9, e.w, at - ES);
        }
        if (EK == STRIP_OUTFLOW && i == nx - 1) {
          put(3, f[3], at + ES);
          put(6, f[6], at + ES);
          put(7, f[7], at + ES);
          put(11, g[2], at + ES);
        }
        if (EK == STRIP_WALL && i == nx - 1) {  // (copies keep their key)
          put(3, f[1], at + ES, 1);
          put(6, f[8], at + ES - pitch_b, 8);
          put(7, f[5], at + ES + pitch_b, 5);
          put(11, tw == tw ? 0.5f * tw - g[0] : g[0], at + ES);
        }
      }
    } else {
      store(j, q, K - 1, xcol);
    }
  };
  const int tb = max(j0 - (m - 1), 0), te = j1 + m - 2;
  // rows ts .. tf of the front: every level active, none at row 0 or nr - 1
  const int ts = m == K ? max(j0 + K - 1, K) : te + 1, tf = min(te, nr - 2);
  float4 qn = make_float4(0.f, 0.f, 0.f, 0.f);
  if (inlet) qn = in_load(tb);
  load_row(tb);
  ready();
  // One row of the front with levels 1 .. N active, none at row 0 or nr - 1.
  const auto fast_row = [&](auto levels, int t) {
    constexpr int N = decltype(levels)::value;
    const float4 q = qn;
    if (inlet) qn = in_load(t + 1);
    next_row(t);
    level(0, t);
#pragma unroll
    for (int l = 0; l < (N < K ? N : K - 1); ++l) {
      float ug[4];
      stored(ug);
      float up[4] = {f[2], f[5], f[6], g[1]};
      fast_edges(l, t - l, ug, up, q);
      if (l == N - 1) {
        march_keep(lev[l], f, g, up);
      } else {
        march_pull(lev[l], f, g, up);
        level(l + 1, t - l - 1);
      }
    }
    if constexpr (N == K) fast_store(t - K + 1, q);
  };
  int t = tb;
  const int calm = late ? tb + (te - tb) * 5 / 8 : te + 1;
  if (late) __builtin_amdgcn_s_setprio(1);
  // away from the domain's first and last rows the levels start one by one,
  // two rows apart
  if (EK != STRIP_EDGE && m == K && tb >= 1 && tb + 2 * K - 3 <= nr - 2)
    below<K>([&](auto levels) {
#pragma unroll 1
      for (int q = 0; q < 2; ++q, ++t) fast_row(levels, t);
    });
  while (t <= te) {
    if ((t >= ts) & (t <= tf)) {
#pragma unroll 1
      do {
        if (t == calm) __builtin_amdgcn_s_setprio(0);
        fast_row(Int<K>(), t++);
      } while (t <= tf);
      continue;
    }
    if (t == calm) __builtin_amdgcn_s_setprio(0);
    const float4 q = qn;
    if (inlet) qn = in_load(t + 1);
    next_row(t);
    int j = t;
    if (j < nr) level(0, j);
#pragma unroll
    for (int l = 0; l < K - 1; ++l) {
      if (l + 1 < m) {
        float up[4] = {f[2], f[5], f[6], g[1]};
        if (j < nr) {
          float ug[4];
          stored(ug);
          up[0] = f[2], up[1] = f[5], up[2] = f[6], up[3] = g[1];
          if ((XE & (j >= 0)) | (j == 0) | (j == nr - 1))
            march_edges<C, XE, true>(d, edge, j, f, g, ug, lev[l].u1, up, in_entry(q, l), key);
        } else {  // the ghost row above the domain, kept by row nr - 1
          f[4] = lev[l].u1[0];
          f[7] = lev[l].u1[1];
          f[8] = lev[l].u1[2];
          g[3] = lev[l].u1[3];
        }
        march_pull(lev[l], f, g, up);
        --j;
        if ((j >= max(j0 - (m - 2 - l), 0)) & (j < nr)) level(l + 1, j);
      }
    }
    if (j >= j0)  // level m's row (j < j1 always)
      store(j, q, m - 1, xcol | (j == 0) | (j == nr - 1));
    ++t;
  }
  if (late) __builtin_amdgcn_s_setprio(0);
  return ok;
}

// ---------------------------------------------------------------------------
// Up to K steps per launch.  A wave owns a strip of 64 - 2 (K - 1) columns
// (one lane a column, K - 1 halo lanes on either side) and `tile_rows` rows,
// and marches up it row by row: level 1 pulls row t from the source buffer
// and collides, level l (the state l - 1 steps later) collides row t - l + 1
// from what level l - 1 computed in this and the two iterations before, and
// the last level's row is stored.  Between levels a population moves along x
// by a lane shift and along r by waiting in a register: of each level the
// wave keeps the upward-moving populations of two rows and the resting and
// x-moving ones of one (13 registers), and uses the downward-moving ones at
// once.  No LDS image, no barrier and no second read of memory per step: a
// step costs its collision, eight lane shifts and the halo (rows and columns
// that the neighbouring waves compute too).
//
// Bound: vector-ALU issue.  An inner row costs 151 VALU instructions per
// level, the two-step kernel 270 per node update with its frame, LDS image
// and addressing; beside it stand the launch (3.6 us), the first row's loads
// (2 us) and the halo (1.3 of a 2048 x 512 jet's own collisions).  K = 4: with
// three steps the launch and the memory weigh more (10.4 us per step on
// 2048 x 512, 43.6 on 4096 x 1024), with four 9.4 and 32.0 us (111 and 131
// GLUPS); the two-step kernel takes 13.1 and 57.0.  K = 5 pays where the
// state is larger than the caches: 29.9 us on 4096 x 1024.  W = 2 waves per SIMD: the
// levels' rows need 190 VGPRs, and held to 128 the kernel spills.
//
// The workgroups fill the CUs once before a second goes on each.  Of two
// waves on a SIMD the older issues first, so that it would be done after
// 22 us of a 2048 x 512 launch and leave the younger 10 us alone, in which
// the SIMD can fill only two thirds of its issue slots.  The workgroups of
// the second filling therefore go first for five eighths of their rows, and
// both end together: 9.4 us per step against 10.1 (half of the rows 9.6, all
// of them 10.2), 15.4 against 16.6 on 3000 x 700; 4096 x 1024, which waits
// for memory more, keeps its 32.3.
//
// The edge rules act between levels as the step epilogue does on the ghost
// ring (march_edges); the constant ghosts of equilibrium sides are read from
// the source buffer's ring.  Intermediate values are rounded through the
// storage codec, so the result is bit-identical to one-step launches.
//
// m = min(K, nsteps, steps to the jet's target) steps are taken: the levels
// past m are skipped and level m's rows stored.  A launch reads one buffer
// and writes the other whatever m, so that an even m toggles the jet's flip
// (advance_kernel; `tog` carries the toggles since the last advance).
// The property table sits in LDS (LT; jets with more entries than
// MARCH_TABLE take the instance that reads it from memory): its gathers then
// do not wait behind the next row's loads, which are in flight through all
// the levels of a row.
// ---------------------------------------------------------------------------
template <class C, int K, int NW, int W, int CP, bool LT>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(W, 8))) void march_kernel(
    const JetDesc *__restrict__ jets, const TileStart *__restrict__ tile_start,
    const BatchHdr *__restrict__ hdr, int32_t koff, int32_t tog, int32_t nsteps,
    int32_t *__restrict__ flags) {
  constexpr int HALO = K - 1, SW = 64 - 2 * HALO;
  __shared__ float4 table[LT ? MARCH_TABLE : 1];
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.y);
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
    int m = min(K, nsteps);
    if (left < m) m = (int)left;
    // The jet's table: one entry a thread, on its way while the tile's first
    // rows are asked for, written when they have been.
    static_assert(!LT || 64 * NW >= MARCH_TABLE, "table fill");
    const int tid = (int)threadIdx.x + 64 * wave;
    const bool fill = LT && jid != table_of;
    float4 entry = make_float4(0.f, 0.f, 0.f, 0.f);
    if (fill && tid < d.table_n) entry = GlobalTable{d.table}(tid);
    const auto ready = [&] {
      if (!fill) return;
      if (table_of >= 0) __syncthreads();  // (the last tile's gathers are done)
      if (LT && tid < d.table_n) table[tid] = entry;
      __syncthreads();
    };
    const int32_t ty = lt / d.mtiles_x;
    const int32_t tx = lt - ty * d.mtiles_x;
    const int i0 = tx * SW;
    const int j0 = (ty * NW + wave) * d.tile_rows;
    const int j1 = min(j0 + d.tile_rows, d.nr);
    if (j0 >= d.nr) {  // (an idle wave of the last tile row)
      ready();
      table_of = jid;
      continue;
    }
    const bool late = ((blockIdx.x / (uint32_t)d.cus) & 1) != 0;
    const bool px = d.bc[0] == BC_PERIODIC;
    const bool left_edge = !px & (i0 == 0), right_edge = !px & (d.nx <= i0 - HALO + 63);
    bool ok;
    if (!left_edge & !right_edge)
      ok = march_tile<C, K, CP, LT, STRIP_INNER>(d, step, tog, m, i0, j0, j1, late, table, ready);
    else if (!right_edge & (d.bc[0] == BC_INLET))
      ok = march_tile<C, K, CP, LT, STRIP_INLET>(d, step, tog, m, i0, j0, j1, late, table, ready);
    else if (!left_edge & (d.bc[1] == BC_OUTFLOW))
      ok = march_tile<C, K, CP, LT, STRIP_OUTFLOW>(d, step, tog, m, i0, j0, j1, late, table, ready);
    else if (!left_edge & (d.bc[1] == BC_WALL))
      ok = march_tile<C, K, CP, LT, STRIP_WALL>(d, step, tog, m, i0, j0, j1, late, table, ready);
    else
      ok = march_tile<C, K, CP, LT, STRIP_EDGE>(d, step, tog, m, i0, j0, j1, late, table, ready);
    table_of = jid;
    if (!ok) flags[d.slot] = 1;
  }
}

}  // namespace lbmx
