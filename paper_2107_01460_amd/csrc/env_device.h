// Device-side pieces of the two grid worlds (foraging, warehouse), shared by the standalone env-step kernels and by
// the fused rollout kernel: the new-episode draw, the lock-step transition of one env resolved redundantly in the
// registers of each of its agents' lanes, and the painting of a lane's egocentric window.
#pragma once
#include "common.h"

namespace marl {

struct EnvParams {
  int G, A, F, L, cap, N;
  int kind;  // 0 foraging; 1 warehouse; 2 warehouse with episode end on collision (L = requested shelves there)
  uint32_t k0, k1;
  uint32_t inv_g20;  // ceil(2^20 / G): (r * inv_g20) >> 20 == r / G exactly for r < G*G <= 4096
};

// Entity packed as row | col << 8 | level << 16.
__device__ __forceinline__ int e_row(uint32_t e) { return (int)(e & 0xff); }
__device__ __forceinline__ int e_col(uint32_t e) { return (int)((e >> 8) & 0xff); }
__device__ __forceinline__ int e_lvl(uint32_t e) { return (int)((e >> 16) & 0xff); }

// The draws of a new episode: draw j is word j % 4 of Philox call j / 4 of the stream (env, episode).
// SHARE = false: the lane computes every call itself.  SHARE = true: the A lanes of the env's agents (consecutive lanes
// of one wavefront, this one being agent a_idx, all of them in here together because the episode ended for the env)
// split the calls -- lane a computes calls a, a + A, ... -- and fetch the others' words across lanes: a call is forty
// quarter-rate multiplies, and every lane of an env computing all of them was a quarter of the env step's time.
template <int NC, bool SHARE>
struct ResetDraws {
  uint32_t buf[4];
  uint32_t mine[SHARE ? NC : 1][4];
  int j, A, base;
  uint32_t env, episode, k0, k1;
  __device__ __forceinline__ void init(const EnvParams& p, uint32_t env_, uint32_t episode_, int ncalls, int a_idx) {
    j = 0; A = p.A; env = env_; episode = episode_; k0 = p.k0; k1 = p.k1;
    buf[0] = buf[1] = buf[2] = buf[3] = 0;
    base = (int)(threadIdx.x & 63) - a_idx;
    if (SHARE) {
#pragma unroll
      for (int s = 0; s < NC; ++s) {
        mine[s][0] = mine[s][1] = mine[s][2] = mine[s][3] = 0;
        const int c = a_idx + s * A;
        if (c < ncalls) philox4x32_10(env, episode, (uint32_t)c, kStreamReset, k0, k1, mine[s]);
      }
    }
  }
  __device__ __forceinline__ uint32_t draw() {
    if ((j & 3) == 0) {
      const int c = j >> 2;
      if (SHARE) {
        int own = c, slot = 0;  // call c was computed by agent c % A as its call number c / A (uniform values)
#pragma unroll
        for (int q = 0; q < NC; ++q) {
          const bool more = own >= A;
          own -= more ? A : 0;
          slot += more ? 1 : 0;
        }
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          uint32_t v = mine[0][w];
#pragma unroll
          for (int s = 1; s < NC; ++s) v = (slot == s) ? mine[s][w] : v;
          buf[w] = (uint32_t)__shfl((int)v, base + own);
        }
      } else {
        philox4x32_10(env, episode, (uint32_t)c, kStreamReset, k0, k1, buf);
      }
    }
    const int w = j & 3;
    ++j;
    return w == 0 ? buf[0] : (w == 1 ? buf[1] : (w == 2 ? buf[2] : buf[3]));
  }
};

// New episode for one env, entirely in registers (every loop is unrolled over the at most 16 entities, so the
// arrays never leave the register file).  Draw order: A agent levels, A + F cells (agents first), F food levels;
// draw j is word j % 4 of Philox call j / 4 of the stream (env, episode).
template <int CA, int CF, bool SHARE = false>
__device__ __forceinline__ void reset_regs(uint32_t ag[CA], uint32_t fd[CF], const EnvParams& p,
                                           uint32_t env, uint32_t episode, int a_idx = 0) {
  constexpr int kMaxEnt = CA + CF;
  ResetDraws<(2 * kMaxEnt + 3) / 4, SHARE> rd;
  rd.init(p, env, episode, (2 * (p.A + p.F) + 3) >> 2, a_idx);
  auto draw = [&]() -> uint32_t { return rd.draw(); };
  int lvl[CA];
#pragma unroll
  for (int a = 0; a < CA; ++a) lvl[a] = 0;
#pragma unroll
  for (int a = 0; a < CA; ++a)
    if (a < p.A) lvl[a] = 1 + (int)rand_below(draw(), (uint32_t)p.L);
  // cells without replacement: the k-th entity draws r in [0, G*G - k) and takes the r-th free cell (ascending)
  int chosen[kMaxEnt];  // ascending
#pragma unroll
  for (int q = 0; q < kMaxEnt; ++q) chosen[q] = 0x7fffffff;
  const int cells = p.G * p.G, ne = p.A + p.F;
#pragma unroll
  for (int k = 0; k < kMaxEnt; ++k) {
    if (k < ne) {
      int r = (int)rand_below(draw(), (uint32_t)(cells - k));
#pragma unroll
      for (int q = 0; q < kMaxEnt; ++q) r += (q < k && chosen[q] <= r) ? 1 : 0;
      int pos = 0;  // entries smaller than r
#pragma unroll
      for (int q = 0; q < kMaxEnt; ++q) pos += (q < k && chosen[q] < r) ? 1 : 0;
#pragma unroll
      for (int q = kMaxEnt - 1; q >= 1; --q) chosen[q] = (q > pos) ? chosen[q - 1] : chosen[q];
#pragma unroll
      for (int q = 0; q < kMaxEnt; ++q) chosen[q] = (q == pos) ? r : chosen[q];
      const uint32_t row = ((uint32_t)r * p.inv_g20) >> 20, col = (uint32_t)r - row * (uint32_t)p.G;
      const uint32_t cell = row | (col << 8);
#pragma unroll
      for (int a = 0; a < CA; ++a)
        if (k == a && a < p.A) ag[a] = cell | ((uint32_t)lvl[a] << 16);  // slots past A keep their off-grid marker
#pragma unroll
      for (int f = 0; f < CF; ++f)
        if (k == p.A + f) fd[f] = cell;
    }
  }
  // food level in 1..Lsum, Lsum = summed level of the (at most four) strongest agents
  int lsum = 0;
  uint32_t used = 0;
#pragma unroll
  for (int k = 0; k < (CA < 4 ? CA : 4); ++k) {
    int best = 0, bl = 0;
#pragma unroll
    for (int a = 0; a < CA; ++a) {
      const bool better = !((used >> a) & 1u) && lvl[a] > bl;
      bl = better ? lvl[a] : bl;
      best = better ? a : best;
    }
    if (k < p.A) {
      used |= 1u << best;
      lsum += bl;
    }
  }
#pragma unroll
  for (int f = 0; f < CF; ++f)
    if (f < p.F) fd[f] |= (1u + rand_below(draw(), (uint32_t)lsum)) << 16;
}

// The env's entities into registers.  All loads are issued branch-free (clamped indices) so that they are in flight
// together; entries past A / F and inactive lanes are masked afterwards (off-grid cells that never match a cell).
// (Indices are 32-bit: the entity arrays hold at most 8 N < 2^31 elements, and a uniform base plus a 32-bit lane offset
// is an address the hardware forms by itself, where a 64-bit index costs several instructions per access.)
template <int CA, int CF, int KIND>
__device__ __forceinline__ void load_env_state(uint32_t (&ag)[CA], uint32_t (&fd)[CF], const marl_env_state& st,
                                               const EnvParams& p, size_t nn, bool active) {
  const unsigned N = (unsigned)p.N, n = (unsigned)nn;
  uint32_t r8[CA], c8[CA], l8[CA], fr8[CF], fc8[CF], fl8[CF];
#pragma unroll
  for (int b = 0; b < CA; ++b) {
    const unsigned i = (unsigned)min(b, p.A - 1) * N + n;
    r8[b] = st.agent_row[i];
    c8[b] = st.agent_col[i];
    l8[b] = st.agent_lvl[i];
  }
#pragma unroll
  for (int f = 0; f < CF; ++f) {
    const unsigned i = (unsigned)min(f, p.F - 1) * N + n;
    fr8[f] = st.food_row[i];
    fc8[f] = st.food_col[i];
    fl8[f] = st.food_lvl[i];
  }
#pragma unroll
  for (int b = 0; b < CA; ++b) ag[b] = (active && b < p.A) ? (r8[b] | (c8[b] << 8) | (l8[b] << 16)) : 0xffffu;
#pragma unroll
  for (int f = 0; f < CF; ++f)  // foraging: level 0 = absent; warehouse: another off-grid cell, state 0
    fd[f] = (active && f < p.F) ? (fr8[f] | (fc8[f] << 8) | (fl8[f] << 16)) : (KIND == 0 ? 0xffffu : 0xfffeu);
}

// The state back to memory: every lane its own agent, the env's lanes share the food.  In the foraging world the
// levels and the food cells change only when a new episode starts (dn).
template <int CA, int CF, int KIND>
__device__ __forceinline__ void store_env_state(const uint32_t (&ag)[CA], const uint32_t (&fd)[CF], const marl_env_state& st,
                                                const EnvParams& p, size_t n_, int a, bool dn, int t, uint32_t episode) {
  const unsigned N = (unsigned)p.N, n = (unsigned)n_;
  const bool all = dn || KIND != 0;
  uint32_t me = 0;
#pragma unroll
  for (int b = 0; b < CA; ++b) me = (b == a) ? ag[b] : me;
  const unsigned ia = (unsigned)a * N + n;
  st.agent_row[ia] = (uint8_t)e_row(me);
  st.agent_col[ia] = (uint8_t)e_col(me);
  if (all) st.agent_lvl[ia] = (uint8_t)e_lvl(me);
#pragma unroll
  for (int f = 0; f < CF; ++f)
    if (f < p.F && (f % p.A) == a) {
      const unsigned i = (unsigned)f * N + n;
      st.food_lvl[i] = (uint8_t)e_lvl(fd[f]);
      if (all) {
        st.food_row[i] = (uint8_t)e_row(fd[f]);
        st.food_col[i] = (uint8_t)e_col(fd[f]);
      }
    }
  if (a == 0) {
    st.t_in_ep[n] = t;
    st.episode_id[n] = episode;
  }
}

// The transitions run in one lane per agent, a chain of instructions that nothing covers where a wavefront holds all environments of its workgroup
// (the rollout kernels), so they are written for few instructions: cells are compared as 16 bits, several comparisons at a time (the smallest of some
// exclusive ors is zero where one of them is), and a distance is one sum of absolute differences of bytes.
// In cycles of a step of ten environments of three agents (five-wide windows): the transition 3870 -> 2250; the window, with 16-byte stores and a reload of a spilled
// address gone from among them, 2810 -> 2300.
constexpr uint32_t kNoCell = 0xfffeu;  // no entity's, and next to none that counts
// The cell an agent's action leads to: 16 bits, the agent's own for actions that do not move; inside: it is in the grid.
__device__ __forceinline__ uint32_t target_cell(uint32_t agent, int action, int G, bool& inside) {
  const int shift = (uint32_t)action < 6u ? 2 * action : 0;
  const int dr = __builtin_amdgcn_sbfe(0x1c, shift, 2), dc = __builtin_amdgcn_sbfe(0x1c0, shift, 2);  // -1, 0, 1: rows of actions 1 and 2, columns of 3 and 4
  const uint32_t nr = (agent & 0xffu) + dr, nc = (agent >> 8 & 0xffu) + dc;
  inside = max(nr, nc) < (uint32_t)G;
  return nr | nc << 8;
}
template <int N>
__device__ __forceinline__ bool any_equal(const uint32_t (&cells)[N], uint32_t cell, int except = -1) {
  uint32_t m = 0xffffffffu;
#pragma unroll
  for (int i = 0; i < N; ++i)
    if (i != except) m = min(m, cells[i] ^ cell);
  return m == 0;
}
__device__ __forceinline__ bool next_to(uint32_t a, uint32_t b) { return __builtin_amdgcn_sad_u8(a, b, 0u) == 1u; }

// One transition of the foraging world for the lane of agent `a` of env `env`: act[] holds the actions of all agents of
// the env, ag / fd the start-of-step entities.  Leaves the post-step (after an auto-reset: the new episode's) entities,
// step count and episode id in place; rew = this agent's reward, dn = the env finished its episode in this step.
template <int CA, int CF>
__device__ __forceinline__ void forage_transition(uint32_t (&ag)[CA], uint32_t (&fd)[CF], const int (&act)[CA], int a,
                                                  bool active, const EnvParams& p, uint32_t env, int& t,
                                                  uint32_t& episode, float& rew_out, bool& dn_out) {
  uint32_t at[CA], food[CF], load[CA];  // cells; the levels of the agents that load
#pragma unroll
  for (int b = 0; b < CA; ++b) {
    at[b] = ag[b] & 0xffffu;
    load[b] = act[b] == 5 ? ag[b] >> 16 : 0u;
  }
#pragma unroll
  for (int f = 0; f < CF; ++f) food[f] = fd[f] >> 16 != 0 ? fd[f] & 0xffffu : kNoCell;
  // ---- targets of every agent against the start-of-step state (an agent that does not move finds itself in its way)
  uint32_t tgt[CA];  // target cell (row | col << 8), 0xffff when the agent does not move
  bool ok[CA];
#pragma unroll
  for (int b = 0; b < CA; ++b) {
    const uint32_t cell = target_cell(at[b], act[b], p.G, ok[b]);
    ok[b] = ok[b] && !any_equal(at, cell) && !any_equal(food, cell);
    tgt[b] = ok[b] ? cell : 0xffffu;
  }
  // ---- cooperative loading: summed level of the adjacent loaders of each food
  float rew = 0.f;
  bool any_food = false, any_got = false, got[CF];
  uint32_t sum[CF];
#pragma unroll
  for (int f = 0; f < CF; ++f) {
    const uint32_t level = fd[f] >> 16;
    sum[f] = 0;
#pragma unroll
    for (int b = 0; b < CA; ++b) sum[f] += next_to(at[b], food[f]) ? load[b] : 0u;
    got[f] = level != 0 && sum[f] >= level;
    any_got = any_got || got[f];
    any_food = any_food || (level != 0 && !got[f]);
  }
  if (any_got) {
    uint32_t mine = 0, my_load = 0;
#pragma unroll
    for (int b = 0; b < CA; ++b) {
      mine = (b == a) ? ag[b] : mine;
      my_load = (b == a) ? load[b] : my_load;
    }
#pragma unroll
    for (int f = 0; f < CF; ++f) {
      if (got[f]) {
        if (my_load != 0 && next_to(mine & 0xffffu, food[f])) rew += __fdiv_rn((float)((fd[f] >> 16) * my_load), (float)sum[f]);
        fd[f] &= 0xffffu;  // collected: level 0
      }
    }
  }
  // ---- movement: two or more valid movers onto one cell all stay
#pragma unroll
  for (int b = 0; b < CA; ++b) {
    const bool go = ok[b] && !any_equal(tgt, tgt[b], b);
    ag[b] = go ? ((ag[b] & 0xff0000u) | tgt[b]) : ag[b];
  }
  // ---- termination
  t += 1;
  const bool dn = active && (!any_food || t == p.cap);
  // ---- auto-reset: every lane of a finished env re-seeds it in its own registers (same result in each)
  if (dn) {
    episode += 1;
    reset_regs<CA, CF, true>(ag, fd, p, env, episode, a);
    t = 0;
  }
  rew_out = rew;
  dn_out = dn;
}

// One channel of one cell of an observation window, as fp32 or as bf16.  Every value a window can hold -- a level of eight
// bits, 0.5, 1, 2 -- is exact in bf16: its lower 16 bits are zero.
__device__ __forceinline__ void paint_cell(float& o, float v) { o = v; }
__device__ __forceinline__ void paint_cell(bf16_t& o, float v) { o = (bf16_t)(__float_as_uint(v) >> 16); }

// The background of a window: channel 2 of cell (y, x) is value(y, x), the other two are zero.  WIDE: w is 16-byte aligned and the elements up to the next
// multiple of 16 bytes belong to the window's row as zeros: 16-byte stores.
template <int V, bool WIDE, typename T, class F>
__device__ __forceinline__ void paint_background(T* w, F value) {
  constexpr int D = 3 * V * V, PER = 16 / (int)sizeof(T);
  if constexpr (!WIDE) {
#pragma unroll
    for (int c = 0; c < V * V; ++c) {
      paint_cell(w[3 * c], 0.f);
      paint_cell(w[3 * c + 1], 0.f);
      paint_cell(w[3 * c + 2], value(c / V, c % V));
    }
  } else {
#pragma unroll
    for (int q = 0; q < (D + PER - 1) / PER; ++q) {
      uint32_t word[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        word[k] = 0u;
#pragma unroll
        for (int j = 0; j < PER / 4; ++j) {
          const int e = q * PER + k * (PER / 4) + j;
          if (e < D && e % 3 == 2) {
            const uint32_t v = __float_as_uint(value(e / 3 / V, e / 3 % V));  // its lower half is zero (paint_cell)
            word[k] = PER == 4 || j == 1 ? v : v >> 16;                       // at most one of a word's two
          }
        }
      }
      *reinterpret_cast<uint4*>(w + q * PER) = make_uint4(word[0], word[1], word[2], word[3]);
    }
  }
}
// Position of an entity in the window whose upper left cell is (r, c); false: outside.
template <int V>
__device__ __forceinline__ bool window_cell(uint32_t e, int r, int c, int& i) {
  const uint32_t y = (uint32_t)(e_row(e) - r), x = (uint32_t)(e_col(e) - c);
  i = 3 * (int)(y * V + x);
  return max(y, x) < (uint32_t)V;
}
template <int CA>
__device__ __forceinline__ uint32_t own_agent(const uint32_t (&ag)[CA], int a) {
  uint32_t me = 0;
#pragma unroll
  for (int b = 0; b < CA; ++b) me = (b == a) ? ag[b] : me;
  return me;
}

// The lane's V x V x 3 window into w[0 .. 3 V V): walls and zeros first, then the entities that fall inside it.  (Slots past A and F lie off the grid,
// absent food has no level.)
template <int V, int CA, int CF, bool WIDE, typename T>
__device__ __forceinline__ void forage_paint(T* w, const uint32_t (&ag)[CA], const uint32_t (&fd)[CF], int a,
                                             const EnvParams& p) {
  constexpr int h = (V - 1) / 2;
  const uint32_t me = own_agent(ag, a);
  const int r0 = e_row(me) - h, c0 = e_col(me) - h;
  float wr[V], wc[V];
#pragma unroll
  for (int i = 0; i < V; ++i) {
    wr[i] = (uint32_t)(r0 + i) >= (uint32_t)p.G ? 1.f : 0.f;
    wc[i] = (uint32_t)(c0 + i) >= (uint32_t)p.G ? 1.f : 0.f;
  }
  paint_background<V, WIDE>(w, [&](int y, int x) { return fmaxf(wr[y], wc[x]); });
#pragma unroll
  for (int b = 0; b < CA; ++b) {
    int i;
    if (window_cell<V>(ag[b], r0, c0, i)) paint_cell(w[i], (float)e_lvl(ag[b]));
  }
#pragma unroll
  for (int f = 0; f < CF; ++f) {
    int i;
    if (window_cell<V>(fd[f], r0, c0, i) && e_lvl(fd[f]) != 0) paint_cell(w[i + 1], (float)e_lvl(fd[f]));
  }
}

__device__ __forceinline__ bool wh_goal(int G, int r, int c) { return r == G - 1 && (c == G / 2 - 1 || c == G / 2); }

// New episode: A + F distinct cells (robots first), then L requested shelves.  Draw j is word j % 4 of Philox
// call j / 4 of the stream (env, episode).
template <int CA, int CF, bool SHARE = false>
__device__ __forceinline__ void wh_reset_regs(uint32_t ag[CA], uint32_t fd[CF], const EnvParams& p, uint32_t env,
                                              uint32_t episode, int a_idx = 0) {
  constexpr int kMaxEnt = CA + CF;
  ResetDraws<(kMaxEnt + CF + 3) / 4, SHARE> rd;
  rd.init(p, env, episode, (p.A + p.F + p.L + 3) >> 2, a_idx);
  auto draw = [&]() -> uint32_t { return rd.draw(); };
  int chosen[kMaxEnt];  // ascending
#pragma unroll
  for (int q = 0; q < kMaxEnt; ++q) chosen[q] = 0x7fffffff;
  const int cells = p.G * p.G, ne = p.A + p.F;
#pragma unroll
  for (int k = 0; k < kMaxEnt; ++k) {
    if (k < ne) {
      int r = (int)rand_below(draw(), (uint32_t)(cells - k));
#pragma unroll
      for (int q = 0; q < kMaxEnt; ++q) r += (q < k && chosen[q] <= r) ? 1 : 0;
      int pos = 0;
#pragma unroll
      for (int q = 0; q < kMaxEnt; ++q) pos += (q < k && chosen[q] < r) ? 1 : 0;
#pragma unroll
      for (int q = kMaxEnt - 1; q >= 1; --q) chosen[q] = (q > pos) ? chosen[q - 1] : chosen[q];
#pragma unroll
      for (int q = 0; q < kMaxEnt; ++q) chosen[q] = (q == pos) ? r : chosen[q];
      const uint32_t row = ((uint32_t)r * p.inv_g20) >> 20, col = (uint32_t)r - row * (uint32_t)p.G;
      const uint32_t cell = row | (col << 8);
#pragma unroll
      for (int a = 0; a < CA; ++a)
        if (k == a && a < p.A) ag[a] = cell;  // nothing carried; slots past A keep their off-grid marker
#pragma unroll
      for (int f = 0; f < CF; ++f)
        if (k == p.A + f) fd[f] = cell | (1u << 16);  // idle
    }
  }
#pragma unroll
  for (int q = 0; q < CF; ++q) {
    if (q < p.L) {
      int r = (int)rand_below(draw(), (uint32_t)(p.F - q));
#pragma unroll
      for (int f = 0; f < CF; ++f) {
        const bool idle = f < p.F && e_lvl(fd[f]) == 1;
        if (idle && r == 0) fd[f] = (fd[f] & 0xffffu) | (2u << 16);
        r -= idle ? 1 : 0;  // after the hit r is negative and nothing else matches
      }
    }
  }
}

// One transition of the warehouse world, arguments as forage_transition.
template <int CA, int CF>
__device__ __forceinline__ void wh_transition(uint32_t (&ag)[CA], uint32_t (&fd)[CF], const int (&act)[CA], int a,
                                              bool active, const EnvParams& p, uint32_t env, int& t, uint32_t& episode,
                                              float& rew_out, bool& dn_out) {
  const uint32_t n = env;
  // ---- targets against the start-of-step state
  uint32_t at[CA], shelf[CF];  // cells
#pragma unroll
  for (int b = 0; b < CA; ++b) at[b] = ag[b] & 0xffffu;
#pragma unroll
  for (int f = 0; f < CF; ++f) shelf[f] = fd[f] & 0xffffu;
  uint32_t tgt[CA];  // target cell, 0xffff when the robot does not move
  bool ok[CA], collided = false;
#pragma unroll
  for (int b = 0; b < CA; ++b) {
    const uint32_t cell = target_cell(at[b], act[b], p.G, ok[b]);
    ok[b] = ok[b] && cell != at[b];
    const bool hit = any_equal(at, cell);
    collided = collided || (ok[b] && hit);
    ok[b] = ok[b] && !hit && !(e_lvl(ag[b]) != 0 && any_equal(shelf, cell));
    tgt[b] = ok[b] ? cell : 0xffffu;
  }
  // ---- contested cells; movement, carried shelves with their robots
  uint32_t moved[CA];
#pragma unroll
  for (int b = 0; b < CA; ++b) {
    const bool contested = any_equal(tgt, tgt[b], b);
    collided = collided || (ok[b] && contested);
    moved[b] = ok[b] && !contested ? ((ag[b] & 0xff0000u) | tgt[b]) : ag[b];
  }
  uint32_t fd0[CF];  // start-of-step shelves, for the toggle
#pragma unroll
  for (int f = 0; f < CF; ++f) fd0[f] = fd[f];
#pragma unroll
  for (int b = 0; b < CA; ++b) {
    const int cy = e_lvl(ag[b]);
#pragma unroll
    for (int f = 0; f < CF; ++f)
      if (cy == f + 1) fd[f] = (fd[f] & 0xff0000u) | (moved[b] & 0xffffu);
  }
  // ---- toggle (togglers have not moved)
  uint32_t carried_mask = 0;
#pragma unroll
  for (int b = 0; b < CA; ++b) carried_mask |= e_lvl(ag[b]) != 0 ? (1u << (e_lvl(ag[b]) - 1)) : 0u;
#pragma unroll
  for (int b = 0; b < CA; ++b) {
    if (b < p.A && act[b] == 5) {
      uint32_t cy = 0;
      if (e_lvl(ag[b]) == 0) {
#pragma unroll
        for (int f = 0; f < CF; ++f)
          if ((fd0[f] & 0xffffu) == (ag[b] & 0xffffu) && !((carried_mask >> f) & 1u)) cy = (uint32_t)(f + 1);
      }
      moved[b] = (moved[b] & 0xffffu) | (cy << 16);
    }
  }
#pragma unroll
  for (int b = 0; b < CA; ++b) ag[b] = moved[b];
  // ---- delivery, robots in ascending index
  float rew = 0.f;
  uint32_t words[4] = {0, 0, 0, 0};
  int ordinal = 0;
#pragma unroll
  for (int b = 0; b < CA; ++b) {
    const int cy = e_lvl(ag[b]);
    bool deliver = false;
    int fsel = 0;
#pragma unroll
    for (int f = 0; f < CF; ++f) {
      const bool mine = cy == f + 1 && e_lvl(fd[f]) == 2;
      deliver = deliver || mine;
      fsel = mine ? f : fsel;
    }
    deliver = deliver && b < p.A && wh_goal(p.G, e_row(ag[b]), e_col(ag[b]));
    if (deliver) {
      if (b == a) rew = 1.0f;
      int n_cand = 0;
#pragma unroll
      for (int f = 0; f < CF; ++f) {
        if (f == fsel) fd[f] = (fd[f] & 0xffffu) | (1u << 16);
        n_cand += (f < p.F && f != fsel && e_lvl(fd[f]) == 1) ? 1 : 0;
      }
      if ((ordinal & 3) == 0) philox4x32_10((uint32_t)n, episode, (uint32_t)t * 2u + (uint32_t)(ordinal >> 2), kStreamRequest, p.k0, p.k1, words);
      const int w = ordinal & 3;
      const uint32_t word = w == 0 ? words[0] : (w == 1 ? words[1] : (w == 2 ? words[2] : words[3]));
      if (n_cand == 0) {
#pragma unroll
        for (int f = 0; f < CF; ++f)
          if (f == fsel) fd[f] = (fd[f] & 0xffffu) | (2u << 16);
      } else {
        int r = (int)rand_below(word, (uint32_t)n_cand);
#pragma unroll
        for (int f = 0; f < CF; ++f) {
          const bool cand = f < p.F && f != fsel && e_lvl(fd[f]) == 1;
          if (cand && r == 0) fd[f] = (fd[f] & 0xffffu) | (2u << 16);
          r -= cand ? 1 : 0;
        }
      }
      ++ordinal;
    }
  }
  // ---- termination, auto-reset
  t += 1;
  const bool dn = active && (t == p.cap || (p.kind == 2 && collided));
  if (dn) {
    episode += 1;
    wh_reset_regs<CA, CF, true>(ag, fd, p, env, episode, a);
    t = 0;
  }
  rew_out = rew;
  dn_out = dn;
}

// (The largest state among the shelves of one cell is painted: a carried shelf may stand over another one.)
template <int V, int CA, int CF, bool WIDE, typename T>
__device__ __forceinline__ void wh_paint(T* w, const uint32_t (&ag)[CA], const uint32_t (&fd)[CF], int a,
                                         const EnvParams& p) {
  constexpr int h = (V - 1) / 2;
  const uint32_t me = own_agent(ag, a);
  const int r0 = e_row(me) - h, c0 = e_col(me) - h;
  float wr[V], wc[V], gr[V], gc[V];  // walls 1; goals where both are 0.5
#pragma unroll
  for (int i = 0; i < V; ++i) {
    wr[i] = (uint32_t)(r0 + i) >= (uint32_t)p.G ? 1.f : 0.f;
    wc[i] = (uint32_t)(c0 + i) >= (uint32_t)p.G ? 1.f : 0.f;
    gr[i] = r0 + i == p.G - 1 ? 0.5f : 0.f;
    gc[i] = c0 + i == p.G / 2 - 1 || c0 + i == p.G / 2 ? 0.5f : 0.f;
  }
  paint_background<V, WIDE>(w, [&](int y, int x) { return fmaxf(fmaxf(wr[y], wc[x]), fminf(gr[y], gc[x])); });
#pragma unroll
  for (int b = 0; b < CA; ++b) {
    int i;
    if (window_cell<V>(ag[b], r0, c0, i)) paint_cell(w[i], e_lvl(ag[b]) != 0 ? 2.f : 1.f);
  }
#pragma unroll
  for (int f = 0; f < CF; ++f) {
    int i, level = e_lvl(fd[f]);
#pragma unroll
    for (int g = 0; g < f; ++g) level = (fd[g] & 0xffffu) == (fd[f] & 0xffffu) ? max(level, e_lvl(fd[g])) : level;
    if (window_cell<V>(fd[f], r0, c0, i)) paint_cell(w[i + 1], (float)level);
  }
}

inline EnvParams env_params(const marl_config& c) {
  EnvParams p;
  p.G = c.grid; p.A = c.n_agents; p.F = c.n_food; p.L = c.max_level; p.cap = c.episode_cap; p.N = c.n_envs;
  p.kind = c.env_kind;
  p.k0 = (uint32_t)(c.seed & 0xffffffffu);
  p.k1 = (uint32_t)(c.seed >> 32);
  p.inv_g20 = ((1u << 20) + (uint32_t)c.grid - 1u) / (uint32_t)c.grid;
  return p;
}

}  // namespace marl
