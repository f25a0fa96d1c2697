// faco_construct.hpp -- focused construction (Alg. 2's inner loop) and the
// nearest-neighbour tour of the initial solution (included by
// faco_kernels.hpp).
//
// An ant works in SOURCE POSITIONS: a city is known by its position p in the
// source tour, and the visited set is a bitmap over positions (LDS).  Where an
// ant follows or copies the source it then visits a run of consecutive
// positions, so a run is marked a word at a time and its end is found by
// scanning words; the Eq. (1) rows are stored by source position with the
// candidates' source positions, so a step needs two tables (weight, position)
// and no city number.  With a bitmap over cities each copied city cost an LDS
// atomic and each step read two more tables (city, cost).  Windows are bound
// by their instructions (1400 a lane before, 800 now): per ant 148 -> 96 us at
// 20k cities (26 windows), 466 -> 358 us at 100k (52); at 200k windows 196 ->
// 146 us, and the pheromone pass, which writes two tables fewer, 45 -> 28 us.
#pragma once

// ===================================================================== //
// Nearest unvisited city by (squared distance, original number).  The cities
// are indexed by source position (SRC) or by label (the nearest-neighbour
// tour); either way 32 consecutive indexes are close in the plane and have a
// bounding box.  Lane l of wave w scans bitmap words w * 64 + l, + 64 TW, ...;
// fully visited words and words whose box lies beyond a bound are skipped.
// Each wave leaves its (distance, index) minimum in LDS (TW > 1).
// ===================================================================== //
template <bool SRC>
struct NearView {
  const int2 *xy;
  const int4 *box;
  const Inst &I;
  FACO_DEV NearView(const Inst &I_) : xy(SRC ? I_.src_xy : I_.xy), box(SRC ? I_.sbox : I_.wbox), I(I_) {}
  FACO_DEV int orig(int j) const { return I.orig_of[SRC ? I.src_route[j] : j]; }
};

template <bool SRC, int TW>
FACO_DEV void nearest_part(const Inst &I, int u, int w, const uint32_t *vis, TeamLds *tl,
                           int64_t &md, int &mj) {
  const int lane = lane_id();
  const NearView<SRC> T(I);
  const int2 xu = T.xy[u];
  const int W = (I.n + 31) >> 5;
  auto free_word = [&](int wi) -> uint32_t {
    if (wi >= W) return 0u;
    uint32_t f = ~vis[wi];
    const int rem = I.n - wi * 32;
    if (rem < 32) f &= (1u << rem) - 1u;
    return f;
  };
  // A bound first: the nearest of the first unvisited cities of the TW 64
  // bitmap words around u's (neighbouring indexes are close in the plane).  A
  // word whose cities' bounding box lies farther than the bound cannot hold
  // the nearest city (nor one tied with it) and is skipped.
  int64_t ub = INT64_MAX;
  {
    constexpr int span = TW * kWave;
    int lo = (u >> 5) - span / 2;
    lo = lo > W - span ? W - span : lo;
    lo = lo < 0 ? 0 : lo;
    const int wi = lo + w * kWave + lane;
    const uint32_t f = free_word(wi);
    if (f) ub = (int64_t)sqd_u64(xu, T.xy[wi * 32 + __builtin_ctz(f)]);
  }
  ub = wave_min_i64(ub);
  if (TW > 1) {
    if (lane == 0) tl->ub[w] = ub;
    team_sync();
    ub = wave_min_i64(lane < TW ? tl->ub[lane] : INT64_MAX);
  }
  // distances only; equal distances are settled by original number below.
  // Lane l of wave w takes words w 64 + l + i TW 64, i = 0, 1, ..., 32 at a
  // time: their boxes are tested with the loads in flight together, then the
  // unvisited cities of the kept words are taken kNearBatch at a time, so that
  // their coordinate loads are in flight together too.
  constexpr int kNearBatch = 8;
  constexpr int stride = TW * kWave;
  int64_t bd = INT64_MAX;
  int bj = 0x7fffffff;
  bool tie = false;
  for (int g0 = w * kWave + lane; g0 < W; g0 += 32 * stride) {
    uint32_t keep = 0u;
    for (int k0 = 0; k0 < 32; k0 += 8) {
      int4 bx[8];
      bool has[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const int wk = g0 + (k0 + k) * stride;
        has[k] = free_word(wk) != 0u;
        bx[k] = has[k] ? T.box[wk] : make_int4(0, 0, 0, 0);
      }
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        if (has[k]) {
          const int64_t dx = xu.x < bx[k].x ? (int64_t)bx[k].x - xu.x
                                            : (xu.x > bx[k].z ? (int64_t)xu.x - bx[k].z : 0);
          const int64_t dy = xu.y < bx[k].y ? (int64_t)bx[k].y - xu.y
                                            : (xu.y > bx[k].w ? (int64_t)xu.y - bx[k].w : 0);
          if (dx * dx + dy * dy <= ub) keep |= 1u << (k0 + k);
        }
      }
      if (g0 + (k0 + 8) * stride >= W) break;
    }
    int wi = 0;
    uint32_t fb = 0u;
    for (;;) {
      int jb[kNearBatch];
      bool vb[kNearBatch];
#pragma unroll
      for (int k = 0; k < kNearBatch; ++k) {
        while (fb == 0u && keep != 0u) {
          wi = g0 + __builtin_ctz(keep) * stride;
          keep &= keep - 1u;
          fb = free_word(wi);
        }
        vb[k] = fb != 0u;
        jb[k] = vb[k] ? wi * 32 + __builtin_ctz(fb) : u;
        fb &= fb - 1u;
      }
      if (!vb[0]) break;
      int2 xb[kNearBatch];
#pragma unroll
      for (int k = 0; k < kNearBatch; ++k) xb[k] = T.xy[jb[k]];
#pragma unroll
      for (int k = 0; k < kNearBatch; ++k) {
        if (vb[k]) {
          const int64_t d = (int64_t)sqd_u64(xu, xb[k]);
          if (d < bd) {
            bd = d;
            bj = jb[k];
            tie = false;
          } else if (d == bd) {
            tie = true;
          }
        }
      }
    }
  }
  md = wave_min_i64(bd);
  int mo = 0x7fffffff;
  mj = 0x7fffffff;
  if (md != INT64_MAX) {
    const uint64_t at_min = ballot(bd == md);
    if (__builtin_popcountll(at_min) == 1 && !ballot(bd == md && tie)) {
      mj = readlane_i(bj, ctz64(at_min));
      mo = uniform_i(T.orig(mj));
    } else {
      // several cities at distance md: the smallest original number
      int bo = 0x7fffffff, bj2 = 0x7fffffff;
      for (int wi = w * kWave + lane; wi < W; wi += TW * kWave) {
        uint32_t free_bits = free_word(wi);
        while (free_bits) {
          const int j = wi * 32 + __builtin_ctz(free_bits);
          free_bits &= free_bits - 1;
          if ((int64_t)sqd_u64(xu, T.xy[j]) == md) {
            const int o = T.orig(j);
            if (o < bo) {
              bo = o;
              bj2 = j;
            }
          }
        }
      }
      mo = wave_min_i32(bo);
      mj = wave_min_i32(bo == mo ? bj2 : 0x7fffffff);
    }
  }
  if (TW > 1 && lane == 0) {
    tl->part[w] = md;
    tl->f[w] = mo;
    tl->f[kMaxTeam + w] = mj;
  }
}

// Leader side: the whole team's nearest unvisited index.  Uniform result.
template <bool SRC, int TW>
FACO_DEV int nearest(const Inst &I, int u, const uint32_t *vis, TeamLds *tl) {
  const int lane = lane_id();
  int64_t md;
  int mj;
  if (TW == 1) {
    nearest_part<SRC, 1>(I, u, 0, vis, tl, md, mj);
    return mj;
  }
  team_post(tl, SRC ? OP_NEAREST : OP_NEAREST_LABEL, u);
  nearest_part<SRC, TW>(I, u, 0, vis, tl, md, mj);
  team_sync();
  const int64_t d = lane < TW ? tl->part[lane] : INT64_MAX;
  const int o = lane < TW ? tl->f[lane] : 0x7fffffff;
  const int j = lane < TW ? tl->f[kMaxTeam + lane] : 0x7fffffff;
  const int64_t dmin = wave_min_i64(d);
  const int omin = wave_min_i32(d == dmin ? o : 0x7fffffff);
  return uniform_i(wave_min_i32(d == dmin && o == omin ? j : 0x7fffffff));
}

// Backup list, then the nearest unvisited city (when no candidate is
// unvisited); u and the result are source positions.
template <int TW>
FACO_DEV int select_fallback(const Inst &I, int pu, const uint32_t *vis, TeamLds *tl,
                             LaneCounters &cnt) {
  const int lane = lane_id();
  const int u = uniform_i(I.src_route[pu]);
  int p = 0;
  bool bu = false;
  if (lane < I.bl) {
    p = I.src_pos[I.bll[(size_t)u * (size_t)I.bl + lane]];
    bu = !bit_get(vis, p);
  }
  const uint64_t bm = ballot(bu);
  if (bm) {
    cnt[CNT_BACKUP]++;
    return readlane_i(p, ctz64(bm));
  }
  // best heuristic value = nearest unvisited city, ties by smaller original number
  cnt[CNT_FALLBACK]++;
  return nearest<true, TW>(I, pu, vis, tl);
}

// ===================================================================== //
// Runs of source positions.
// ===================================================================== //
// Unvisited positions after p in direction dir (+1 or -1) up to the first
// visited one (cyclic; p itself is visited).  A wave scans 2048 positions per
// step.  Uniform result.
FACO_DEV int free_run(const uint32_t *vis, int p, int dir, int n) {
  const int lane = lane_id();
  if (dir > 0) {
    for (int part = 0; part < 2; ++part) {
      const int lo = part ? 0 : p + 1, hi = part ? p + 1 : n;
      for (int w0 = lo >> 5; w0 * 32 < hi; w0 += kWave) {
        const int wi = w0 + lane;
        uint32_t x = wi * 32 < hi ? vis[wi] : 0u;
        if (wi == lo >> 5) x &= ~0u << (lo & 31);
        const uint64_t m = ballot(x != 0u);
        if (m) {
          const int l = ctz64(m);
          const int q = (w0 + l) * 32 + __builtin_ctz((uint32_t)readlane_i((int)x, l));
          return part ? n - 1 - p + q : q - p - 1;
        }
      }
    }
    return n - 1;  // not reached: p is visited
  }
  for (int part = 0; part < 2; ++part) {
    // downward from hi - 1 to lo
    const int hi = part ? n : p, lo = part ? p : 0;
    for (int w0 = (hi - 1) >> 5; hi > 0 && w0 >= lo >> 5; w0 -= kWave) {
      const int wi = w0 - lane;
      uint32_t x = wi >= lo >> 5 ? vis[wi] : 0u;
      if (wi == (hi - 1) >> 5) x &= ~0u >> (31 - ((hi - 1) & 31));
      const uint64_t m = ballot(x != 0u);
      if (m) {
        const int l = ctz64(m);
        const int q = (w0 - l) * 32 + 31 - __builtin_clz((uint32_t)readlane_i((int)x, l));
        return part ? p + n - 1 - q : p - 1 - q;
      }
    }
  }
  return n - 1;
}

// Mark the L consecutive positions from p on (cyclic), words over the lanes.
// One wave; no other wave writes the bitmap meanwhile.
FACO_DEV void mark_run(uint32_t *vis, int p, int L, int n) {
  const int lane = lane_id();
  for (int part = 0; part < 2; ++part) {
    const int lo = part ? 0 : p, hi = part ? p + L - n : (p + L < n ? p + L : n);
    for (int wi = (lo >> 5) + lane; wi * 32 < hi; wi += kWave) {
      uint32_t m = ~0u;
      if (wi == lo >> 5) m &= ~0u << (lo & 31);
      const int rem = hi - wi * 32;
      if (rem < 32) m &= (1u << rem) - 1u;
      vis[wi] |= m;
    }
  }
}

// Append J consecutive source positions, the first at pcur + dir, at tour
// positions k on: wave w's share; the edge costs go to the lanes' sums.  The
// next positions are loaded before the present ones are stored, so a wave
// always has loads in flight (a copy is bound by the latency of what one CU
// keeps in flight: 193k cities in 195 us load-then-store, 8 a lane).
template <int TW>
FACO_DEV void copy_part(const Inst &I, int pcur, int dir, int k, int J, int w, int32_t *route,
                        int32_t *pos, int2 *rxy, int64_t &lane_len) {
  const int n = I.n, lane = lane_id();
  constexpr int CH = 4;  // positions per lane and step
  constexpr int STEP = TW * CH * kWave;
  struct Buf {
    int c[CH], d[CH], x[CH], y[CH];
  };
  auto load = [&](int i0, Buf &B) {
#pragma unroll
    for (int h = 0; h < CH; ++h) {
      const int i = i0 + h * kWave + lane;
      if (i < J) {
        const int q = wrapc(pcur + dir * (i + 1), n);
        B.c[h] = at(I.src_route, q);
        const int2 x = at(I.src_xy, q);
        B.x[h] = x.x;
        B.y[h] = x.y;
        B.d[h] = at(I.src_d, dir > 0 ? (q == 0 ? n - 1 : q - 1) : q);
      }
    }
  };
  auto store = [&](int i0, const Buf &B) {
#pragma unroll
    for (int h = 0; h < CH; ++h) {
      const int i = i0 + h * kWave + lane;
      if (i < J) {
        at(route, k + i) = B.c[h];
        at(rxy, k + i) = make_int2(B.x[h], B.y[h]);
        at(pos, B.c[h]) = k + i;
        lane_len += B.d[h];
      }
    }
  };
  Buf A, B;
  int i0 = w * CH * kWave;
  if (i0 < J) load(i0, A);
  while (i0 < J) {
    if (i0 + STEP < J) load(i0 + STEP, B);
    store(i0, A);
    i0 += STEP;
    if (i0 >= J) break;
    if (i0 + STEP < J) load(i0 + STEP, A);
    store(i0, B);
    i0 += STEP;
  }
}

// Copy-from-source (Alg. 2, reading: forward from pv while unvisited, else
// backward).  Returns the count; pu becomes the last appended position.
template <int TW>
FACO_DEV int copy_from(const Inst &I, int pv, int &k, int &pu, int64_t &lane_len, TeamLds *tl,
                       int32_t *route, int32_t *pos, int2 *rxy, uint32_t *vis) {
  const int n = I.n;
  int dir = 1;
  int J = uniform_i(free_run(vis, pv, 1, n));
  if (J == 0) {
    dir = -1;
    J = uniform_i(free_run(vis, pv, -1, n));
    if (J == 0) return 0;
  }
  // short runs are the leader's alone
  const bool team = TW > 1 && J > 8 * kWave;
  if (team) {
    team_post(tl, OP_COPY, pv, dir, k, J);
    copy_part<TW>(I, pv, dir, k, J, 0, route, pos, rxy, lane_len);
  } else {
    copy_part<1>(I, pv, dir, k, J, 0, route, pos, rxy, lane_len);
  }
  mark_run(vis, dir > 0 ? wrapc(pv + 1, n) : wrapc(pv - J, n), J, n);
  if (team) team_sync();
  wave_fence();
  k += J;
  pu = wrapc(pv + dir * J, n);
  return J;
}

// ===================================================================== //
// Roulette draws.  The draw of a step depends on the step's number only, so a
// team keeps the draws of the coming steps in LDS: the waves that do not
// evaluate a window compute the next ones meanwhile (64 x 64-bit products, a
// third of a window's vector instructions, and only 2 of 5 draws were used
// when every window computed its own).  Ring of kDraws entries; draws of
// steps have - kDraws .. have - 1 are in it.
// ===================================================================== //
FACO_DEV float roulette(const Inst &I, uint64_t t, uint64_t ant, int step) {
  return unit24(philox_word0(I.seed, t, ant, (uint64_t)step, kPurposeRoulette));
}
FACO_DEV void fill_draws(const Inst &I, uint64_t t, uint64_t ant, int step, TeamLds *tl) {
  tl->draws[step & (kDraws - 1)] = roulette(I, t, ant, step);
}

// Leader's draws outside windows: lane j holds the draw of step base + j.
struct Draws {
  int base;  // < 0: none
  float u;
};

// ===================================================================== //
// Speculative source-following window.  Lane g evaluates ACO step `step + g`
// as if the ant had followed the source in direction dir for the previous g
// steps: its current position is pu + dir g, its visited set V + {the next g
// positions}.  The first lane whose choice is not the next source position
// ends the window; its choice is exact because every earlier lane confirmed
// the assumption.  Same draws, same weights, same order as the
// one-step-at-a-time rule.
// ===================================================================== //
struct WinOut {
  int acc;        // steps that followed the source
  int pv;         // choice of step `step + acc` (-2: window ran out, -1: no
                  // candidate is unvisited)
};

// Waves that evaluate a window (64 steps each): one per SIMD of a CU.  A
// window ends at the first step off the source, after 105 steps on average at
// 20k cities and 400 at 100k.
template <int TW>
constexpr int win_waves() { return TW < 4 ? TW : 4; }
template <int TW>
constexpr bool cached_draws() { return TW > win_waves<TW>(); }

// Wave w's part of one window: evaluates steps step + 64 w + lane, then
// appends the accepted steps it evaluated (route, pos, rxy).  The visited
// bits are marked by the caller.
template <int KT, int TW>
FACO_DEV void window_part(const Inst &I, uint64_t t, uint64_t ant, int step, int pu, int dir,
                          int k, int w, int &have, TeamLds *tl, const uint32_t *vis,
                          int32_t *route, int32_t *pos, int2 *rxy, int64_t &lane_len, WinOut &o,
                          int round = 0) {
  constexpr int WW = win_waves<TW>();
  const int n = I.n, K4 = I.ks, lane = lane_id();
  const int g = w * kWave + lane;
  const int valid = n - k < WW * kWave ? n - k : WW * kWave;  // steps left
  int choice = -1, qn = 0, ed = 0, qpos = 0;
  int2 qxy = make_int2(0, 0);
  int F = WW * kWave;
  if (w < WW) {
    // every load below is addressed by source position: one round trip
    const int rpos = wrap_off(pu, dir * g, n);
    qpos = wrap_off(pu, dir * (g + 1), n);
    const int row = (rpos >> 6) * K4 * 64 + (rpos & 63);  // srow(rpos, 0, K4)
    // rows are padded to whole groups of four slots (weight 0, the row's own
    // position, which is visited), so only whole groups are skipped
    int sp[KT];
    float wt[KT];
#pragma unroll
    for (int s0 = 0; s0 < KT; s0 += 4) {
      if (s0 < K4) {
#pragma unroll
        for (int s = s0; s < s0 + 4; ++s) {
          wt[s] = at(I.sw, row + 64 * s);
          sp[s] = at(I.ssp, row + 64 * s);
        }
      }
    }
    qn = at(I.src_route, qpos);
    qxy = at(I.src_xy, qpos);
    ed = at(I.src_d, dir > 0 ? rpos : qpos);
    const float U = cached_draws<TW>() ? tl->draws[(step + g) & (kDraws - 1)]
                                       : roulette(I, t, ant, step + g);
    // positions pu + dir .. pu + dir g are visited at this lane's step: with
    // off = dir (sp - pu), those with off - 1 < g (unsigned); off is taken
    // modulo n only where the window crosses the array's end
    const int dm = dir > 0 ? 0 : -1, c = dir > 0 ? -pu - 1 : pu;
    const bool cross = dir > 0 ? pu + WW * kWave >= n : pu - WW * kWave < 0;
    float P[KT];
    float total = 0.0f;
    uint32_t open = 0u;  // slots not visited
#pragma unroll
    for (int s0 = 0; s0 < KT; s0 += 4) {
      if (s0 < K4) {
        uint32_t word[4];
#pragma unroll
        for (int s = s0; s < s0 + 4; ++s) word[s - s0] = vis[sp[s] >> 5];
#pragma unroll
        for (int s = s0; s < s0 + 4; ++s) {
          int off = (sp[s] ^ dm) + c;
          if (cross) off += off < 0 ? n : 0;
          const bool visited = ((word[s - s0] >> (sp[s] & 31)) & 1u) || (uint32_t)off < (uint32_t)g;
          total = total + (visited ? 0.0f : wt[s]);
          open |= visited ? 0u : 1u << s;
          P[s] = total;
        }
      }
    }
    if (open) {
      const float r = U * total;
      // P ascends, so the first slot above r is the number of slots not above
      int sel = 0;
#pragma unroll
      for (int s0 = 0; s0 < KT; s0 += 4) {
        if (s0 < K4) {
#pragma unroll
          for (int s = s0; s < s0 + 4; ++s) sel += P[s] > r ? 0 : 1;
        }
      }
      if (sel >= K4) sel = 31 - __builtin_clz(open);
#pragma unroll
      for (int s = 0; s < KT; ++s)
        if (s == sel) choice = sp[s];
    }
    const bool match = choice == qpos && g < valid;
    const uint64_t mm = ballot(!match);
    F = mm ? w * kWave + ctz64(mm) : WW * kWave;
  } else if (have < step + 2 * WW * kWave) {
    fill_draws(I, t, ant, have + (w - WW) * kWave + lane, tl);
  }
  if (cached_draws<TW>() && have < step + 2 * WW * kWave) have += (TW - WW) * kWave;
  if (TW > 1) {
    int *f = tl->f + (round & 1) * kMaxTeam;
    if (lane == 0 && w < WW) f[w] = F;
    team_sync();  // every wave's evaluation is done before any append
    F = f[0];
#pragma unroll
    for (int i = 1; i < WW; ++i) F = f[i] < F ? f[i] : F;
    F = uniform_i(F);
  }
  const int acc = F < valid ? F : valid;
  o.acc = acc;
  o.pv = -2;
  if (w < WW) {
    if (g < acc) {
      at(route, k + g) = qn;
      at(rxy, k + g) = qxy;
      at(pos, qn) = k + g;
      lane_len += ed;
    }
    if (acc < valid) {
      if (TW == 1)
        o.pv = readlane_i(choice, acc);
      else if (g == acc)
        tl->res[1] = choice;
    }
  }
  if (TW > 1 && acc < valid) o.pv = 0;  // left in tl->res[1], read after a barrier
}

// A team runs up to kWinRounds windows in one command: while a window is
// followed to its end, the next one starts from where it stopped (every wave
// derives the new start alike).  Wave 0 marks the followed positions between
// barriers.  The followed edges' costs go to the lanes' sums; o.acc is the total.
// The command ends at its last round's barrier.
constexpr int kWinRounds = 32;
template <int KT, int TW>
FACO_DEV void window_rounds(const Inst &I, uint64_t t, uint64_t ant, int step, int pu, int dir,
                            int k, int w, int &have, TeamLds *tl, uint32_t *vis, int32_t *route,
                            int32_t *pos, int2 *rxy, int64_t &lane_len, WinOut &o) {
  constexpr int NW = win_waves<TW>() * kWave;
  const int n = I.n;
  int total = 0;
  if (cached_draws<TW>() && have < step + NW) {
    // the first window, or a restart behind one-step choices
    have = step;
    fill_draws(I, t, ant, have + w * kWave + lane_id(), tl);
    have += TW * kWave;
    team_sync();
  }
  for (int r = 0;; ++r) {
    WinOut q;
    window_part<KT, TW>(I, t, ant, step, pu, dir, k, w, have, tl, vis, route, pos, rxy,
                        lane_len, q, r);
    const int acc = uniform_i(q.acc);
    total += acc;
    if (w == 0 && acc > 0)
      mark_run(vis, dir > 0 ? wrap_off(pu, 1, n) : wrap_off(pu, -acc, n), acc, n);
    const int valid = n - k < NW ? n - k : NW;
    team_sync();  // this window's marks and results are visible
    if (acc < valid || r + 1 >= kWinRounds || k + acc >= n) {
      o = q;
      break;
    }
    pu = wrap_off(pu, dir * acc, n);
    k += acc;
    step += acc;
  }
  o.acc = total;
}

// Leader side of a window (TW > 1: posts it, takes wave 0's share, collects).
template <int KT, int TW>
FACO_DEV WinOut team_window(const Inst &I, uint64_t t, uint64_t ant, int step, int pu, int dir,
                            int k, int &have, TeamLds *tl, uint32_t *vis, int32_t *route,
                            int32_t *pos, int2 *rxy, int64_t &lane_len) {
  WinOut o;
  if (TW == 1) {
    window_part<KT, TW>(I, t, ant, step, pu, dir, k, 0, have, tl, vis, route, pos, rxy, lane_len,
                        o);
    if (o.acc > 0)
      mark_run(vis, dir > 0 ? wrap_off(pu, 1, I.n) : wrap_off(pu, -o.acc, I.n), o.acc, I.n);
    return o;
  }
  if (lane_id() == 0) tl->arg64[0] = t;
  team_post(tl, OP_WINDOW, pu, dir, k, step, have);
  window_rounds<KT, TW>(I, t, ant, step, pu, dir, k, 0, have, tl, vis, route, pos, rxy,
                        lane_len, o);
  o.acc = uniform_i(o.acc);
  have = uniform_i(have);
  o.pv = uniform_i(o.pv) == 0 ? uniform_i(tl->res[1]) : -2;
  return o;
}

// One ACO step from source position pu, lane s = candidate slot s (used once
// new_edges >= m, when every step is followed by a copy).  Returns the chosen
// source position, -1 when no candidate is unvisited.
FACO_DEV int one_step(const Inst &I, uint64_t t, uint64_t ant, int step, int pu,
                      const uint32_t *vis, Draws &D) {
  const int K = I.k, lane = lane_id();
  const bool act = lane < K;
  const size_t row = srow(pu, act ? lane : 0, I.ks);
  const float w = act ? I.sw[row] : 0.0f;
  const int sp = act ? I.ssp[row] : 0;
  const bool unv = act && !bit_get(vis, sp);
  const uint64_t um = ballot(unv);
  if (!um) return -1;
  if (!(D.base >= 0 && step >= D.base && step < D.base + kWave)) {
    D.u = roulette(I, t, ant, step + lane);
    D.base = step;
  }
  const float U = readlane_f(D.u, step - D.base);
  const float wv = unv ? w : 0.0f;
  // cumulative sum in slot order: lane s holds fl(...fl(w_0 + w_1)... + w_s)
  float P = 0.0f;
  for (int j = 0; j < K; ++j) {
    const float wj = readlane_f(wv, j);
    if (j <= lane) P = P + wj;
  }
  const float r = U * readlane_f(P, K - 1);
  const uint64_t sm = ballot(act && P > r);
  return readlane_i(sp, sm ? ctz64(sm) : msb64(um));
}

// ===================================================================== //
// Focused construction.  The checklist is written into ring[0..nchk) with its
// LDS bits set in inq.
//   tk: [5] speculative windows, [6] one-step calls, [7] copies, [8..10] their
//   ticks, [11] ticks in backup/nearest-city choices
// ===================================================================== //
template <int KT, int TW>
FACO_DEV int64_t construct(const Inst &I, uint64_t t, int ant, int32_t *route, int32_t *pos,
                           int2 *rxy, int32_t *ring, uint32_t *vis, uint32_t *inq, TeamLds *tl,
                           int W, int &nchk, LaneCounters &cnt, LaneCounters &tk) {
  const int n = I.n, lane = lane_id();
  for (int w = lane; w < W; w += kWave) {
    vis[w] = 0u;
    inq[w] = 0u;
  }
  wave_fence();
  // start: a uniform draw (original numbers)
  const int r0 = uniform_i(
      I.int_of[uniform_node(philox_word0(I.seed, t, (uint64_t)ant, 0, kPurposeStart), n)]);
  const int2 x0 = I.xy[r0];
  int pu = uniform_i(I.src_pos[r0]);
  if (lane == 0) {
    route[0] = r0;
    pos[r0] = 0;
    rxy[0] = x0;
    bit_set(vis, pu);
  }
  // calc_num_new_edges() (Alg. 2): the constant min_new_edges, or this ant's
  // uniform draw from [min_new_edges, min_new_edges_max]
  int m = I.m;
  if (I.m_hi > I.m)
    m += (int)__umul64hi(philox_word0(I.seed, t, (uint64_t)ant, 0, kPurposeNewEdges),
                         (uint64_t)(I.m_hi - I.m) + 1u);
  m = uniform_i(m);
  int k = 1, new_edges = 0, dir = 1;
  nchk = 0;
  int64_t len = 0, lane_len = 0;  // edge costs: of single steps, of runs by lane
  int step = 0, have = 0;
  Draws D;
  D.base = -1;
  D.u = 0.0f;
  while (k < n) {
    // Loop state is wave-uniform; keep it in scalar registers so that the
    // team barriers below sit in scalar control flow.
    k = uniform_i(k);
    new_edges = uniform_i(new_edges);
    pu = uniform_i(pu);
    dir = uniform_i(dir);
    step = uniform_i(step);
    // Once new_edges >= m every ACO step is followed by a copy, so the
    // window is one step wide.
    const bool single = new_edges >= m;
    int pv;
    const int64_t c0 = fine_ticks();
    if (single) {
      pv = uniform_i(one_step(I, t, (uint64_t)ant, step, pu, vis, D));
      tk[6]++;
      tk[9] += fine_ticks() - c0;
    } else {
      // accepted steps follow the source, appended at k on
      const WinOut o = team_window<KT, TW>(I, t, (uint64_t)ant, step, pu, dir, k, have, tl, vis,
                                           route, pos, rxy, lane_len);
      tk[5]++;
      tk[8] += fine_ticks() - c0;
      const int acc = uniform_i(o.acc);
      pv = uniform_i(o.pv);
      k += acc;
      step += acc;
      pu = wrapc(pu + dir * acc, n);
      wave_fence();
    }
    if (pv == -2) {
      // the whole window followed the source; no step off the path
      pv = pu;
    } else {
      if (pv == -1) {
        const int64_t c1 = fine_ticks();
        pv = uniform_i(select_fallback<TW>(I, pu, vis, tl, cnt));
        tk[11] += fine_ticks() - c1;
      }
      ++step;
      const int v = uniform_i(I.src_route[pv]);
      const int2 xv = I.src_xy[pv];
      len += cost(I.src_xy[pu], xv);
      const int fwd = pu + 1 == n ? 0 : pu + 1, bwd = pu == 0 ? n - 1 : pu - 1;
      const bool fresh = pv != fwd && pv != bwd;  // not a source edge
      if (lane == 0) {
        route[k] = v;
        pos[v] = k;
        rxy[k] = xv;
        bit_set(vis, pv);
        if (fresh) {
          ring[nchk] = v;
          bit_set(inq, v);
        }
      }
      ++k;
      new_edges += fresh ? 1 : 0;
      nchk += fresh ? 1 : 0;
      dir = pv == bwd ? -1 : 1;
    }
    pu = uniform_i(pv);
    new_edges = uniform_i(new_edges);
    k = uniform_i(k);
    dir = uniform_i(dir);
    if (new_edges >= m && k < n) {
      const int64_t c2 = fine_ticks();
      const int app = copy_from<TW>(I, pv, k, pu, lane_len, tl, route, pos, rxy, vis);
      cnt[CNT_COPIED] += app;
      tk[7]++;
      tk[10] += fine_ticks() - c2;
    }
  }
  len += cost(I.src_xy[pu], x0);
  len += wave_sum_i64(lane_len);
  if (TW > 1) {
    // the helpers' sums
    team_post(tl, OP_LENGTH);
    team_sync();
    len += wave_sum_i64(lane > 0 && lane < TW ? tl->part[lane] : 0);
  }
  cnt[CNT_ACO_STEPS] += step;
  cnt[CNT_NEW_EDGES] += new_edges;
  wave_fence();
  return uniform_i64(len);
}

// ===================================================================== //
// Wave 1 of a team while wave 0 builds the nearest-neighbour tour: the rows of
// the candidates of the candidates of the city that wave 0 is at (tl->arg[0])
// are brought into the CU's L1 until wave 0 sets tl->arg[1] (which it does
// before every barrier).  Nothing but time depends on what it reads.  The tour is
// bound by the latency of one candidate row per city; wave 0's own touches of the
// rows ahead held its next load up, as loads return in order.  A build of 1000
// cities went from 1.44 to 1.37 ms, of 20000 from 25.4 to 23.8, of 200000 from
// 381 to 364 ms against touches by wave 0.
// ===================================================================== //
FACO_DEV void greedy_rows(const Inst &I, TeamLds *tl) {
  const int K = I.k, lane = lane_id();
  const int s1 = (lane >> 2) < K ? lane >> 2 : K - 1, s2 = (lane & 3) < K ? lane & 3 : K - 1;
  int last = -1;
  for (;;) {
    if (uniform_i(__hip_atomic_load(&tl->arg[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)))
      return;
    const int u = uniform_i(
        __hip_atomic_load(&tl->arg[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
    if (u == last) {
      __builtin_amdgcn_s_sleep(1);
      continue;
    }
    last = u;
    const int c1 = at(I.cl, u * K + s1);
    const int c2 = at(I.cl, c1 * K + s2);
    const int c3 = at(I.cl, c2 * K + (K >> 1));
    asm volatile("" : : "v"(c3));
  }
}

// ===================================================================== //
// The nearest-neighbour tour from city 0 (initial solution), by labels: first
// unvisited candidate (lists are sorted by distance), else the fallback chain.
// The chain of one step is a candidate row's load and its visited bits.  A load
// is waited for behind every memory operation issued before it, so nothing is
// stored per step (64 cities leave together), and the rows of the next steps are
// brought into the CU's L1 beforehand: by another wave (greedy_rows), or, where
// the ant has one wave only, by touching the rows of the present city's
// candidates after the next row's own load.  A build of 20000 cities went from
// 26.9 to 25.4 ms with one wave's touches and without the stores.  Positions,
// coordinates and the length follow in one pass over the tour.
// ===================================================================== //
template <int TW>
FACO_DEV void greedy_stop(TeamLds *tl) {
  if (TW == 1) return;
  if (lane_id() == 0)
    __hip_atomic_store(&tl->arg[1], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  team_sync();
}

template <int TW>
FACO_DEV int64_t construct_greedy(const Inst &I, int32_t *route, int32_t *pos, int2 *rxy,
                                  uint32_t *vis, uint32_t *inq, TeamLds *tl, int W,
                                  LaneCounters &cnt) {
  const int n = I.n, K = I.k, lane = lane_id();
  for (int w = lane; w < W; w += kWave) {
    vis[w] = 0u;
    inq[w] = 0u;
  }
  wave_fence();
  int u = uniform_i(I.int_of[0]);
  if (lane == 0) bit_set(vis, u);
  int held = u;            // lane l: city 64 j + l of the tour, j the present group
  int c = lane < K ? at(I.cl, u * K + lane) : 0;
  int touch = 0, sink = 0;
  if (TW > 1) team_post(tl, OP_GREEDY, u, 0);
  for (int k = 1; k < n; k = uniform_i(k + 1)) {
    const uint64_t um = ballot(lane < K && !bit_get(vis, c));
    int v;
    if (um) {
      v = readlane_i(c, ctz64(um));
    } else {
      int b = 0;
      bool bu = false;
      if (lane < I.bl) {
        b = I.bll[(size_t)u * (size_t)I.bl + lane];
        bu = !bit_get(vis, b);
      }
      const uint64_t bm = ballot(bu);
      if (bm) {
        cnt[CNT_BACKUP]++;
        v = readlane_i(b, ctz64(bm));
      } else {
        cnt[CNT_FALLBACK]++;
        greedy_stop<TW>(tl);
        v = nearest<false, TW>(I, u, vis, tl);
        if (TW > 1) team_post(tl, OP_GREEDY, v, 0);
      }
    }
    u = uniform_i(v);
    const int row = c;
    if (lane < K) c = at(I.cl, u * K + lane);
    if (lane == 0) {
      bit_set(vis, u);
      if (TW > 1)
        __hip_atomic_store(&tl->arg[0], u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    if (TW == 1) {
      sink ^= touch;
      if (lane < K) touch = at(I.cl, row * K + (K >> 1));
    }
    if ((k & (kWave - 1)) == 0) at(route, k - kWave + lane) = held;
    held = lane == (k & (kWave - 1)) ? u : held;
  }
  greedy_stop<TW>(tl);
  {
    const int first = (n - 1) & ~(kWave - 1);
    if (first + lane < n) at(route, first + lane) = held;
  }
  // (never so: city numbers are below 2^18)
  if (sink == -1) bit_set(inq, 0);
  wave_fence();
  int64_t len = 0;
  for (int i0 = 0; i0 < n; i0 += 4 * kWave) {
    int c[4], d[4];
    int2 xc[4], xd[4];
#pragma unroll
    for (int h = 0; h < 4; ++h) {
      const int i = i0 + h * kWave + lane;
      c[h] = i < n ? at(route, i) : 0;
      d[h] = i < n ? at(route, i + 1 == n ? 0 : i + 1) : 0;
    }
#pragma unroll
    for (int h = 0; h < 4; ++h) {
      xc[h] = at(I.xy, c[h]);
      xd[h] = at(I.xy, d[h]);
    }
#pragma unroll
    for (int h = 0; h < 4; ++h) {
      const int i = i0 + h * kWave + lane;
      if (i < n) {
        at(rxy, i) = xc[h];
        at(pos, c[h]) = i;
        len += cost(xc[h], xd[h]);
      }
    }
  }
  wave_fence();
  return wave_sum_i64(len);
}
